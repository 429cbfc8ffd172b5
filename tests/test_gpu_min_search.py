"""Subtree ends and chain parents across the groups of the range minima (16 positions, then
64 entries a level): subtrees of one path up to thousands of them, at every offset."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, csr, gpu_tree, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 5])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 255, 1023, 1024, 1025, 4095, 4097, 66000])
def test_subtrees_of_every_size(n, m):
    torch_or_skip()
    # path k: the binary digits of k (so subtrees of 2, 4, 8, ... paths), under one frame
    # more for the second half (a chain parent far back), then a leaf of its own
    bits = max(1, (n - 1).bit_length())
    k = np.arange(n)
    digits = (k[:, None] >> np.arange(bits - 1, -1, -1)) & 1
    paths = [[9] + [int(x) for x in row] + [100 + i % 7] for i, row in enumerate(digits)]
    paths += [[9], [9, 0], [10]]
    rng = np.random.default_rng(n)
    paths = [paths[i] for i in rng.permutation(len(paths))]
    o, f = csr(paths)
    w = rng.integers(0, 1 << 62, (len(paths), m), dtype=np.uint64)
    assert_same(gpu_tree(o, f, w), oracle.build_tree(o, f, w))

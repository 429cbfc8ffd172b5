"""Neighbouring paths that part at, before and after the edges of the LCP kernel's steps
(eight lanes compare 64 frames at a time, two pieces of 32, four frames of each a lane)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, csr, gpu_tree, torch_or_skip

pytestmark = pytest.mark.gpu

EDGES = (0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 62, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 320)


@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("extra", [1, 2, 17])
def test_lcp_at_step_edges(extra, merged):
    torch_or_skip()
    rng = np.random.default_rng(7 + extra)
    stem = rng.integers(1, 1 << 32, max(EDGES) + extra + 1, dtype=np.uint32)
    paths = []
    for n in EDGES:  # a prefix, its extension, and siblings parting right after n frames
        tail = [int(x) for x in rng.integers(0, 1 << 32, extra, dtype=np.uint32)]
        p = [int(x) for x in stem[:n]]
        paths += [p, p + tail, p + [int(stem[n]) - 1] + tail, p + [0xFFFFFFFF] + tail, p + [0] * extra]
    paths = [paths[i] for i in rng.permutation(len(paths))]
    w = rng.integers(0, 1 << 63, (len(paths), 2), dtype=np.uint64)
    o, f = csr(paths)
    want = oracle.build_tree(o, f, w)
    if not merged:
        assert_same(gpu_tree(o, f, w), want)
        return
    import paper_2411_02797_amd as cct
    from gpu_util import to_dev
    cut = len(paths) // 2
    tree = cct.build(*to_dev(*csr(paths[:cut]), w[:cut]))
    tree.merge(*to_dev(*csr(paths[cut:]), w[cut:]))
    got = tree.to_numpy()
    tree.free()
    assert_same(got, want)

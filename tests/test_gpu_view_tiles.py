"""The bottom-up view at the edges of its tiles: 1,024 sorted nodes to a tile of the sums
and 4,096 to one of the sort, groups that end at, cross and span tiles, frames that differ
in some bytes only, every number of metrics.  Whole numbers: compared for equality."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, torch_or_skip

pytestmark = pytest.mark.gpu

U32 = np.uint32


@pytest.fixture(autouse=True)
def _gpu():
    torch_or_skip()


def flat(frames):
    return np.arange(frames.size + 1, dtype=np.int64), frames.astype(U32)


def shape(kind, n):
    i = np.arange(n, dtype=np.int64)
    if kind == "distinct":            # a group a node
        return flat(i * 3 + 7)
    if kind == "top_byte":            # frames that differ in the highest byte alone
        return flat(((i % 256) << 24) + 5)
    if kind == "hot":                 # one frame below every other: a group over all tiles
        return np.arange(n + 1, dtype=np.int64) * 2, np.stack([i + 10, np.full(n, 4)], 1).ravel().astype(U32)
    if kind == "chain":               # one frame only, recursing: one topmost node
        return np.array([0, n], np.int64), np.full(n, 9, U32)
    assert kind == "pairs"            # groups of two, half of them recursions
    f = np.stack([i + 1, np.where(i % 2, i + 1, (i + 1) | 0x10000)], 1)
    return np.arange(n + 1, dtype=np.int64) * 2, f.ravel().astype(U32)


@pytest.mark.parametrize("kind", ["distinct", "top_byte", "hot", "chain", "pairs"])
@pytest.mark.parametrize("n,m", [(1, 1), (1023, 2), (1024, 3), (1025, 4), (2047, 5), (4095, 6), (4096, 7), (4097, 8)])
def test_view_at_tile_edges(kind, n, m):
    import paper_2411_02797_amd as cct
    o, f = shape(kind, n)
    w = np.random.default_rng(n).integers(0, 2**64, (o.size - 1, m), dtype=np.uint64)  # (sums wrap)
    tree = cct.build(*to_dev(o, f, w))
    v = tree.bottom_up(device="cpu")
    tree.free()
    for name, g, want in zip(("frames", "excl", "incl"), (v["frames"].numpy().view(U32), v["excl"].numpy().view(np.uint64),
                             v["incl"].numpy().view(np.uint64)), oracle.bottom_up(o, f, w)):
        assert np.array_equal(g, want), name

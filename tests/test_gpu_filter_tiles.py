"""Filters over trees at the edges of the tile counts: one tile, the workgroup's four, and more
than the second pass adds up by itself (8,192 tiles of 2,048 nodes)."""
import numpy as np
import pytest

from gpu_util import to_dev, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_paths,length", [(1, 1), (1, 2046), (1, 2047), (1, 2048), (4, 2047), (4, 2048), (5, 1638), (2801, 6000)])
def test_filter_counts_and_places(n_paths, length):
    torch_or_skip()
    # path i: its own first frame, then a chain, so its nodes are one range of ids and all
    # have the path's sum
    import paper_2411_02797_amd as cct
    rng = np.random.default_rng(n_paths + length)
    f = np.tile(np.arange(length, dtype=np.uint32), (n_paths, 1))
    f[:, 0] = np.arange(n_paths, dtype=np.uint32) + 7
    o = np.arange(n_paths + 1, dtype=np.int64) * length
    w = rng.integers(1, 1000, (n_paths, 1), dtype=np.uint64)
    tree = cct.build(*to_dev(o, f.reshape(-1), w))
    try:
        u = 1 + n_paths * length
        assert tree.n_nodes == u
        for thr in (0, 500, 10**6, 10**9):
            per_node = np.concatenate([[w.sum()], np.repeat(w[:, 0], length)])
            want = np.flatnonzero(per_node > thr)
            for noalloc in (False, True):
                got = tree.filter(0, +1, thr, 1, noalloc=noalloc).cpu().numpy()
                assert np.array_equal(got, want), (thr, noalloc, got.size, want.size)
    finally:
        tree.free()

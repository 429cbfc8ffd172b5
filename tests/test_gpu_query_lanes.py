"""Lookups through the prefix index at the edges of the lookup kernel's tiling: eight lanes
share a query, four frames each, 32 per step, and the first 96 frames stay in registers."""
import numpy as np
import pytest

import oracle
from gpu_util import csr, node_paths, to_dev, torch_or_skip

pytestmark = pytest.mark.gpu

LENGTHS = (1, 3, 4, 5, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 131, 159, 160, 161, 255, 300)


@pytest.mark.parametrize("m", [1, 3, 8])
def test_query_lengths_around_lane_steps(m):
    torch_or_skip()
    import paper_2411_02797_amd as cct
    rng = np.random.default_rng(100 + m)
    stem = rng.integers(0, 1 << 32, max(LENGTHS), dtype=np.uint32)
    paths = [list(stem[:n]) for n in LENGTHS] + [[]]
    for n in LENGTHS:  # branches that leave the stem at and next to each edge
        for at in {0, n // 2, n - 1}:
            p = list(stem[:n])
            p[at] = int(p[at]) ^ 1
            paths.append(p)
    o, f = csr(paths)
    w = rng.integers(0, 1 << 40, (len(paths), m), dtype=np.uint64)
    want = oracle.build_tree(o, f, w)
    nodes = np.arange(want.n_nodes)
    of_node = node_paths({"parent": want["parent"], "frame": want["frame"]}, nodes)
    # every node, and every node's path with its last frame changed or one frame more
    absent = [p[:-1] + [int(p[-1]) ^ 2] for p in of_node if p] + [list(p) + [7] for p in of_node]
    known = {tuple(int(x) for x in p) for p in of_node}
    absent = [p for p in absent if tuple(int(x) for x in p) not in known]
    queries = of_node + absent
    order = rng.permutation(len(queries))  # starts at every alignment
    qo, qf = csr([queries[i] for i in order])
    tree = cct.build(*to_dev(o, f, w))
    try:
        to, tf, _ = to_dev(qo, qf, np.zeros((0, 1), np.uint64))
        ids, ex, inc = (t.cpu().numpy() for t in tree.query(to, tf))
    finally:
        tree.free()
    hit = order < len(of_node)
    assert np.array_equal(ids[hit], order[hit])
    assert (ids[~hit] == -1).all() and not ex[~hit].any() and not inc[~hit].any()
    assert np.array_equal(ex[hit].view(np.uint64), want["excl"].reshape(-1, m)[order[hit]])
    assert np.array_equal(inc[hit].view(np.uint64), want["incl"].reshape(-1, m)[order[hit]])

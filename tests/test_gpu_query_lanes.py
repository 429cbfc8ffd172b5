"""Lookups through the prefix index at the edges of the lookup kernel's tiling: eight lanes
share a query, four frames each, 32 per step, and the first 96 frames stay in registers; two or four
lanes in batches of short queries (16 and 32 frames in registers)."""
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


@pytest.mark.parametrize("m", [1, 3, 4, 8])
@pytest.mark.parametrize("mean", [16, 32])
@pytest.mark.parametrize("above", [False, True])
def test_batches_of_short_queries(mean, above, m):
    """Batches whose mean length is just at and just above the ones at which a query takes two, four
    and eight lanes, with queries longer and shorter than their lanes keep, absent ones, empty ones."""
    torch_or_skip()
    import paper_2411_02797_amd as cct
    rng = np.random.default_rng(10 * mean + m)
    edges = (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 40, 47, 48, 49, 64, 130)
    paths = []
    for n in edges:
        p = [int(x) for x in rng.integers(0, 1 << 32, n)]
        paths += [p] + [p[:k] + [p[k] ^ 1] + p[k + 1:] for k in {0, n // 2, n - 1}]
    o, f = csr(paths)
    w = rng.integers(0, 1 << 40, (len(paths), m), dtype=np.uint64)
    want = oracle.build_tree(o, f, w)
    of_path = {tuple(int(x) for x in p): v for v, p in
               enumerate(node_paths({"parent": want["parent"], "frame": want["frame"]}, np.arange(want.n_nodes)))}
    queries = paths + [p[:-1] for p in paths] + [p[:-1] + [p[-1] ^ 2] for p in paths]
    queries += [max(paths, key=len)] * mean
    total = sum(len(p) for p in queries)
    fill = -(-(total - mean * len(queries)) // (mean - 1))  # one-frame queries that bring the mean to `mean`
    assert fill > 0
    queries += [[paths[k % len(paths)][0]] for k in range(fill - above)]
    assert (sum(len(p) for p in queries) > mean * len(queries)) == above
    queries = [queries[i] for i in rng.permutation(len(queries))]
    tree = cct.build(*to_dev(o, f, w))
    try:
        to, tf, _ = to_dev(*csr(queries), np.zeros((0, 1), np.uint64))
        ids, ex, inc = (t.cpu().numpy() for t in tree.query(to, tf))
    finally:
        tree.free()
    expect = np.array([of_path.get(tuple(p), -1) for p in queries])
    assert np.array_equal(ids, expect)
    for got, k in ((ex, "excl"), (inc, "incl")):
        assert np.array_equal(got.view(np.uint64), np.where(expect[:, None] >= 0, want[k].reshape(-1, m)[expect], 0))

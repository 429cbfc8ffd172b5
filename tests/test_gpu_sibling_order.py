"""Sibling order in the block trie at the edges of its rules: groups counted whole (up to 512,
or up to 2,048 in a small trie), groups split into buckets, blocks that share long prefixes,
and blocks that end early or hold zero frames."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, csr, gpu_tree, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shared", [0, 13, 15])  # frames all siblings' blocks share
@pytest.mark.parametrize("sizes", [(1,), (2,), (64, 65), (511, 512, 513), (1023, 1025), (2048,), (2049,), (513, 2, 700, 1, 9000),
                                   (40000,)])
def test_groups_of_siblings(sizes, shared, monkeypatch):
    torch_or_skip()
    monkeypatch.setenv("CCT_TEST_REQUIRE_TRIE", "1")
    rng = np.random.default_rng(sum(sizes) + shared)
    paths = []
    for g, n in enumerate(sizes):  # group g: n blocks below a first block of their own
        head = [7] * 15 + [g] if len(sizes) > 1 else []
        stem = [3] * shared
        kids = set()
        while len(kids) < n:
            room = 16 - shared
            k = int(rng.integers(1, room + 1))
            kids.add(tuple(int(x) for x in rng.integers(0, 60000 if room == 1 else 250, k)) if rng.random() < 0.8
                     else (0,) * k if rng.random() < 0.1 else tuple([0] * (k - 1) + [int(rng.integers(0, 1 << 32))]))
        paths += [head + stem + list(k) for k in kids]
    paths += [[], [3] * shared] if shared else [[]]
    paths = [paths[i] for i in rng.permutation(len(paths))]
    o, f = csr(paths)
    w = rng.integers(0, 1 << 62, (len(paths), 1), dtype=np.uint64)
    assert_same(gpu_tree(o, f, w), oracle.build_tree(o, f, w))


@pytest.mark.parametrize("bits", [1, 2])
def test_equal_blocks_among_siblings(bits, monkeypatch):
    # checkpoint hashes of one or two bits join the paths' full blocks in a few nodes, whose
    # children hold the same blocks many times over (the same ends at different depths): the
    # sampled splitters tie, the exact check refuses the order and the comparison sort takes
    # over.  A first build leaves large values in the scratch memory the second one reuses.
    torch_or_skip()
    rng = np.random.default_rng(bits)
    big = [[int(x) for x in rng.integers(1 << 31, 1 << 32, 40)] for _ in range(6000)]
    o, f = csr(big)
    w = np.ones((len(big), 1), np.uint64)
    assert_same(gpu_tree(o, f, w), oracle.build_tree(o, f, w))
    monkeypatch.setenv("CCT_TEST_CP_HASH_BITS", str(bits))
    paths = [[1 + d % 5] * (16 * d) + [e, e % 3] for d in range(40) for e in range(60)]
    paths = [paths[i] for i in rng.permutation(len(paths))]
    o, f = csr(paths)
    w = rng.integers(0, 1 << 62, (len(paths), 1), dtype=np.uint64)
    assert_same(gpu_tree(o, f, w), oracle.build_tree(o, f, w))


@pytest.mark.parametrize("n,trie", [(150_000, True), (600_000, False)])
def test_wide_groups(n, trie, monkeypatch):
    # buckets of hundreds of siblings, and of more than are counted (the comparison sort takes over)
    torch_or_skip()
    if trie:
        monkeypatch.setenv("CCT_TEST_REQUIRE_TRIE", "1")
    rng = np.random.default_rng(n)
    f = np.full((n, 16), 5, np.uint32)
    f[:, 13:] = rng.integers(0, 1 << 32, (n, 3), dtype=np.uint32)
    o = np.arange(n + 1, dtype=np.int64) * 16
    w = rng.integers(0, 1 << 62, (n, 1), dtype=np.uint64)
    assert_same(gpu_tree(o, f.ravel(), w), oracle.build_tree(o, f.ravel(), w))

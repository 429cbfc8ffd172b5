"""Merges whose new paths the prefix hashes mislead: the exact comparisons have to find out
whatever the ranks do.  The paths are searched for here with the library's hash of a prefix of
16 frames, cut to a few bits by a test setting."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, csr, to_dev, torch_or_skip

pytestmark = pytest.mark.gpu
BITS = 6


def _hashes(paths):
    """hash of the first 16 (k + 1) frames, [paths][k], of paths [n][16 K]"""
    f = np.asarray(paths, np.uint32)
    k = np.arange(f.shape[1], dtype=np.uint32)
    with np.errstate(over="ignore"):
        x = f + k * np.uint32(0x9E3779B9)
        y = ((f ^ np.uint32(0x5BD1E995)) + k * np.uint32(0x85EBCA6B)) | np.uint32(1)
        s = np.cumsum(x.astype(np.uint64) * y.astype(np.uint64), axis=1)[:, 15::16]
        h = s + (np.arange(1, s.shape[1] + 1, dtype=np.uint64) * np.uint64(16)) * np.uint64(0x9E3779B97F4A7C15)
        for mul in (0xFF51AFD7ED558CCD, 0xC4CEB9FE1A85EC53):
            h = (h ^ (h >> np.uint64(33))) * np.uint64(mul)
        return (h ^ (h >> np.uint64(33))) & np.uint64((1 << BITS) - 1)


def _merged(old, new, rng):
    import paper_2411_02797_amd as cct
    w = rng.integers(0, 1 << 62, (len(old) + len(new), 1), dtype=np.uint64)
    tree = cct.build(*to_dev(*csr(old), w[:len(old)]))
    tree.merge(*to_dev(*csr(new), w[len(old):]))
    got = tree.to_numpy()
    tree.free()
    o, f = csr(old + new)
    assert_same(got, oracle.build_tree(o, f, w))


@pytest.mark.parametrize("head", [1, 9])
def test_cycles_before_the_first_old_path(head, monkeypatch):
    """Three new paths y < x < z by their first 16 frames, z < y by the second 16 where the hashes
    of y's and z's first block are equal: each has one of the others before it, and no path takes
    the first place of the order (head 1) or of a later gap."""
    torch_or_skip()
    monkeypatch.setenv("CCT_TEST_CP_HASH_BITS", str(BITS))
    rng = np.random.default_rng(head)
    for case in range(12):
        c = rng.integers(10, 1 << 31, (4000, 32), dtype=np.uint32)
        c[:, 0] = head
        h = _hashes(c)
        by0 = np.lexsort(c[:, 15::-1].T)
        y = by0[0]
        z = next(k for k in by0[::-1] if h[k, 0] == h[y, 0])
        c[z, 16] = min(int(c[z, 16]), int(c[y, 16]) - 1)
        h = _hashes(c)
        if h[z, 1] == h[y, 1]:
            continue
        x = next(k for k in by0[len(by0) // 2:] if h[k, 0] != h[y, 0])
        new = [[int(v) for v in c[k]] for k in (y, x, z)]
        old = [[5] * 20, [5] * 20 + [3], [7, 2], [20] * (1 + case)]
        _merged(old, [new[i] for i in rng.permutation(3)], rng)


@pytest.mark.parametrize("n_old,n_new,pairs", [(40, 60, 12), (1500, 1030, 1), (1500, 1100, 12), (1500, 3000, 150)])
def test_pairs_that_tie_in_one_gap(n_old, n_new, pairs, monkeypatch):
    """Pairs of new paths of one gap with equal hashes, lengths and ends: neither is before the other,
    so both take one rank, and one of them is lost where another path comes twice.  Every merge
    leaves an order of as many paths in the memory that the next one takes."""
    torch_or_skip()
    monkeypatch.setenv("CCT_TEST_CP_HASH_BITS", str(BITS))
    for case in range(12):
        rng = np.random.default_rng(1000 * pairs + case)
        old = [[10 + 2 * h] + [int(v) for v in rng.integers(0, 1 << 32, 3)] for h in range(n_old)]
        c = rng.integers(0, 1 << 32, (64 * pairs + n_new, 16), dtype=np.uint32)
        c[:, 0] = 11 + 2 * rng.integers(0, n_old, len(c))
        c[:64 * pairs, 0] = np.repeat(c[:pairs, 0], 64)
        h = _hashes(c)[:, 0]
        new = []
        for p in range(pairs):
            first = {}
            for k in range(64 * p, 64 * p + 64):
                if first.setdefault(int(h[k]), k) != k:
                    tail = [int(v) for v in rng.integers(0, 9, 4)]
                    new += [[int(v) for v in c[i]] + tail for i in (first[int(h[k])], k)]
                    break
        new += [[int(v) for v in r] for r in c[64 * pairs:][:n_new - len(new)]]
        _merged(old, [new[i] for i in rng.permutation(len(new))], rng)


@pytest.mark.parametrize("n_new", [26 * 1024, 26 * 1024 + 1, 33_000, 64 * 1024 + 1])
@pytest.mark.parametrize("gaps", [1, 3000])
@pytest.mark.parametrize("tied", [False, True])
def test_large_merges_count_or_sort(n_new, gaps, tied, monkeypatch):
    """Merges past the size from which the new paths' gaps decide how they are ordered: most of
    them in one gap or spread over many, an odd and an even number of merge passes, ranks and
    passes; and with hashes of few bits, which leave many pairs in a tie."""
    torch_or_skip()
    if tied:
        if n_new > 30_000:
            pytest.skip("the exact comparison sort of as many paths adds nothing here")
        monkeypatch.setenv("CCT_TEST_CP_HASH_BITS", "14")
    rng = np.random.default_rng(n_new + gaps)
    old = [[10 + 2 * h] + [int(v) for v in rng.integers(0, 1 << 32, 3)] for h in range(3000)]
    c = rng.integers(0, 1 << 32, (n_new, 18), dtype=np.uint32)
    c[:, 0] = 11 + 2 * rng.integers(0, gaps, n_new)
    if tied:
        c[:, 16:] = rng.integers(0, 60, (n_new, 2))
        c = np.unique(c, axis=0)
    _merged(old, [[int(v) for v in r] for r in c[rng.permutation(len(c))]], rng)

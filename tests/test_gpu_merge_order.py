"""The order of a merge's new paths: one block and several, gaps with one new path and with
many, no old paths to speak of, and prefix hashes that collide."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same, csr, to_dev, torch_or_skip

pytestmark = pytest.mark.gpu


def _paths(rng, n, heads, tail):
    """n distinct paths of 17 to 40 frames: a head of `heads` kinds, a stem of two kinds, a tail."""
    out = set()
    stems = rng.integers(0, 1 << 32, (2, 16), dtype=np.uint32)
    while len(out) < n:
        h, s = int(rng.integers(heads)), int(rng.integers(2))
        k = int(rng.integers(1, tail + 1))
        out.add((1000 + h,) + tuple(int(x) for x in stems[s]) + tuple(int(x) for x in rng.integers(0, 50, k)))
    out = [list(p) for p in out]
    return [out[i] for i in rng.permutation(len(out))]


@pytest.mark.parametrize("bits", [None, 6])
@pytest.mark.parametrize("heads", [1, 5000])  # every new path in few gaps, or about one per gap
@pytest.mark.parametrize("n_old,n_new", [(1, 1), (1, 1500), (3000, 31), (3000, 33), (3000, 1023), (3000, 1024), (3000, 1025),
                                         (4000, 2049), (900, 20000), (2000, 66000)])
def test_merge_orders_new_paths(n_old, n_new, heads, bits, monkeypatch):
    torch_or_skip()
    import paper_2411_02797_amd as cct
    if bits is not None:
        if n_new > 3000:
            pytest.skip("the exact comparison sort of many paths that share 17 frames adds nothing here")
        monkeypatch.setenv("CCT_TEST_CP_HASH_BITS", str(bits))
    rng = np.random.default_rng(n_old + 7 * n_new + heads)
    paths = _paths(rng, n_old + n_new, heads, 23)
    w = rng.integers(0, 1 << 63, (len(paths), 2), dtype=np.uint64)
    tree = cct.build(*to_dev(*csr(paths[:n_old]), w[:n_old]))
    tree.merge(*to_dev(*csr(paths[n_old:]), w[n_old:]))
    got = tree.to_numpy()
    tree.free()
    o, f = csr(paths)
    assert_same(got, oracle.build_tree(o, f, w))

"""Error paths of the C ABI, forced from the host; every kernel still exits normally."""
import numpy as np
import pytest

import oracle
import tracegen
from gpu_util import assert_same, gpu_tree, to_dev, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    torch_or_skip()


def _status(fn):
    import paper_2411_02797_amd as cct
    with pytest.raises(cct.CctError) as ei:
        fn()
    return ei.value.name


@pytest.mark.parametrize("kind", ["first_nonzero", "decreasing", "last_mismatch", "huge"])
def test_malformed_offsets(kind):
    import paper_2411_02797_amd as cct
    torch = torch_or_skip()
    o, f, w = tracegen.random_paths(5000, 30, 10, 1, seed=1)
    to, tf, tw = to_dev(o, f, w)
    bad = to.clone()
    if kind == "first_nonzero":
        bad[0] = 1
    elif kind == "decreasing":
        bad[2500] = bad[2499] - 1
    elif kind == "last_mismatch":
        bad[-1] = bad[-1] - 1
    else:
        bad[1000] = 2**40
    assert _status(lambda: cct.build(bad, tf, tw)) == "CCT_EINVAL"


def test_merge_failure_leaves_tree_unchanged():
    import paper_2411_02797_amd as cct
    o, f, w = tracegen.random_paths(4000, 60, 10, 2, seed=2)
    tree = cct.build(*to_dev(o, f, w))
    before = tree.to_numpy()
    o2, f2, w2 = tracegen.random_paths(3000, 60, 10, 2, seed=3)
    to2, tf2, tw2 = to_dev(o2, f2, w2)
    bad = to2.clone()
    bad[1500] = bad[1499] - 1
    assert _status(lambda: tree.merge(bad, tf2, tw2)) == "CCT_EINVAL"
    assert_same(tree.to_numpy(), before, "after failed merge")
    _, _, tw3 = to_dev(o2, f2, np.zeros((3000, 3), np.uint64))
    assert _status(lambda: tree.merge(to2, tf2, tw3)) == "CCT_EMISMATCH"
    tree.merge(to2, tf2, tw2)  # still usable
    orc = oracle.Oracle(2)
    orc.ingest(o, f, w)
    orc.ingest(o2, f2, w2)
    assert_same(tree.to_numpy(), orc.tree(), "merge after failures")
    tree.free()


@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 12, 16, 20, 24, 28, 32, 36])
def test_allocation_failure(monkeypatch, k):
    import paper_2411_02797_amd as cct
    o, f, w = tracegen.random_paths(3000, 40, 10, 1, seed=k)
    tree = cct.build(*to_dev(o, f, w))
    before = tree.to_numpy()
    o2, f2, w2 = tracegen.random_paths(2000, 80, 10, 1, seed=100 + k)
    d2 = to_dev(o2, f2, w2)
    monkeypatch.setenv("CCT_TEST_FAIL_ALLOC", str(k))
    try:
        tree.merge(*d2)
        merged = True
    except cct.CctError as e:
        assert e.name == "CCT_ENOMEM"
        merged = False
    monkeypatch.delenv("CCT_TEST_FAIL_ALLOC")
    orc = oracle.Oracle(1)
    orc.ingest(o, f, w)
    orc.ingest(o2, f2, w2)
    if merged:
        assert_same(tree.to_numpy(), orc.tree(), "merged")
    else:
        assert_same(tree.to_numpy(), before, "unchanged after ENOMEM")
        # the failed call left no trace in the tree's table, path store or sums
        tree.merge(*d2)
        assert_same(tree.to_numpy(), orc.tree(), "merge after ENOMEM")
    orc.close()
    tree.free()
    monkeypatch.setenv("CCT_TEST_FAIL_ALLOC", str(k))
    try:
        t = gpu_tree(o, f, w)
        assert_same(t, oracle.build_tree(o, f, w))
    except cct.CctError as e:
        assert e.name == "CCT_ENOMEM"


def test_bad_tensor_arguments():
    import paper_2411_02797_amd as cct
    torch = torch_or_skip()
    o, f, w = tracegen.random_paths(10, 5, 4, 1, seed=1)
    to, tf, tw = to_dev(o, f, w)
    with pytest.raises(ValueError):
        cct.build(to.to(torch.int32), tf, tw)
    with pytest.raises(ValueError):
        cct.build(to, tf, tw[:5])
    with pytest.raises(ValueError):
        cct.build(to, tf, torch.zeros((10, 9), dtype=torch.int64, device=to.device)[:, ::2])
    assert _status(lambda: cct.build(to, tf, torch.zeros((10, 9), dtype=torch.int64, device=to.device))) \
        == "CCT_EINVAL"


@pytest.mark.parametrize("kind", ["first_nonzero", "decreasing", "last_mismatch", "overflow"])
def test_early_exit_after_pool_reuse(monkeypatch, kind):
    # Regression: a wave that stops early (malformed offsets, or a table overflow that the
    # host retries) must still mark the rest of its events unresolved, because the
    # aggregation reads every event's slot id.  The pool is first filled with large
    # words (an activity merge with IDs near 2^64) so that stale memory would be out of
    # range.
    import paper_2411_02797_amd as cct
    torch = torch_or_skip()
    dev = torch.device("cuda", 0)
    for rep in range(3):
        n = 4000 + 1000 * rep
        ro, rf, _ = tracegen.random_paths(n, 30, 10, 1, seed=rep)
        ids = (np.arange(n, dtype=np.uint64) + np.uint64(2**64 - 2 * n))
        big = torch.from_numpy(ids.view(np.int64)).to(dev)
        t0 = cct.build(*to_dev(ro, rf, np.ones((n, 1), np.uint64)))
        tro, trf, _ = to_dev(ro, rf, np.zeros((n, 1), np.uint64))
        t0.merge_activity(tro, trf, big, big.flip(0).contiguous(), torch.ones((n, 1), dtype=torch.int64, device=dev))
        t0.free()
    o, f, w = tracegen.random_paths(5000, 30, 10, 1, seed=1)
    to, tf, tw = to_dev(o, f, w)
    if kind == "overflow":
        monkeypatch.setenv("CCT_TEST_TABLE_CAP", "64")  # far fewer slots than paths: overflow, then retries
        t = cct.build(to, tf, tw)
        got = t.to_numpy()
        t.free()
        assert_same(got, oracle.build_tree(o, f, w), "after overflow retries")
        return
    bad = to.clone()
    if kind == "first_nonzero":
        bad[0] = 1
    elif kind == "decreasing":
        bad[2500] = bad[2499] - 1
    else:
        bad[-1] = bad[-1] - 1
    assert _status(lambda: cct.build(bad, tf, tw)) == "CCT_EINVAL"
    t = cct.build(to, tf, tw)  # the library is still usable
    assert_same(t.to_numpy(), oracle.build_tree(o, f, w), "after EINVAL")
    t.free()


@pytest.mark.parametrize("k", [1, 4, 7, 9, 10, 12, 15, 18, 21, 24, 27, 30, 34, 38, 42, 46, 50])
def test_allocation_failure_with_statistics(monkeypatch, k):
    # a tree keeping statistics allocates more per merge (slot -> path map, staging lists,
    # larger path arrays): a failure at any of them leaves the tree and its statistics as
    # they were, and the same merge then succeeds
    import paper_2411_02797_amd as cct
    o, f, w = tracegen.random_paths(3000, 40, 10, 2, seed=k)
    tree = cct.build(*to_dev(o, f, w), stats=True)
    before = tree.to_numpy()
    stats_before = {n: v.cpu() for n, v in tree.stats().items()}
    o2, f2, w2 = tracegen.random_paths(2000, 80, 10, 2, seed=200 + k)
    d2 = to_dev(o2, f2, w2)
    monkeypatch.setenv("CCT_TEST_FAIL_ALLOC", str(k))
    try:
        tree.merge(*d2)
        merged = True
    except cct.CctError as e:
        assert e.name == "CCT_ENOMEM"
        merged = False
    monkeypatch.delenv("CCT_TEST_FAIL_ALLOC")
    orc = oracle.Oracle(2, stats=True)
    orc.ingest(o, f, w)
    orc.ingest(o2, f2, w2)
    want = orc.tree()
    orc.close()
    if not merged:
        assert_same(tree.to_numpy(), before, "unchanged after ENOMEM")
        after = tree.stats()
        for n, v in stats_before.items():
            assert np.array_equal(v.numpy(), after[n].cpu().numpy(), equal_nan=True), n
        tree.merge(*d2)
    assert_same(tree.to_numpy(), want, "merged")
    got = tree.stats(device="cpu")
    for n in ("count_excl", "count_incl", "min_excl", "min_incl", "sumsq_excl", "sumsq_incl"):
        assert np.array_equal(got[n].numpy().view(np.uint64), want[n]), n
    tree.free()


@pytest.mark.parametrize("stats", [False, True])
def test_failure_after_publish_leaves_tree_unchanged(monkeypatch, stats):
    # a merge that fails after its new paths are published and its sums folded (forced by
    # a test setting) leaves the tree, its statistics and its table as they were: a merge
    # of another batch, which reuses the failed call's path ids, and then the failed batch
    # itself, equal the oracle
    import paper_2411_02797_amd as cct
    o, f, w = tracegen.random_paths(3000, 40, 10, 2, seed=71)
    tree = cct.build(*to_dev(o, f, w), stats=stats)
    before = tree.to_numpy()
    stats_before = {n: v.cpu() for n, v in tree.stats().items()} if stats else None
    oa, fa, wa = tracegen.random_paths(2000, 80, 10, 2, seed=72)   # the batch that fails
    ob, fb, wb = tracegen.random_paths(2500, 90, 12, 2, seed=73)   # another batch
    monkeypatch.setenv("CCT_TEST_FAIL_AFTER_PUBLISH", "1")
    assert _status(lambda: tree.merge(*to_dev(oa, fa, wa))) == "CCT_EDEVICE"
    monkeypatch.delenv("CCT_TEST_FAIL_AFTER_PUBLISH")
    assert_same(tree.to_numpy(), before, "unchanged after a failure past publish")
    if stats:
        after = tree.stats()
        for n, v in stats_before.items():
            assert np.array_equal(v.numpy(), after[n].cpu().numpy(), equal_nan=True), n
    tree.merge(*to_dev(ob, fb, wb))
    tree.merge(*to_dev(oa, fa, wa))
    orc = oracle.Oracle(2, stats=stats)
    orc.ingest(o, f, w)
    orc.ingest(ob, fb, wb)
    orc.ingest(oa, fa, wa)
    want = orc.tree()
    orc.close()
    assert_same(tree.to_numpy(), want, "merges after the failure")
    if stats:
        got = tree.stats(device="cpu")
        for n in ("count_excl", "count_incl", "min_excl", "min_incl", "sumsq_excl", "sumsq_incl"):
            assert np.array_equal(got[n].numpy().view(np.uint64), want[n]), n
    # every node is still found by a query (the table and the path store agree)
    ids, _, _ = tree.query(*to_dev(oa, fa, wa)[:2])
    assert bool((ids >= 0).all())
    tree.free()


@pytest.mark.parametrize("kind", ["first_nonzero", "decreasing", "last_mismatch"])
def test_malformed_query_offsets_leave_outputs_untouched(kind):
    import ctypes
    import paper_2411_02797_amd as cct
    torch = torch_or_skip()
    o, f, w = tracegen.random_paths(3000, 30, 10, 2, seed=5)
    tree = cct.build(*to_dev(o, f, w))
    qo, qf, _ = to_dev(o[:501], f[:o[500]], w[:500])
    if kind == "first_nonzero":
        qo[0] = 1
    elif kind == "decreasing":
        qo[250] = qo[249] - 1
    else:
        qo[-1] = qo[-1] - 1
    ids = torch.full((500,), -7, dtype=torch.int64, device="cuda")
    ex = torch.full((500, 2), -7, dtype=torch.int64, device="cuda")
    inc = torch.full((500, 2), -7, dtype=torch.int64, device="cuda")
    p, _ = cct._paths(qo, qf, None, need_metrics=False)
    st = cct.load_library().cct_query(tree.handle, ctypes.byref(p), cct._stream(), ids.data_ptr(), ex.data_ptr(),
                                      inc.data_ptr())
    torch.cuda.synchronize()
    assert st == -1
    assert bool((ids == -7).all()) and bool((ex == -7).all()) and bool((inc == -7).all())
    tree.free()


@pytest.mark.parametrize("short", range(5))
def test_export_to_a_short_array_is_refused(short):
    # one of the arrays is an allocation of 256 bytes (the runtime maps a whole page for it),
    # shorter than the tree's array; nothing is written to it
    import ctypes
    import paper_2411_02797_amd as cct
    torch = torch_or_skip()
    tree = cct.build(*to_dev(*tracegen.random_paths(60, 40, 6, 1, seed=3)))
    u = tree.n_nodes
    assert 64 < u < 400
    hip = lib = cct.load_library()  # (its runtime's symbols are found through it)
    p, host = ctypes.c_void_p(), (ctypes.c_uint8 * 256)()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(256)) == 0
    assert hip.hipMemset(p, 0xA5, ctypes.c_size_t(256)) == 0
    long = [torch.full((8 * u,), 7, dtype=torch.uint8, device="cuda") for _ in range(5)]
    args = [ctypes.c_void_p(t.data_ptr()) for t in long]
    args[short] = p
    assert lib.cct_export(tree.handle, cct._stream(), *args) != 0
    torch.cuda.synchronize()
    assert hip.hipMemcpy(host, p, ctypes.c_size_t(256), 2) == 0
    assert bytes(host) == b"\xa5" * 256
    args[short] = ctypes.c_void_p(long[short].data_ptr())  # the same arrays, long enough
    assert lib.cct_export(tree.handle, cct._stream(), *args) == 0
    want = tree.to_numpy()
    for t, k in zip(long, ("parent", "frame", "depth", "excl", "incl")):
        n = want[k].nbytes
        assert t[:n].cpu().numpy().tobytes() == want[k].tobytes() and bool((t[n:] == 7).all()), k
    assert hip.hipFree(p) == 0
    tree.free()

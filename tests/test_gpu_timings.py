"""What last_timings() reports where a call takes an uncommon way."""
import time

import numpy as np
import pytest

import tracegen
from gpu_util import to_dev, torch_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5000, 100_000])  # one stream, two streams
def test_whole_call_counts_the_attempts_before_a_regrow(n, monkeypatch):
    # the table overflows and grows several times; some memory of earlier calls is left for the
    # larger control block of a later attempt
    torch_or_skip()
    import paper_2411_02797_amd as cct
    o, f, w = tracegen.random_paths(n, 50_000, 12, 2, seed=n)
    d = to_dev(o, f, w)
    for cap in (64, 256, 4096):
        cct.build(*d).free()
        plain = cct.last_timings()
        monkeypatch.setenv("CCT_TEST_TABLE_CAP", str(cap))
        t0 = time.perf_counter()
        cct.build(*d).free()
        wall = (time.perf_counter() - t0) * 1e3
        monkeypatch.delenv("CCT_TEST_TABLE_CAP")
        got = cct.last_timings()
        assert all(np.isfinite(got)), got
        assert sum(got[:4]) <= got[4] * 1.001 <= wall * 1.01, (cap, got, wall)
        assert got[4] > plain[4] * 0.5, (cap, got, plain)


@pytest.mark.parametrize("n", [20, 3000])  # one tile of nodes, several
def test_filter_time_lies_within_the_call(n):
    torch = torch_or_skip()
    import paper_2411_02797_amd as cct
    tree = cct.build(*to_dev(*tracegen.random_paths(n, 300, 20, 1, seed=n)))
    for thr in (0, 1 << 60):  # every node with a sum, none
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        tree.filter(0, +1, thr, 1)
        wall = (time.perf_counter() - t0) * 1e3
        assert 0 < cct.last_timings()[7] <= wall * 1.01
    tree.free()

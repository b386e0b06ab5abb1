"""Parent offsets of batched runs on both sides of the size (1024 blocks of 256
parents, by the run's capacity) from which a run's block sums are scanned by a
launch of their own, mixed in one batch and with runs refused for capacity:
equal to the same runs advanced alone."""
import math

import numpy as np
import pytest

import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu


def _cap(R):
    return R + math.ceil(10.0 * math.sqrt(R)) + 64


EDGE = 1024 * 256


@pytest.mark.parametrize("theta", [0, 1])
@pytest.mark.parametrize("sizes", [(1, 255, 257), (EDGE - 8192, 300), (EDGE, 300, EDGE - 8192)])
def test_offsets_of_small_and_large_runs(sizes, theta):
    print("case batch scatter sizes=%s theta=%d" % (sizes, theta), flush=True)
    assert _cap(EDGE - 8192) <= EDGE < _cap(EDGE)
    runs = [dict(L=16, R=R, seed=51 + i, layout="bits") for i, R in enumerate(sizes)]
    sched = [dict(beta_f=0.06, dbeta=0.02, theta=theta, mode="fixed")] * len(runs)
    b = pa.Batch(runs, sched)
    b.run()
    for i, spec in enumerate(runs):
        g = pa.Run(**spec)
        trace = [g.observables()] + g.anneal(beta_f=0.06, dbeta=0.02, theta=theta, mode="fixed")
        hist = b.history(i)
        assert len(hist) == len(trace) == 4
        for h, t in zip(hist, trace):
            assert all(h[k] == t[k] for k in ("R", "sumE", "sumE2", "sumAbsM", "sumM2", "sumM4", "beta", "lnQ"))
        for ours, alone in zip(b.download_population(i), g.download_population()):
            assert np.array_equal(ours, alone)
        g.close()
    b.close()


def test_refused_run_beside_others():
    print("case batch scatter refused", flush=True)
    # no room above R: a run is refused at its first step with R_1 > R
    runs = [dict(L=16, R=900, seed=s, capacity=900, layout="bits") for s in range(6)] + [dict(L=16, R=900, seed=9)]
    b = pa.Batch(runs, [dict(beta_f=0.2, dbeta=0.05, theta=1, mode="fixed")] * len(runs))
    b.run()
    refused = 0
    for i, spec in enumerate(runs):
        g = pa.Run(**spec)
        try:
            g.anneal(beta_f=0.2, dbeta=0.05, theta=1, mode="fixed")
            assert b.status(i) == pa.PA_OK
        except pa.PaError:
            assert b.status(i) == pa.PA_ECAPACITY
            refused += 1
        assert b.state(i)["step"] == g.state()["step"]
        for ours, alone in zip(b.download_population(i), g.download_population()):
            assert np.array_equal(ours, alone)
        g.close()
    assert 0 < refused < len(runs)
    b.close()

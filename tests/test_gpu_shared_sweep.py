"""The sweep of few replicas of L >= 64, four waves to a replica, and the
ordinary one beyond: sizes around the change (1280 replicas at L = 64, 2048 at
L = 128 and 256), both updates and stores, thresholds with empty high halves,
all-ones runs and 2^32, the gathering sweep with the statistics in its epilogue
or in a pass, and the overflow routes of the ordinary path's tie queue.
Bit-exact against the oracle."""
import math

import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu

BETAS = [0.0, 1e-6, math.log(2.0) / 8.0, 0.4406868, 5.6]


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)


@pytest.mark.parametrize("layout", ["int8", "bits"])
@pytest.mark.parametrize("heatbath", [False, True])
@pytest.mark.parametrize("L,R", [(64, 1), (64, 7), (64, 300), (128, 1), (128, 5), (256, 1), (256, 3)])
def test_few_replicas(L, R, heatbath, layout):
    spins = inputs.mixed_spins(R, L, seed=R)
    for beta in BETAS:
        print("case shared sweep L=%d R=%d hb=%d %s beta=%g" % (L, R, heatbath, layout, beta), flush=True)
        for path in ("epilogue", "pass"):
            g = pa.Run(L, R, seed=43, run_id=5, layout=layout, heatbath=heatbath, capacity=4 * R + 8)
            g.set_stats_path(path)
            o = oracle.Run(L, R, seed=43, run_id=5, heatbath=heatbath, capacity=4 * R + 8)
            g.upload_population(spins, step=1, sweeps=3, beta=beta)
            o.set_population(spins, step=1, sweeps=3, beta=beta)
            g.sweep(2)
            o.sweep(2)
            _same(g, o)
            bn = beta + 0.05 / L
            got = g.anneal(beta_f=bn, dbeta=bn, theta=1, mode="fixed", max_steps=1)
            o.resample(got[0]["beta"])
            o.sweep(1)
            _same(g, o)
            m = o.measure()
            assert all(got[0][k] == m[k] for k in ("R", "sumE", "sumE2", "sumAbsM", "sumM2", "sumM4"))
            g.close()


@pytest.mark.parametrize("L,R,qcap,heatbath", [(64, 1280, None, False), (64, 1281, None, True), (128, 2048, None, True),
                                               (128, 2049, None, False), (128, 2049, 0, True), (128, 2049, 8, False),
                                               (256, 2048, None, False), (256, 2049, 0, False)])
def test_around_the_change(L, R, qcap, heatbath):
    print("case shared sweep edge L=%d R=%d qcap=%s hb=%d" % (L, R, qcap, heatbath), flush=True)
    spins = np.tile(inputs.mixed_spins(16, L, seed=L), (R // 16 + 1, 1, 1))[:R]
    g = pa.Run(L, R, seed=47, layout="bits", heatbath=heatbath)
    o = oracle.Run(L, R, seed=47, heatbath=heatbath)
    if qcap is not None:
        g.set_tie_queue_cap(qcap)
    g.upload_population(spins, step=1, sweeps=3, beta=0.44)
    o.set_population(spins, step=1, sweeps=3, beta=0.44)
    g.sweep(1)
    o.sweep(1)
    _same(g, o)
    g.close()

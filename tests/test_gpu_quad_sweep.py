"""The sweep of small launches of L = 16 and 32, whose words are shared by four
lanes, and the ordinary one beyond: sizes around the change (4096 waves of 4
replicas at L = 16, of 1 at L = 32), partly filled waves, thresholds with empty
high halves, all-ones runs and 2^32, both updates and stores, and the gathering
sweep of a resampled population.  Bit-exact against the oracle."""
import math

import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu

BETAS = [0.0, 1e-12, 1e-6, math.log(2.0) / 8.0, 0.4406868, 2.9, 5.6]


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)


@pytest.mark.parametrize("layout", ["int8", "bits"])
@pytest.mark.parametrize("heatbath", [False, True])
@pytest.mark.parametrize("L,R", [(16, 1), (16, 3), (16, 1021), (32, 1), (32, 67), (16, 16384), (16, 16385), (32, 4096),
                                 (32, 4097)])
def test_sweep_matches_oracle(L, R, heatbath, layout):
    spins = inputs.mixed_spins(R, L, seed=R)
    for beta in BETAS if R < 2000 else BETAS[4:5]:
        print("case quad sweep L=%d R=%d hb=%d %s beta=%g" % (L, R, heatbath, layout, beta), flush=True)
        g = pa.Run(L, R, seed=41, run_id=2, layout=layout, heatbath=heatbath)
        o = oracle.Run(L, R, seed=41, run_id=2, heatbath=heatbath)
        g.upload_population(spins, step=1, sweeps=3, beta=beta)
        o.set_population(spins, step=1, sweeps=3, beta=beta)
        g.sweep(2)
        o.sweep(2)
        _same(g, o)
        if R < 2000:  # and the sweep that loads the parents
            bn = beta + 0.2 / L
            got = g.anneal(beta_f=bn, dbeta=bn, theta=2, mode="fixed", max_steps=1)
            o.resample(got[0]["beta"])
            o.sweep(2)
            _same(g, o)
        g.close()

"""The sweep's comparison of bit planes and its tie queue at their edges:
thresholds with few set bits, all-ones runs and empty high halves, and queues
that overflow between two groups of words.  Bit-exact against the oracle."""
import math

import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)


# T_2 = 2^31 and T_4 = 2^30; T_4 = 2^31; T_2 just below 2^32; high halves 0
# (every plane bit 0); T_4 = 1
EDGES = [math.log(2.0) / 4.0, math.log(2.0) / 8.0, 1e-6, 2.9, 5.6]


@pytest.mark.parametrize("heatbath", [False, True])
@pytest.mark.parametrize("L,R", [(16, 37), (32, 9), (64, 5), (128, 5), (256, 2)])
def test_threshold_edges(L, R, heatbath):
    spins = inputs.mixed_spins(R, L, seed=L)
    for beta in EDGES:
        print("case plane edges L=%d hb=%d beta=%g" % (L, heatbath, beta), flush=True)
        g = pa.Run(L, R, seed=23, heatbath=heatbath)
        o = oracle.Run(L, R, seed=23, heatbath=heatbath)
        g.upload_population(spins, step=1, sweeps=3, beta=beta)
        o.set_population(spins, step=1, sweeps=3, beta=beta)
        g.sweep(3)
        o.sweep(3)
        _same(g, o)
        g.close()


@pytest.mark.parametrize("cap", [24, 40, 56])
@pytest.mark.parametrize("L,R", [(128, 7), (256, 3)])
def test_queue_overflow_between_groups(L, R, cap):
    # a group of four words queues about 28 entries: at L = 256 the second
    # group of a chunk then finds the queue partly full
    print("case queue groups L=%d cap=%d" % (L, cap), flush=True)
    spins = inputs.mixed_spins(R, L, seed=L + 1)
    g = pa.Run(L, R, seed=29)
    o = oracle.Run(L, R, seed=29)
    g.set_tie_queue_cap(cap)
    g.upload_population(spins, step=2, sweeps=5, beta=0.5)
    o.set_population(spins, step=2, sweeps=5, beta=0.5)
    g.sweep(4)
    o.sweep(4)
    _same(g, o)

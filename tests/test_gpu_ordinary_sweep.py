"""The sweep kernels with one wave to a replica or to several (the ones large
populations take) at the edges that small populations otherwise meet only on
the kernels for few replicas: thresholds with few set bits, all-ones runs, empty
high halves and 2^32, partly filled waves of the int8 store's stores, and every
overflow route of the tie queue.  pa_anneal sizes its launches by the capacity,
so a small population with a large one takes them (L >= 64: beyond 1280 and 2048
replicas); L = 16 and 32 do with the statistics in the sweep's epilogue.
Bit-exact against the oracle."""
import math

import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu

# T = 2^32; T_4 alone below it; both just below it; T_4 = 2^31; T_2 = 2^31 and T_4 = 2^30;
# the transition; high halves 0 (every plane bit 0); T_4 = 1
BETAS = [1e-12, 3.5e-11, 1e-6, math.log(2.0) / 8.0, math.log(2.0) / 4.0, 0.4406868, 2.9, 5.6]
CAPACITY = {16: 0, 32: 0, 64: 1281, 128: 2049, 256: 2049}


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)


def _pair(L, R, seed, layout, heatbath, beta):
    """A run and the oracle's just below beta, on the same mixed population."""
    g = pa.Run(L, R, seed=seed, run_id=3, capacity=CAPACITY[L], layout=layout, heatbath=heatbath)
    o = oracle.Run(L, R, seed=seed, run_id=3, capacity=CAPACITY[L], heatbath=heatbath)
    g.set_stats_path("epilogue")
    spins = inputs.mixed_spins(R, L, seed=L + R)
    for run in (g, o):
        (run.upload_population if run is g else run.set_population)(spins, step=0, sweeps=3, beta=beta * (1.0 - 1e-9))
    return g, o


@pytest.mark.parametrize("layout", ["int8", "bits"])
@pytest.mark.parametrize("heatbath", [False, True])
@pytest.mark.parametrize("L,R", [(16, 1), (16, 15), (16, 37), (32, 1), (32, 3), (32, 9), (64, 5), (128, 5), (256, 2)])
def test_threshold_edges(L, R, heatbath, layout):
    for beta in BETAS:
        print("case ordinary edges L=%d R=%d hb=%d %s beta=%g" % (L, R, heatbath, layout, beta), flush=True)
        g, o = _pair(L, R, 61, layout, heatbath, beta)
        got = g.anneal(beta_f=beta, dbeta=beta, theta=3, mode="fixed", max_steps=1)
        o.resample(beta)
        o.sweep(3)
        _same(g, o)
        m = o.measure()
        assert all(got[0][k] == m[k] for k in ("R", "sumE", "sumE2", "sumAbsM", "sumM2", "sumM4"))
        if L <= 32:  # and at beta = 0, in place
            g.upload_population(inputs.mixed_spins(R, L, seed=R), step=1, sweeps=5, beta=0.0)
            o.set_population(inputs.mixed_spins(R, L, seed=R), step=1, sweeps=5, beta=0.0)
            g.sweep(2)
            o.sweep(2)
            _same(g, o)
        g.close()


@pytest.mark.parametrize("layout", ["int8", "bits"])
@pytest.mark.parametrize("heatbath", [False, True])
@pytest.mark.parametrize("cap", [0, 8, 24, 40, 56, 127])
@pytest.mark.parametrize("L,R", [(128, 5), (256, 2)])
def test_tie_queue_overflow(L, R, cap, heatbath, layout):
    # a group of four words queues about 28 words, so that a chunk of eight
    # overflows in its first group, in its second or not at all
    print("case ordinary queue L=%d cap=%d hb=%d %s" % (L, cap, heatbath, layout), flush=True)
    g, o = _pair(L, R, 67, layout, heatbath, 0.5)
    g.set_tie_queue_cap(cap)
    got = g.anneal(beta_f=0.5, dbeta=0.5, theta=5, mode="fixed", max_steps=1)
    o.resample(got[0]["beta"])
    o.sweep(5)
    _same(g, o)
    g.close()


@pytest.mark.parametrize("L,R", [(64, 8200), (16, 131100)])
@pytest.mark.parametrize("layout", ["int8", "bits"])
def test_lcg_where_the_waves_just_exceed_the_gpu(L, R, layout):
    # (8192 waves of the register path fit at once)
    print("case ordinary lcg L=%d R=%d %s" % (L, R, layout), flush=True)
    spins = np.tile(inputs.mixed_spins(20, L, seed=L), (R // 20 + 1, 1, 1))[:R]
    g = pa.Run(L, R, seed=71, layout=layout, lcg=True)
    o = oracle.Run(L, R, seed=71, lcg=True)
    g.upload_population(spins, step=1, sweeps=2, beta=0.44)
    o.set_population(spins, step=1, sweeps=2, beta=0.44)
    g.sweep(1)
    o.sweep(1)
    _same(g, o)
    g.close()


@pytest.mark.parametrize("L,R", [(16, 16384), (16, 16385), (32, 4096), (32, 4097), (64, 1024), (64, 1025), (128, 1024),
                                 (128, 1025), (256, 1024), (256, 1025)])
@pytest.mark.parametrize("layout", ["int8", "bits"])
def test_lcg_around_one_wave_per_simd(L, R, layout):
    # up to 1024 waves the comparisons go in pairs and without wave priorities
    print("case lcg 1024 waves L=%d R=%d %s" % (L, R, layout), flush=True)
    spins = np.tile(inputs.mixed_spins(16, L, seed=L + 1), (R // 16 + 1, 1, 1))[:R]
    g = pa.Run(L, R, seed=72, layout=layout, lcg=True)
    o = oracle.Run(L, R, seed=72, lcg=True)
    g.upload_population(spins, step=1, sweeps=2, beta=0.44)
    o.set_population(spins, step=1, sweeps=2, beta=0.44)
    g.sweep(1)
    o.sweep(1)
    _same(g, o)
    g.close()

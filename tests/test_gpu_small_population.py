"""Resampling and statistics of small populations (one block each) and the first
sizes beyond them, against the oracle: ends of the block's turns (4096 parents),
of its own range (16384), windows wider than its LDS tables (4096 bins), and
refused steps.  All results are whole numbers and must be equal."""
import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa
import torch

pytestmark = pytest.mark.gpu

SUMS = ("sumE", "sumE2", "sumAbsM", "sumM2", "sumM4", "R")


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)
    gobs, oobs = g.observables(), o.measure()
    assert [gobs[k] for k in SUMS] == [oobs[k] for k in SUMS]


def _observe(g, L):
    _, E, M = g.download_population()
    obs, got = g.observables(), pa.observables_static(L, torch.from_numpy(E).cuda(), torch.from_numpy(M).cuda())
    assert [got[k] for k in SUMS] == [obs[k] for k in SUMS]


# (the wide windows are those of mixed populations: about N of N + 1 bins)
@pytest.mark.parametrize("L,R", [(16, 1), (16, 3), (16, 64), (16, 257), (16, 4095), (16, 4097), (16, 16384),
                                 (16, 16385), (32, 8193), (64, 33), (128, 9), (256, 7)])
def test_steps_match_oracle(L, R):
    print("case small population L=%d R=%d" % (L, R), flush=True)
    spins = inputs.mixed_spins(R, L, seed=R)
    spins[0] = 1  # the ground state: the window's lower end
    g, o = pa.Run(L, R, seed=31, capacity=3 * R + 64), oracle.Run(L, R, seed=31, capacity=3 * R + 64)
    g.set_stats_path("pass")
    g.upload_population(spins, step=2, sweeps=5, beta=0.2)
    o.set_population(spins, step=2, sweeps=5, beta=0.2)
    _same(g, o)
    _observe(g, L)
    for beta in (0.2, 0.2 + 2.0 / (L * L)):
        gi, oi = g.resample(beta), o.resample(beta)
        assert gi["R_new"] == oi["R_new"] and gi["lnQ"] == oi["lnQ"]
        assert np.array_equal(g.download_counts(g.capacity), o.get_counts())
        _same(g, o)
    got = g.anneal(beta_f=beta + 2.0 / (L * L), dbeta=beta + 2.0 / (L * L), theta=1, mode="fixed", max_steps=1)
    assert len(got) == 1
    o.resample(got[0]["beta"])
    o.sweep(1)
    _same(g, o)
    g.close()


@pytest.mark.parametrize("R", [70, 5000])
def test_refused_step_writes_nothing_beyond_the_capacity(R):
    print("case small population refused R=%d" % R, flush=True)
    g = pa.Run(16, R, seed=3, capacity=R)
    s = np.ones((2 * R // 3, 16, 16), np.int8)
    refused = 0
    for seed_step in range(1, 9):  # equal replicas: R_new is about R
        g.upload_population(s, step=seed_step, beta=0.1)
        o = oracle.Run(16, R, seed=3, capacity=4 * R)
        o.set_population(s, step=seed_step, beta=0.1)
        R_new = o.resample(0.3)["R_new"]
        try:
            assert g.resample(0.3)["R_new"] == R_new
        except pa.PaError:
            assert R_new > R
            refused += 1
    print("refused", refused, flush=True)
    g.close()

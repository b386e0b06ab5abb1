"""The interleaved store's packing into the bit store and back at the edges of
its tiles (64 replicas per wave): population sizes around them, capacities that
leave room in the last tile, several calls in a row, and a refused step, which
leaves the population as it was."""
import numpy as np
import pytest

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu


def _same(g, o):
    for ours, theirs in zip(g.download_population(), o.get_population()):
        assert np.array_equal(ours, theirs)


@pytest.mark.parametrize("L", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("R", [1, 63, 64, 65, 130])
def test_tiles(L, R):
    if L >= 128 and R == 130:
        R = 66
    print("case interleaved tiles L=%d R=%d" % (L, R), flush=True)
    g = pa.Run(L, R, seed=31, layout="interleaved")
    o = oracle.Run(L, R, seed=31)
    o.init()
    _same(g, o)  # initial state
    spins = inputs.mixed_spins(R, L, seed=L + R)
    g.upload_population(spins, step=1, sweeps=2, beta=0.4)
    o.set_population(spins, step=1, sweeps=2, beta=0.4)
    _same(g, o)  # E and M counted from the bytes
    for n in (1, 2):
        g.sweep(n)
        o.sweep(n)
        _same(g, o)
    g.close()


@pytest.mark.parametrize("steps", [1, 2, 3])
def test_anneal_then_single_calls(steps):
    # an odd number of steps ends in the other buffer than an even one
    L, R = 32, 200
    print("case interleaved anneal steps=%d" % steps, flush=True)
    g = pa.Run(L, R, seed=37, layout="interleaved")
    b = pa.Run(L, R, seed=37, layout="bits")
    for r in (g, b):
        r.anneal(beta_f=1.0, dbeta=0.02, theta=2, mode="fixed", max_steps=steps)
        r.anneal(beta_f=1.0, dbeta=0.02, theta=0, mode="fixed", max_steps=1)
        r.resample(0.02 * (steps + 2))
        r.sweep(1)
    for x, y in zip(g.download_population(), b.download_population()):
        assert np.array_equal(x, y)
    assert g.observables() == b.observables()


def test_refused_step_keeps_the_population():
    L, R = 32, 100
    print("case interleaved refused step", flush=True)
    spins = inputs.mixed_spins(R, L, seed=5)
    runs = [pa.Run(L, R, seed=41, capacity=R, layout=lay) for lay in ("interleaved", "bits")]
    outcome = []
    for r in runs:
        r.upload_population(spins, step=0, sweeps=0, beta=0.01)
        try:
            r.anneal(beta_f=1.0, dbeta=0.03, theta=1, mode="fixed", max_steps=40)
            outcome.append("done")
        except pa.CapacityError:
            outcome.append("capacity")
    assert outcome[0] == outcome[1]
    assert runs[0].state() == runs[1].state()
    for x, y in zip(runs[0].download_population(), runs[1].download_population()):
        assert np.array_equal(x, y)

"""The last population whose resampling and statistics take one block (4096
replicas) and the first beyond, and steps whose population would exceed the
capacity: they are refused, write no
parent index beyond the capacity's, and leave the run as it was.  The indices
end inside a 256-byte aligned region of the caller's workspace, whose rest is
filled with a pattern before the step and looked at after it; the region is found
by the run's layout and checked by its contents after a step that succeeds."""
import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_1703_03676_amd as pa

pytestmark = pytest.mark.gpu

GUARD = 0xA5


def _parent_region(L, capacity):
    """(first byte, bytes, aligned bytes) of the parent indices: behind two spin
    stores of N/8 bytes per replica with their E and M, and the copy counts."""
    def up(n):
        return (n + 255) // 256 * 256
    before = 2 * (up(capacity * L * L // 8) + 2 * up(4 * capacity)) + up(4 * capacity)
    return before, 4 * capacity, up(4 * capacity)


def _parents(ws, L, capacity, n):
    at, _, _ = _parent_region(L, capacity)
    return ws[at:at + 4 * n].cpu().numpy().view(np.uint32)


def _set_guard(ws, L, capacity):
    at, size, aligned = _parent_region(L, capacity)
    assert aligned > size
    ws[at + size:at + aligned] = GUARD
    torch.cuda.synchronize()


def _check_guard(ws, L, capacity):
    at, size, aligned = _parent_region(L, capacity)
    torch.cuda.synchronize()
    assert bool((ws[at + size:at + aligned] == GUARD).all())


@pytest.mark.parametrize("R", [4096, 4097])
def test_steps_at_the_limit_of_one_block(R):
    print("case one block R=%d" % R, flush=True)
    L = 32
    spins = np.tile(inputs.mixed_spins(241, L, seed=9), (R // 241 + 1, 1, 1))[:R]
    g, o = pa.Run(L, R, seed=5, capacity=2 * R), oracle.Run(L, R, seed=5, capacity=2 * R)
    g.set_stats_path("pass")
    g.upload_population(spins, step=2, sweeps=5, beta=0.2)
    o.set_population(spins, step=2, sweeps=5, beta=0.2)
    for beta in (0.2, 0.202):
        gobs, oobs = g.observables(), o.measure()
        assert all(gobs[k] == oobs[k] for k in ("R", "sumE", "sumE2", "sumAbsM", "sumM2", "sumM4"))
        _, E, M = g.download_population()
        got = pa.observables_static(L, torch.from_numpy(E).cuda(), torch.from_numpy(M).cuda())
        assert all(got[k] == oobs[k] for k in ("R", "sumE", "sumE2", "sumAbsM", "sumM2", "sumM4"))
        gi, oi = g.resample(beta), o.resample(beta)
        assert gi["R_new"] == oi["R_new"] and gi["lnQ"] == oi["lnQ"]
        assert np.array_equal(g.download_counts(g.capacity), o.get_counts())
        for ours, theirs in zip(g.download_population(), o.get_population()):
            assert np.array_equal(ours, theirs)
    g.close()


# 2 R / 3 parents: one block for counts and parents up to 4096 of them (the last
# two sizes are its last and the first beyond)
@pytest.mark.parametrize("call", ["resample", "anneal"])
@pytest.mark.parametrize("R", [70, 1000, 6144, 6146, 9000])
def test_no_parent_beyond_the_capacity(R, call):
    print("case refused step R=%d %s" % (R, call), flush=True)
    L, n = 16, 2 * R // 3
    g = pa.Run(L, R, seed=3, capacity=R + 2)
    s = np.ones((n, L, L), np.int8)  # equal replicas: R_new is about R
    refused = done = 0
    for step in range(1, 25):
        g.upload_population(s, step=step, beta=0.1)
        o = oracle.Run(L, R, seed=3, capacity=4 * R)
        o.set_population(s, step=step, beta=0.1)
        R_new = o.resample(0.3)["R_new"]
        _set_guard(g.workspace, L, g.capacity)
        before = g.state()
        try:
            if call == "resample":
                assert g.resample(0.3)["R_new"] == R_new
            else:
                got = g.anneal(beta_f=0.3, dbeta=0.3 / (step + 1), theta=1, mode="fixed", max_steps=1)
                assert got[0]["R"] == R_new
            assert R_new <= g.capacity
            assert np.array_equal(_parents(g.workspace, L, g.capacity, R_new), np.repeat(np.arange(n), o.get_counts()))
            done += 1
        except pa.CapacityError:
            assert R_new > g.capacity
            assert g.state() == before
            refused += 1
        _check_guard(g.workspace, L, g.capacity)
    assert refused > 0 and done > 0
    g.close()


def test_no_parent_beyond_the_capacity_in_a_batch():
    print("case refused step of a batch", flush=True)
    L, R = 16, 100
    refused = done = 0
    for seed in range(1, 17):
        b = pa.Batch([dict(L=L, R=R, seed=seed, capacity=R, layout="bits")],
                     [dict(beta_f=0.3, dbeta=0.002, theta=1, mode="fixed")])
        o = oracle.Run(L, R, seed=seed, capacity=4 * R)
        o.init()
        R_new = o.resample(0.002)["R_new"]
        _set_guard(b.workspace, L, R)
        b.step()
        _check_guard(b.workspace, L, R)
        if R_new > R:
            assert b.status(0) == pa.PA_ECAPACITY and b.state(0)["step"] == 0
            refused += 1
        else:
            assert b.status(0) == pa.PA_OK and b.state(0)["R"] == R_new
            assert np.array_equal(_parents(b.workspace, L, R, R_new), np.repeat(np.arange(R), o.get_counts()))
            done += 1
        b.close()
    assert refused > 0 and done > 0


def test_refused_step_of_the_interleaved_store():
    # refused in the first, an odd and an even number of steps into the call
    L, R = 32, 100
    spins = inputs.mixed_spins(R, L, seed=5)
    steps = set()
    for seed in range(1, 8):
        print("case interleaved refused step seed=%d" % seed, flush=True)
        runs = [pa.Run(L, R, seed=seed, capacity=R + 6, layout=lay) for lay in ("interleaved", "bits")]
        for r in runs:
            r.upload_population(spins, step=0, sweeps=0, beta=0.0)
            with pytest.raises(pa.CapacityError):
                r.anneal(beta_f=4.0, dbeta=0.01, theta=1, mode="fixed", max_steps=400)
        assert runs[0].state() == runs[1].state()
        steps.add(runs[0].state()["step"])
        for x, y in zip(runs[0].download_population(), runs[1].download_population()):
            assert np.array_equal(x, y)
        for r in runs:  # and they go on alike
            r.sweep(2)
        for x, y in zip(runs[0].download_population(), runs[1].download_population()):
            assert np.array_equal(x, y)
        for r in runs:
            r.close()
    assert any(k % 2 for k in steps) and any(k % 2 == 0 for k in steps)

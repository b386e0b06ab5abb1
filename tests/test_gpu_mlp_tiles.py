"""The proposer's gradient and training at the edges of its kernels: sample
counts around the tiles of 16, more tiles than blocks, workspaces without room
for any block's partial sums or for more than one minibatch's sample order."""
import numpy as np
import pytest

from oracle import mlp

import paper_1703_03676_amd as pa
import torch

pytestmark = pytest.mark.gpu


def _data(seed, n):
    rng = np.random.default_rng(seed)
    params = rng.normal(0, 0.25, mlp.NPARAMS).astype(np.float32)
    norm = np.concatenate([rng.normal(0, 1, 8), rng.uniform(0.5, 2, 8), [-5.0, 1.5]]).astype(np.float32)
    x = (rng.normal(0, 1, (n, 8)) * norm[8:16] + norm[:8]).astype(np.float32)
    t = rng.normal(-5.0, 1.5, n).astype(np.float32)
    return params, norm, x, t


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("n,max_batch", [(1, 1), (15, 15), (16, 16), (17, 17), (17, 40), (33, 64), (1023, 1024),
                                         (1025, 1025), (2500, 3000)])
def test_gradient(n, max_batch):
    # FP32 sums of n terms: error at most n 2^-24 of the sum of their sizes,
    # which random signs keep below the largest entry's scale times sqrt(n)
    print("case mlp gradient n=%d max_batch=%d" % (n, max_batch), flush=True)
    params, norm, x, t = _data(n, n)
    m = pa.Mlp(max_batch=max_batch, seed=1)
    m.set_params(params, norm)
    p, nm, xd, td = (a.astype(np.float64) for a in (params, norm, x, t))
    gr, lr = mlp.gradient(p, nm, xd, td), mlp.loss(p, nm, xd, td)
    for _ in range(2):  # the second call finds the first one's partial sums
        g, loss = m.gradient(_cuda(x), _cuda(t))
        assert np.all(np.abs(g - gr) <= 1e-4 * np.abs(gr).max())
        assert loss == pytest.approx(lr, rel=1e-5)


@pytest.mark.parametrize("n,max_batch", [(40, 40), (100, 128), (300, 512)])
def test_full_batch_training_follows_gradient_descent(n, max_batch):
    print("case mlp full-batch training n=%d" % n, flush=True)
    params, norm, x, t = _data(n, n)
    m = pa.Mlp(max_batch=max_batch, seed=1)
    m.set_params(params, norm)
    losses = m.train(_cuda(x), _cuda(t), batch=n, epochs=4, lr=1e-2, momentum=0.9, seed=2)
    p, nm, xd, td = (a.astype(np.float64) for a in (params, norm, x, t))
    mom = np.zeros_like(p)
    for e in range(4):
        assert losses[e] == pytest.approx(mlp.loss(p, nm, xd, td), rel=1e-4)
        mom = 0.9 * mom + mlp.gradient(p, nm, xd, td)
        p = p - 1e-2 * mom
    # four steps of 1e-2 times a gradient good to 1e-4 of its largest entry
    assert np.abs(m.params()[0] - p).max() <= 4e-5 * max(1.0, np.abs(mom).max())


def test_training_does_not_depend_on_the_room_for_the_order():
    # max_batch = batch: the order of one or two minibatches fits at a time
    print("case mlp order uploads", flush=True)
    n, batch = 1000, 48
    params, norm, x, t = _data(9, n)
    out = []
    for max_batch in (48, 2000):
        m = pa.Mlp(max_batch=max_batch, seed=1)
        m.set_params(params, norm)
        losses = m.train(_cuda(x), _cuda(t), batch=batch, epochs=5, lr=2e-3, momentum=0.9, seed=4)
        out.append((m.params()[0], losses))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])

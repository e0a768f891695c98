"""Loss and gradients of the learned step's training over network and batch
shapes: fewer inputs and outputs than hidden units, remainders of the 16-, 32-
and 64-wide tiles, one row, and a batch smaller than the one laid out for.

Tolerances: a value is an FP32 sum of up to K = 2100 products, whose rounding
errors of varying sign come to about sqrt(K) 2^-24 = 2.7e-6 of its terms: loss
relative 1e-5 (an FP64 mean over many elements), gradients relative Frobenius
1e-4 per tensor (three such products in a chain, and sums that cancel)."""
import numpy as np
import pytest

import workloads as wl
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nin,w,nout,batch,n", [
    (65, 128, 64, 32, 32),
    (20, 96, 7, 16, 16),
    (1, 1, 1, 1, 1),
    (17, 33, 15, 48, 31),
    (16, 16, 16, 16, 16),
    (130, 65, 129, 100, 100),
    (541, 128, 540, 128, 65),
    (37, 1100, 1090, 520, 520),    # 32-wide tiles
    (70, 2050, 2060, 2049, 2049),  # 64-wide tiles
])
def test_loss_and_gradients(nin, w, nout, batch, n):
    import torch
    import paper_2603_12550_amd as vds

    print(f"MLP {nin}-{w}-{w}-{nout}, {n} of {batch} rows", flush=True)
    rng = np.random.default_rng(nin + w + nout + n)
    r32 = lambda a: wl.f32_as_f64(wl.to_f32(a))
    sizes = [nin, w, w, nout]
    layers = [(r32(W), r32(0.1 * rng.standard_normal(b.shape))) for W, b in wl.mlp_init(5, sizes)]
    X, T = r32(rng.standard_normal((n, nin))), r32(rng.standard_normal((n, nout)))
    dev = lambda a: torch.from_numpy(wl.to_f32(a)).cuda()
    m = vds.Mlp(nin, w, nout, batch)
    m.set_params(dev(np.concatenate([np.concatenate([W.reshape(-1), b]) for W, b in layers])))
    loss = m.loss_grad(dev(X), dev(T))
    loss_o, grads_o = omlp.backward(layers, X, T)
    assert loss == pytest.approx(loss_o, rel=1e-5)
    g = m.get_grads().cpu().numpy().astype(np.float64)
    off = 0
    for gW, gb in grads_o:
        for o in (gW, gb):
            v = g[off:off + o.size].reshape(o.shape)
            off += o.size
            assert np.linalg.norm(v - o) <= 1e-4 * np.linalg.norm(o)
    assert off == g.size
    Y_o, _ = omlp.forward(layers, X)
    assert np.linalg.norm(m.forward(dev(X)).cpu().numpy() - Y_o) <= 1e-5 * np.linalg.norm(Y_o)

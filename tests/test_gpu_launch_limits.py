"""Calls so large that a launch with one workgroup per tile would have 2^32 threads or
more in one dimension, of which only the rest would run."""
import math

import pytest

pytestmark = pytest.mark.gpu


def test_density_at_very_many_points():
    """Five blocks of 16 points and 512 threads a workgroup: 2^32 threads from 671088640
    points on.  Tolerance as in the density tests: 1e-4 of the value, 1e-6 of the largest."""
    import torch
    import paper_2603_12550_amd as vds

    ny, P, h = (1 << 32) // 512 * 80 + 1001, 3, 0.7
    print(f"density at {ny} points", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q = torch.randn((1, P, 3), generator=g, device="cuda")
    y = torch.randn((ny, 3), generator=g, device="cuda")
    f = vds.Context(1, P, h).density_at(q, y)
    at = torch.cat([torch.arange(1000), torch.arange(ny - 5000, ny), torch.randint(0, ny, (5000,))]).cuda()
    d2 = ((y[at].double()[:, None] - q[0].double()) ** 2).sum(-1)
    ref = torch.exp(-d2 / (2 * h * h)).sum(1) / P * (2 * math.pi * h * h) ** -1.5
    assert bool(((f[at].double() - ref).abs() <= 1e-4 * ref + 1e-6 * ref.max()).all())


def test_gradients_of_a_very_large_layer():
    """512 threads per 16 x 16 tile, which the narrow last layer's weight gradient asks of
    the whole launch: 2^32 threads for 2^20 rows and 2048 units.  The rows are 256 rows
    over and over, whose mean gradient is that of the 256; both are FP32 sums good to
    some 1e-6 (three chained products of up to 2048 terms): 1e-5 of each tensor."""
    import torch
    import paper_2603_12550_amd as vds

    nin, w, nout, n, few = 16, 2048, 16, 1 << 20, 256
    print(f"gradients: {nin}-{w}-{w}-{nout}, {n} rows", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    par = torch.cat([t.reshape(-1) for t in (rnd(w, nin) / 4, rnd(w), rnd(w, w) / 45, rnd(w), rnd(nout, w) / 45, rnd(nout))])
    X, T = rnd(few, nin), rnd(few, nout)

    def grads(k):
        m = vds.Mlp(nin, w, nout, few * k)
        m.set_params(par)
        return m.loss_grad(X.repeat(k, 1), T.repeat(k, 1)), m.get_grads().double()

    loss_o, ref = grads(1)
    loss, got = grads(n // few)
    assert loss == pytest.approx(loss_o, rel=1e-6)
    at = 0
    for size in (w * nin, w, w * w, w, nout * w, nout):
        v, r = got[at:at + size], ref[at:at + size]
        assert float((v - r).norm()) <= 1e-5 * float(r.norm())
        at += size

"""Weight gradients of batches far beyond the training minibatch, whose sums over the
rows are the longest of the library.

All terms are made positive, so that no error hides in a sum that cancels.  Tolerance:
rows go to FP64 in groups of 256 per wave, in FP32 instructions of 4 rows: 64 roundings
of varying sign, sqrt(64) 2^-25 = 2.4e-7 of the sum; the wave's sum and the result are
rounded once each (2 x 2^-25 = 6e-8), in 64-wide tiles FP32 adds the 64 groups of 2^17
rows (sqrt(64) 2^-25 again); and every term carries what three layers' SiLU,
its derivative and the products round, of which a part (some units of 2^-25) is the same
in all rows: 8e-7 of each tensor's Frobenius norm in all.  One FP32 sum over a wave's
rows would round 32768 times at 2^20 rows, some sqrt(32768) 2^-25 = 5e-6."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nin,w,nout,n", [
    (16, 16, 16, 1 << 20),       # 16-wide tiles
    (20, 24, 40, 300001),        # remainders of tiles, rounds and groups
    (32, 768, 768, 1 << 17),     # 32-wide tiles
    (24, 2048, 2060, 1 << 17),   # 64-wide tiles
    (64, 16, 16, 2049), (64, 16, 16, 4097),  # one group of rows per wave, and just more
])
def test_weight_gradients_of_many_rows(nin, w, nout, n):
    import torch
    import paper_2603_12550_amd as vds

    print(f"weight gradients: {nin}-{w}-{w}-{nout}, {n} rows", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(nin + n)
    rand = lambda *s: torch.rand(s, generator=g, device="cuda")
    W = [(rand(w, nin) + 0.2) / nin, rand(w), (rand(w, w) + 0.2) / w, rand(w), (rand(nout, w) + 0.2) / w, rand(nout)]
    X, T = rand(n, nin) + 0.5, -1.0 - 2.0 * rand(n, nout)
    m = vds.Mlp(nin, w, nout, n)
    m.set_params(torch.cat([t.reshape(-1) for t in W]))
    loss = m.loss_grad(X, T)
    D = [t.double() for t in W]

    def silu(z):
        s = torch.sigmoid(z)
        return z * s, s * (1 + z * (1 - s))

    ref, ref_loss = [torch.zeros_like(t) for t in D], 0.0
    for i in range(0, n, 1 << 15):
        x, t = X[i:i + (1 << 15)].double(), T[i:i + (1 << 15)].double()
        a1, s1 = silu(x @ D[0].T + D[1])
        a2, s2 = silu(a1 @ D[2].T + D[3])
        d = a2 @ D[4].T + D[5] - t
        ref_loss += float((d * d).sum())
        d3 = 2 * d / (n * nout)
        d2 = (d3 @ D[4]) * s2
        d1 = (d2 @ D[2]) * s1
        for k, v in enumerate((d1.T @ x, d1.sum(0), d2.T @ a1, d2.sum(0), d3.T @ a2, d3.sum(0))):
            ref[k] += v
    assert loss == pytest.approx(ref_loss / (n * nout), rel=1e-6)
    v, err = m.get_grads().double(), []
    for r in ref:
        err.append(float((v[:r.numel()].reshape(r.shape) - r).norm() / r.norm()))
        v = v[r.numel():]
    print("errors", ["%.1e" % e for e in err], flush=True)
    assert max(err) <= 8e-7

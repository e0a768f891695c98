"""A Gram matrix of snapshots that are not numbers: NaN where FP32 makes them NaN, and
about as fast as any other (what is not a number costs no second pass over the rest of
its column)."""
import pytest

pytestmark = pytest.mark.gpu


def test_gram_of_nan_snapshots():
    import torch
    import paper_2603_12550_amd as vds

    m, n = 60000, 300
    print(f"Gram matrices of {m} x {n} with and without NaN", flush=True)
    ctx = vds.Context(1, m // 3, 0.4)
    X = torch.randn((n, m), device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    one = X.clone()
    one[7, m - 3] = float("nan")
    every = torch.full_like(X, float("nan"))

    def gram(x):
        ctx.pod_gram(x)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        G = ctx.pod_gram(x)
        b.record()
        b.synchronize()
        return G, a.elapsed_time(b)

    (G, t), (G1, t1), (Gn, tn) = gram(X), gram(one), gram(every)
    print(f"{t:.3f} ms, one NaN {t1:.3f}, all NaN {tn:.3f}", flush=True)
    row = torch.zeros((n, n), dtype=torch.bool, device="cuda")
    row[7], row[:, 7] = True, True
    assert torch.equal(G1.isnan(), row) and torch.equal(G1[~row], G[~row])
    assert bool(Gn.isnan().all())
    assert tn <= 4 * t  # 405000 sums of 60000 terms one after the other take a thousand times as long

"""Density at given points where its one-pass form changes shape: remainders of
16 points and of 32 particles, few points against many particles (columns split
over workgroups), many points (two to five row blocks a wave), points far outside.

Tolerance: an FP32 sum of positive terms in groups of 16, the groups in FP64;
each term's exponent (up to 40 here at any point that counts) is formed to 2^-24
of its largest product, |x|^2 / (2 h^2) <= 100, so a term is good to
100 x 2^-24 x ln 2 x a few = 2e-5; 1e-4 of the value, or 1e-6 of the largest one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,P,ny", [
    (1, 1, 1), (1, 33, 17), (2, 257, 1), (3, 8193, 15), (2, 70001, 100), (3, 300, 8192), (1, 100, 8193),
    (2, 65, 12289), (5, 70, 16385), (3, 33, 20481), (4, 16500, 31), (5, 999, 513),
])
def test_density_shapes(nb, P, ny):
    import torch
    import paper_2603_12550_amd as vds

    D, h = 3 * nb, 0.7
    print(f"density: D = {D}, P = {P}, {ny} points", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(nb * 1000 + ny)
    q = torch.randn((nb, P, 3), generator=g, device="cuda")
    y = 0.8 * torch.randn((ny, D), generator=g, device="cuda")
    if ny > 16:
        y[3] = 1e4
    f = vds.Context(nb, P, h).density_at(q, y).double()
    x = q.permute(1, 0, 2).reshape(P, D).double()
    yd = y.double()
    ref = torch.empty(ny, dtype=torch.float64, device="cuda")
    for i in range(0, ny, 512):
        d2 = ((yd[i:i + 512, None, :] - x[None]) ** 2).sum(-1) if P * 512 * D < 2e8 else torch.stack(
            [((v - x) ** 2).sum(-1) for v in yd[i:i + 512]])
        ref[i:i + 512] = torch.exp(-d2 / (2 * h * h)).sum(1) / P * (2 * np.pi * h * h) ** (-D / 2)
    err = (f - ref).abs()
    assert bool(torch.isfinite(f).all())
    assert bool((err <= 1e-4 * ref + 1e-6 * ref.max()).all()), float((err / (ref + 1e-2 * ref.max())).max())

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

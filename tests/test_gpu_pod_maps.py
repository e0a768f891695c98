"""Projection and reconstruction over shapes: each number of bonds, ranks about
the groups of 8 rows and the four waves' quarters, positions about the groups of
64 and 256, a rank above the number of positions' groups, one particle; on both sides
of what one launch projects (256 rows; 73728 numbers of a row and its bonds) and of its
trips of 8192 positions.

Tolerance: FP32 products summed in FP32 over at most K = R / 4 + 4 terms
(reconstruction) or the positions of a chunk (projection), whose rounding errors
of varying sign come to about sqrt(K) 2^-24 < 1e-5 of the terms' norm: 1e-5 of
|U_row| |p| and of |U_col| |q|."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,P,R", [
    (1, 1, 1), (1, 1, 3), (2, 21, 5), (3, 85, 8), (4, 86, 9), (5, 1001, 17), (3, 64, 63), (2, 333, 130),
    (1, 30011, 3), (3, 7013, 65), (3, 20, 700),
    (1, 2730, 256), (1, 2731, 257), (2, 8192, 4), (2, 8193, 4), (4, 4915, 255), (4, 4916, 9), (5, 342, 257), (5, 341, 6),
])
def test_map_shapes(nb, P, R):
    import torch
    import paper_2603_12550_amd as vds

    print(f"POD maps: nb = {nb}, P = {P}, R = {R}", flush=True)
    m = 3 * P
    g = torch.Generator(device="cuda")
    g.manual_seed(R)
    U = torch.randn((R, m), generator=g, device="cuda")
    q = torch.randn((nb, P, 3), generator=g, device="cuda")
    p0 = torch.randn((nb, R), generator=g, device="cuda")
    ctx = vds.Context(nb, P, 0.5)
    p = ctx.pod_project(U, q).double()
    Ud, qd = U.double(), q.reshape(nb, m).double()
    bound = qd.norm(dim=1)[:, None] * Ud.norm(dim=1)[None]
    assert bool(((p.reshape(nb, R) - qd @ Ud.T).abs() <= 1e-5 * bound).all())
    r = ctx.pod_reconstruct(U, p0).double().reshape(nb, m)
    bound = p0.double().norm(dim=1)[:, None] * Ud.norm(dim=0)[None]
    assert bool(((r - p0.double() @ Ud).abs() <= 1e-5 * bound).all())

"""Reduced explicit Euler steps with frozen operators, at the edges of the ranks
and for every number of bonds that the resident stepper is made for, against FP64
steps with the same operators.

Tolerance: a step rounds the state to 2^-24 of itself a few times and adds
dt times a sum of R products; 40 steps make at most 40 x 4 x 2^-24 = 1e-5 of the
state's norm even if every rounding pointed the same way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,R", [(1, 1), (2, 16), (3, 17), (4, 32), (5, 33), (3, 48), (3, 49), (1, 64), (2, 65),
                                  (5, 96), (3, 97), (4, 128), (3, 129), (5, 192), (1, 192), (2, 193)])
def test_steps_with_frozen_operators(nb, R):
    import torch
    import paper_2603_12550_amd as vds

    P, n, dt, zeta, kT = 96, 40, 2e-3, 4.0, 1.0
    print(f"reduced steps: nb = {nb}, R = {R}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * R + nb)
    U = torch.linalg.qr(torch.randn((3 * P, R), generator=g, device="cuda", dtype=torch.float64))[0].T
    U = U.float().contiguous()
    p0 = torch.randn((nb, R), generator=g, device="cuda")
    H = np.linspace(0.7, 1.3, nb)
    G = np.zeros((3, 3))
    G[0, 1] = 1.0
    ctx = vds.Context(nb, P, 1.0, H=H, G=G, dt=dt, zeta=zeta, kT=kT, scheme="explicit")
    rom = vds.Rom(ctx, U)
    XH, XB1, XB2 = (t.double().reshape(R, R) for t in rom.operators(p0))
    XB = XB1 + XB2
    p = p0.clone()
    rom.run(p, n, n)
    A = 2.0 * torch.eye(nb, dtype=torch.float64, device="cuda")
    for k in range(nb - 1):
        A[k, k + 1] = A[k + 1, k] = -1.0
    Hd = torch.from_numpy(H).cuda()[:, None]
    x = p0.double()
    for _ in range(n):
        x = x + dt * (x @ XH.T - kT / zeta * (A @ x) @ XB.T - A @ (Hd * x) / zeta)
    assert float((p.double() - x).norm()) <= 1e-5 * float(x.norm())

"""Batched steps where the column ranges of an ensemble change: one particle, one
range and two (256, 257 particles), as many as there can be (4096, 4097), ranges
longer than the shortest, and both sides of the rows (196608) from which the ensembles
stay whole.

Tolerances as in the other batch tests: states 1e-5, stress 1e-4, relative to the
FP64 oracle."""
import numpy as np
import pytest

import workloads as wl
from oracle import vds as ovds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,rb,P", [
    (1, 2, [256, 1, 257, 4096, 31]), (3, 2, [4097, 255, 513, 33, 2]), (3, 1, [257, 1025, 256]), (5, 2, [1, 300, 2049]),
    (3, 2, [11777, 700, 1]), (2, 2, [350] * 383), (2, 2, [350] * 384),
])
def test_batch_column_ranges(nb, rb, P):
    import torch
    import paper_2603_12550_amd as vds

    print(f"batch nb = {nb} rb = {rb} P = {P[:5]}", flush=True)
    n, h = len(P), 0.6
    G = np.stack([wl.shear_gradient(1.0 + e % 5) for e in range(n)])
    states = [wl.gaussian_bonds(70 + e, nb, p, 1 / 3) for e, p in enumerate(P)]
    b = vds.Batch(P, [h] * n, G, nb=nb, poison=True)
    b.set_tuning(rb, 1024)
    q = b.pack([torch.from_numpy(wl.to_f32(s)).cuda() for s in states])
    tau = b.step(q, nsteps=2, stress=True)
    out = b.unpack(q)
    for e in range(n if n < 10 else 3):
        w, prob = ovds.uniform_weights(P[e]), ovds.Problem(nb=nb, h=h, dt=1e-3, G=G[e])
        x = wl.f32_as_f64(wl.to_f32(states[e]))
        for _ in range(2):
            x = ovds.step_explicit(x, w, prob, threads=8)
        assert np.linalg.norm(out[e].cpu().numpy() - x) <= 1e-5 * np.linalg.norm(x), e
        t = ovds.stress(x, w, prob)
        assert np.linalg.norm(tau[e] - t) <= 1e-4 * np.linalg.norm(t), e

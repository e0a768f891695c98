"""Pair sums of the general default pair kernel where its launch changes: one row block
per wave (4097 to 9216 particles, and D >= 12) and two (above), at remainders of 32 columns,
64 and 256, and of a row group, for several grids; and with particles far from the rest.

Tolerances as in the particle tests: S 1e-5 relative, Brownian term 1e-5 of the 2-norm
and 1e-4 per row; with far particles, whose own terms vanish, 1e-5 of the norm of all rows
for each row (their weights among the others are FP32 zeros on both sides)."""
import math

import numpy as np
import pytest

import workloads as wl
from oracle import vds as ovds

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(wl.to_f32(a)).cuda()


def _sums(nb, P, h, q, w, shapes):
    import paper_2603_12550_amd as vds
    ctx = vds.Context(nb, P, h, poison=True, scheme="explicit")
    for rb, sp in shapes:
        print(f"pair sums nb={nb} P={P} rb={rb} splits={sp}", flush=True)
        ctx.set_tuning(4, rb, sp)
        S, t1, t2 = (t.cpu().numpy().astype(np.float64) for t in ctx.pair_sums(_dev(q), _dev(w)))
        yield (rb, sp), S, t1 + t2


@pytest.mark.parametrize("P", [9217, 9249, 9473, 9729])
@pytest.mark.parametrize("nb", [1, 2, 3])
def test_two_row_blocks(nb, P):
    q = wl.f32_as_f64(wl.to_f32(wl.gaussian_bonds(500 + P, nb, P, 0.5)))
    w = wl.f32_as_f64(wl.to_f32(wl.random_weights(11 + P, P)))
    S_o, t1_o, t2_o = ovds.brownian_terms(ovds.particle_major(q), w, 0.6, threads=8)
    b_o = ovds.bond_major(t1_o + t2_o, nb)
    den = np.sqrt((b_o ** 2).sum((0, 2)))
    for shape, S, b in _sums(nb, P, 0.6, q, w, [(2, 1), (2, 4), (2, 7), (2, 16), (1, 4)]):
        num = np.sqrt(((b - b_o) ** 2).sum((0, 2)))
        assert np.abs(S / S_o - 1).max() <= 1e-5, shape
        assert (num <= 1e-4 * den).all() and np.linalg.norm(num) <= 1e-5 * np.linalg.norm(den), shape


@pytest.mark.parametrize("nb,P", [(1, 4500), (3, 5001), (5, 4500), (1, 9473), (2, 9473), (3, 9473), (4, 9473)])
def test_far_particles(nb, P):
    h = 0.45
    q64 = wl.gaussian_bonds(41 + nb, nb, P, 0.5)
    far = np.array([5, 6, 333, 700, P - 1])
    d = np.random.default_rng(9).normal(size=(nb, far.size, 3))
    q64[:, far, :] += 9.0 * d / np.sqrt((d ** 2).sum(axis=(0, 2)))[None, :, None]  # |offset| = 9 in R^D
    q = wl.f32_as_f64(wl.to_f32(q64))
    w = wl.f32_as_f64(wl.to_f32(wl.random_weights(17, P)))
    x = ovds.particle_major(q)
    xc = x - (w[:, None] * x).sum(axis=0)
    assert (math.log2(math.e) / (2 * h * h) * (xc ** 2).sum(axis=1))[far].min() > 150
    S_o, t1_o, t2_o = ovds.brownian_terms(x, w, h, threads=8)
    b_o = ovds.bond_major(t1_o + t2_o, nb)
    for shape, S, b in _sums(nb, P, h, q, w, [(1, 1), (2, 4), (2, 8)]):
        assert np.abs(S / S_o - 1).max() <= 1e-5, shape
        row = np.sqrt(((b - b_o) ** 2).sum((0, 2)))
        assert np.linalg.norm(row) <= 1e-5 * np.linalg.norm(b_o), shape
        assert row.max() <= 1e-5 * np.linalg.norm(b_o), shape

"""GPU parity of the kernels that take FP32 products from three BF16 parts, at
the edges of their tiles, against the FP64 oracle.

Tolerances: as in the particle tests, 1e-5 of the 2-norm and 1e-4 per row (the
parts hold FP32's 24 bits; what rounds is the FP32 accumulation, over fewer
terms at a time than in the forms those bounds were set for).
"""
import numpy as np
import pytest

import workloads as wl
from oracle import vds as ovds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    import paper_2603_12550_amd as pkg
    return pkg


def _dev(a):
    import torch
    return torch.from_numpy(wl.to_f32(a)).cuda()


def _check_rows(b, b_o, S, S_o, label):
    num = np.sqrt(((b - b_o) ** 2).sum((0, 2)))
    den = np.sqrt((b_o ** 2).sum((0, 2)))
    print(label, "max row rel", (num / den).max(), "S", np.abs(S / S_o - 1).max(), flush=True)
    assert (num <= 1e-4 * den).all()
    assert np.linalg.norm(num) <= 1e-5 * np.linalg.norm(den)
    assert np.abs(S / S_o - 1).max() <= 1e-5


# chunk (32 columns), stage (64), accumulation group (256) and row group (16; 128, 256) edges, on both sides of
# the size (4096) up to which a pass and what follows it are one launch
@pytest.mark.parametrize("P", [31, 32, 33, 65, 257, 513, 2047, 2048, 2049, 2305, 4095, 4096, 4097, 4129, 4353, 4609])
@pytest.mark.parametrize("nb,rb", [(1, 2), (2, 1), (2, 2), (3, 1), (3, 2), (4, 2), (5, 2)])
def test_pair_sums_tile_edges(lib, P, nb, rb):
    q = wl.f32_as_f64(wl.to_f32(wl.gaussian_bonds(300 + P, nb, P, 0.5)))
    w = wl.f32_as_f64(wl.to_f32(wl.random_weights(9 + P, P)))
    S_o, t1_o, t2_o = ovds.brownian_terms(ovds.particle_major(q), w, 0.6)
    ctx = lib.Context(nb, P, 0.6, poison=True, scheme="explicit")
    for sp in (1, 4, 8):
        ctx.set_tuning(rows_per_wave=rb, col_splits=sp)
        S, t1, t2 = (t.cpu().numpy().astype(np.float64) for t in ctx.pair_sums(_dev(q), _dev(w)))
        _check_rows(t1 + t2, ovds.bond_major(t1_o + t2_o, nb), S, S_o, f"P={P} nb={nb} rb={rb} sp={sp}")


# both sides of the size up to which a wave takes one row block whatever the tuning says
@pytest.mark.parametrize("P", [9216, 9217])
def test_pair_sums_row_block_line(lib, P):
    test_pair_sums_tile_edges(lib, P, 3, 2)


# tile (96), round (32 k) and split edges, rows that do and do not start on 16 bytes
@pytest.mark.parametrize("m,n", [(3, 2), (31, 96), (33, 97), (129, 1), (600, 95), (1999, 193), (6001, 40), (20000, 300)])
def test_gram_tile_edges(lib, m, n):
    import torch
    g = torch.Generator().manual_seed(m + n)
    X = torch.randn((n, m), generator=g) * torch.logspace(-3, 3, n)[:, None]
    ctx = lib.Context(1, max(1, m // 3), 1.0)
    G = ctx.pod_gram(X.cuda()).cpu().double()
    Xd = X.double()
    ref = Xd @ Xd.T
    # FP32 accumulation against the entry's own scale |x_i| |x_j|: a few 2^-24 per round of 32 within a split
    scale = Xd.norm(dim=1)[:, None] * Xd.norm(dim=1)[None, :]
    err = ((G - ref).abs() / scale).max().item()
    print(f"m={m} n={n} err {err:.2e}", flush=True)
    assert err <= 1e-6 and torch.equal(G, G.T)


def test_gram_of_infinite_snapshots(lib):
    """Entries with an infinite factor are what FP32 arithmetic makes of them."""
    import torch
    g = torch.Generator().manual_seed(1)
    X = torch.randn((5, 200), generator=g)
    X[1, 7] = float("inf")
    X[3, 9] = float("-inf")
    X[4, 11] = 3.4e38
    G = lib.Context(1, 66, 1.0).pod_gram(X.cuda()).cpu().numpy()
    with np.errstate(all="ignore"):
        ref = np.zeros((5, 5), np.float32)
        for k in range(200):
            ref += np.outer(X[:, k].numpy(), X[:, k].numpy())
    assert (np.isnan(G) == np.isnan(ref)).all() and (G[np.isinf(ref)] == ref[np.isinf(ref)]).all()
    ok = np.isfinite(ref)
    assert np.allclose(G[ok], ref[ok], rtol=1e-5, atol=1e-4)

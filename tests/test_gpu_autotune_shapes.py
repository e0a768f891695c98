"""The autotuners time the launches that steps run, each once: no shape of small
problems, which have one, and no second row block where it counts as the first."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,P", [(1, 1), (3, 4096), (3, 4097), (2, 9216), (2, 9217), (4, 9300)])
def test_autotuned_shape_is_one_of_those_that_differ(nb, P):
    import torch
    import paper_2603_12550_amd as vds

    print(f"autotune nb = {nb}, P = {P}", flush=True)
    ctx = vds.Context(nb, P, 0.6)
    q = torch.from_numpy(wl.to_f32(wl.gaussian_bonds(5, nb, P, 0.5))).cuda()
    ctx.set_tuning(rows_per_wave=2, col_splits=7)
    t = ctx.autotune(q)
    if P <= 4096:
        assert (t["rows_per_wave"], t["col_splits"]) == (2, 7)
    elif P <= 9216 or nb >= 4:
        assert t["rows_per_wave"] == 1
    else:
        assert t["rows_per_wave"] in (1, 2)


@pytest.mark.parametrize("nb,P,rows", [(3, [300, 700], (1,)), (5, [8000] * 24, (1,)), (2, [8000] * 24, (1, 2))])
def test_autotuned_batch_shape(nb, P, rows):
    import torch
    import paper_2603_12550_amd as vds

    print(f"batch autotune nb = {nb}, {len(P)} ensembles", flush=True)
    b = vds.Batch(P, [0.6] * len(P), [wl.shear_gradient(1.0)] * len(P), nb=nb)
    q = b.pack([torch.from_numpy(wl.to_f32(wl.gaussian_bonds(e, nb, p, 0.5))).cuda() for e, p in enumerate(P)])
    assert b.autotune(q)["rows_per_wave"] in rows
    b.step(q)
    assert bool(torch.isfinite(q).all())

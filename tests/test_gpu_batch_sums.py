"""An ensemble's step does not depend on how the batch cuts its columns.

The same states alone in a batch (column ranges) and among so many others that every
ensemble is one range.  The ranges are whole FP32 accumulation groups and their sums are
FP64, so that only the order of FP64 additions differs: an FP32 rounding of one of the
numbers behind a coordinate (some hundred) turns out differently once in about 1e7
coordinates, taking 2^-53 of terms up to 100 times the sum against 2^-24.  Up to 3 of
the some 50000 coordinates may differ, by one unit of FP32 of the largest.  A time step
of 1 makes the drift, not the state, what a coordinate holds."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,P", [(3, [4097, 300, 1025]), (1, [4609, 513, 257]), (5, [3000, 31, 2049])])
def test_ensembles_do_not_depend_on_the_batch(nb, P):
    import torch
    import paper_2603_12550_amd as vds

    print(f"batch composition: nb = {nb}, P = {P}", flush=True)
    full = P + [4097] * 46
    states = [torch.from_numpy(wl.to_f32(wl.gaussian_bonds(50 + e, nb, p, 1 / 3))).cuda() for e, p in enumerate(full)]
    G = wl.shear_gradient(1.0)

    def step(n):
        b = vds.Batch(full[:n], [0.5] * n, [G] * n, nb=nb, dt=1.0)
        q = b.pack(states[:n])
        b.step(q)
        return [t.clone() for t in b.unpack(q)[:len(P)]]

    differ = 0
    for x, y in zip(step(len(P)), step(len(full))):
        assert bool(torch.isfinite(x).all())
        gap, top = float((x - y).abs().max()), float(x.abs().max())
        assert gap <= 2.0 ** -23 * top
        differ += int((x != y).sum())
    print(f"{differ} coordinates differ", flush=True)
    assert differ <= 3

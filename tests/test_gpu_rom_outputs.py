"""Stress histories of a reduced run on both sides of the 56 that one block of result
memory holds: bit for bit the first entries of a longer one (the same launches on the
same states), each of its own step, the last one the stress of the final state."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_stress_history_lengths():
    import torch
    import paper_2603_12550_amd as vds

    P, R, nb = 96, 8, 2
    g = torch.Generator(device="cuda").manual_seed(3)
    U = torch.linalg.qr(torch.randn((3 * P, R), generator=g, device="cuda", dtype=torch.float64))[0].T.float().contiguous()
    p0 = torch.randn((nb, R), generator=g, device="cuda")
    G = np.zeros((3, 3))
    G[0, 1] = 1.0
    ctx = vds.Context(nb, P, 1.0, G=G, dt=1e-2, scheme="explicit")
    rom = vds.Rom(ctx, U)

    def history(n):
        print(f"{n} outputs", flush=True)
        p = p0.clone()
        h = rom.run(p, n, 1000, output_every=1)
        assert np.array_equal(h[-1], rom.stress(p))
        return h

    whole = history(169)
    assert np.isfinite(whole).all() and (np.abs(np.diff(whole, axis=0)).max(axis=(1, 2)) > 0).all()
    for n in (1, 55, 56, 57, 111, 112, 113, 168):
        assert np.array_equal(history(n), whole[:n])


@pytest.mark.parametrize("other", [0, 1, 2, 3])
def test_operators_after_another_form(other):
    """The basis parts that the default form keeps with a model are laid out again after
    another form has used their memory, also if the model was made under that form."""
    import torch
    import paper_2603_12550_amd as vds

    P, R, nb = 700, 20, 3
    print(f"operators: default, form {other}, default", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    U = torch.linalg.qr(torch.randn((3 * P, R), generator=g, device="cuda", dtype=torch.float64))[0].T.float().contiguous()
    p = torch.randn((nb, R), generator=g, device="cuda")
    ctx = vds.Context(nb, P, 1.0, scheme="explicit")
    tuned = lambda impl: ctx.set_tuning(impl, 2 if impl != 1 else 1, 4)
    first = vds.Rom(ctx, U)
    want = [t.clone() for t in first.operators(p)]
    tuned(other)
    second = vds.Rom(ctx, U)
    for rom in (first, second):
        for a, b in zip(rom.operators(p), want):
            assert float((a - b).norm()) <= 1e-4 * float(b.norm())  # as against the oracle
    tuned(4)
    for rom in (first, second):
        assert all(torch.equal(a, b) for a, b in zip(rom.operators(p), want))

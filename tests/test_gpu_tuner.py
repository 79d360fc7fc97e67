"""The launch-shape tuner keeps a choice per lattice and launch form: lattices of
equal volume and other extents (a candidate visits tiles of z and t) are tuned
by themselves, launches over one parity and over both and with internal and
canonical output too, and no two lines of the report stand for the same launch.
Results do not change."""
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")


def test_choices_per_extents_and_form():
    specs = [((4, 4, 8, 12), -1), ((8, 12, 4, 4), -1)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    with w.Context(specs) as ctx:
        v = []
        for l, (dims, _) in enumerate(specs):
            ctx.set_gauge(inputs.gauge_field_torch(dims, 0.3, 87 + l, device="cuda"), lat=l)
            ctx.set_clover(0.1, 1.0, lat=l)
            shape = (5,) + tuple(reversed(dims)) + (4, 3)
            v.append(torch.complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64),
                                   torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)))

        def applies():
            return [ctx.apply_D(v[l], op, w.F32, lat=l) for l in (0, 1) for op in (w.OP_FULL, w.OP_SCHUR)]

        plain = applies()
        ctx.autotune(True)
        tuned = applies()
        rep = ctx.autotune_report()
    assert all(torch.equal(a, b) for a, b in zip(plain, tuned))
    lines = [tuple(r[k] for k in ("prec", "diag", "postinv", "nrhs", "form", "Lx", "Ly", "Lz", "Lt")) for r in rep]
    assert len(set(lines)) == len(lines)
    for dims, _ in specs:
        mine = [r for r in rep if (r["Lx"], r["Ly"], r["Lz"], r["Lt"]) == dims]
        assert sorted(r["form"] for r in mine) == [0, 2, 3]  # first hop of D_r, its last, D
        assert all(r["Vh"] == 768 and r["nrhs"] == 5 and r["us"] > 0 for r in mine)

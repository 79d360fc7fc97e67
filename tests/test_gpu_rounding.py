"""Rounding of FP64 results against extended precision (64-bit mantissa).

An entry is a sum of many products; only what is rounded at the size of the
result counts (u / sqrt 3 each, u = 2^-53), and the kernels keep that to a few
roundings: short sums from zero, added in a tree or in two words.  Bounds on
the relative error (Frobenius):

* link force with and without its clover part: eight (the six sides of a link
  added one by one, the two halves of the hop), 1.63 u.
"""
import numpy as np
import pytest
import torch

import inputs
from oracle import force as F
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

U = 2.0 ** -53


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 4, 2, 8)])
def test_force(dims, monkeypatch):
    V = int(np.prod(dims))
    links = inputs.gauge_field(dims, 0.4, 85)
    op = WilsonClover(dims, links, -0.1, 1.0, -1)
    rng = np.random.default_rng(12)
    x, lam = (rng.standard_normal((V, 4, 3)) + 1j * rng.standard_normal((V, 4, 3)) for _ in range(2))
    with w.Context([(dims, -1)]) as ctx:
        ctx.set_gauge(torch.from_numpy(links).cuda())
        ctx.set_clover(-0.1, 1.0)
        shape = (1,) + tuple(reversed(dims)) + (4, 3)
        got = {c: ctx.force(torch.from_numpy(x.reshape(shape)).cuda(), torch.from_numpy(lam.reshape(shape)).cuda(),
                            c).cpu().numpy().reshape(V, 4, 3, 3) for c in (True, False)}
    op.U = op.U.astype(np.clongdouble)
    monkeypatch.setattr(np, "complex128", np.clongdouble)  # what the oracle accumulates in
    for c in (True, False):
        want = F.force(op, x.astype(np.clongdouble), lam.astype(np.clongdouble), c)
        assert want.dtype == np.clongdouble
        err = float(np.linalg.norm((got[c] - want).astype(complex)) / np.linalg.norm(want.astype(complex)))
        print(dims, c, err / U, flush=True)
        assert err < np.sqrt(8 / 3) * U, (c, err / U)

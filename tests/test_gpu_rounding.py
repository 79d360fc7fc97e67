"""Rounding of FP64 results against extended precision (64-bit mantissa).

An entry is a sum of many products; only what is rounded at the size of the
result counts (u / sqrt 3 each, u = 2^-53), and the kernels keep that to a few
roundings: short sums from zero, added in a tree or in two words.  Bounds on
the relative error (Frobenius):

* restriction of one vector and of batches (matrix instructions), with the
  null vectors as prolongation gives them, blocks of 16 to 1024 sites: twelve
  roundings (the products of a lane's units, six to eight levels of sums), 2 u;
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


def split(v, dims, block):
    """[n][Lt][Lz][Ly][Lx][4][3] -> [n][blocks][2][sites x 6]"""
    nb = [d // b for d, b in zip(dims, block)]
    n = v.shape[0]
    v = v.reshape(n, nb[3], block[3], nb[2], block[2], nb[1], block[1], nb[0], block[0], 2, 6)
    return v.transpose(0, 1, 3, 5, 7, 9, 2, 4, 6, 8, 10).reshape(n, int(np.prod(nb)), 2, -1)


@pytest.mark.parametrize("dims,block,nvec", [((8, 8, 4, 8), (4, 4, 4, 4), 17), ((8, 8, 8, 8), (8, 8, 4, 4), 5),
                                             ((4, 8, 8, 8), (4, 4, 4, 4), 33), ((8, 4, 4, 8), (4, 4, 4, 4), 64),
                                             ((8, 8, 8, 4), (2, 2, 2, 2), 5), ((8, 8, 8, 4), (2, 2, 2, 2), 20)])
def test_restriction(dims, block, nvec):
    rng = np.random.default_rng(11)
    cplx = lambda s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    shape = tuple(reversed(dims)) + (4, 3)
    f = cplx((12,) + shape)
    with w.Context(dims) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(dims, 0.3, 84)).cuda())
        ctx.set_clover(0.1, 1.0)
        ctx.set_mg_params(w.default_params(block=[block], nvec=[nvec]))
        ctx.set_null_vectors(torch.from_numpy(cplx((nvec,) + shape)).cuda())
        ctx.build_coarse()
        nb = int(np.prod(ctx.coarse_dims()))
        unit = np.zeros((nvec, nb, 2, nvec), dtype=np.complex128)
        for k in range(nvec):
            unit[k, :, :, k] = 1.0
        V = split(ctx.prolong(torch.from_numpy(unit.reshape(nvec, nb, 2 * nvec)).cuda()).cpu().numpy(), dims, block)
        fs = split(f, dims, block).astype(np.clongdouble)
        want = np.stack([(V[k].conj().astype(np.clongdouble) * fs).sum(-1) for k in range(nvec)], -1)
        want[:, :, 1] *= -1
        for n in (1, 2, 8, 9, 12):
            got = ctx.restrict(torch.from_numpy(f[:n]).cuda()).cpu().numpy().reshape(n, nb, 2, nvec)
            err = float(np.linalg.norm((got - want[:n]).astype(complex)) / np.linalg.norm(want[:n].astype(complex)))
            print(dims, nvec, n, err / U, flush=True)
            assert err < 2 * U, (n, err / U)


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

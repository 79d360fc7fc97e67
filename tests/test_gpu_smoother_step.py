"""The cycle with 0, 1, 2 and 4 smoothing steps against the cycle written out:
restriction, dense inverse of the coarse operator, prolongation, minimal-
residual steps on the even half.  After one outer step the solution is that
cycle's result times the outer step's coefficient, so a missing, doubled or
wrong last step shows itself, alone and in a batch.

Tolerances: FP64 the rounding of some ten operator applies, times the condition
of the coarse operator (1e3), 1e-11; FP32 (smoother, transfers and the applied
inverse) the same number of roundings at 6e-8, 1e-4 with that condition.  The
result without the last step is further off than a hundred times that.
"""
import numpy as np
import pytest
import torch

import inputs
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS, NVEC, M0 = (4, 4, 4, 6), 4, 0.1


@pytest.mark.parametrize("prec,tol", [("F64", 1e-11), ("F32", 1e-4)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_cycle_with_smoothing(nrhs, prec, tol):
    links = inputs.gauge_field(DIMS, 0.3, 63)
    op = WilsonClover(DIMS, links, M0, 1.0)
    even, odd = op.lat.even, op.lat.odd
    rng = np.random.default_rng(9)
    shape = tuple(reversed(DIMS)) + (4, 3)

    def cplx(s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    b = cplx((nrhs,) + op.shape)
    b[:, odd] = 0.0
    bt = torch.from_numpy(b.reshape((nrhs,) + shape)).cuda()
    with w.Context(DIMS) as ctx:
        ctx.set_gauge(torch.from_numpy(links).cuda())
        ctx.set_clover(M0, 1.0)

        def params(nu):
            return w.default_params(block=[(2, 2, 2, 2)], nvec=[NVEC], nu_post=nu, smoother_prec=getattr(w, prec),
                                    coarsest=1, outer_max_iter=1)

        ctx.set_mg_params(params(1))
        vecs = torch.from_numpy(cplx((NVEC,) + shape)).cuda()
        ctx.set_null_vectors(vecs)
        ctx.build_coarse()
        rhs = ctx.restrict(bt)
        n = rhs[0].numel()
        unit = torch.eye(n, dtype=torch.complex128, device="cuda").reshape((n,) + rhs.shape[1:])
        Y = ctx.apply_coarse(unit).reshape(n, n).cpu().numpy().T
        c = np.linalg.solve(Y, rhs.reshape(nrhs, n).cpu().numpy().T).T
        e0 = ctx.prolong(torch.from_numpy(c.reshape(rhs.shape)).cuda()).cpu().numpy().reshape((nrhs,) + op.shape)
        for nu in (0, 1, 2, 4):
            ctx.set_mg_params(params(nu))
            ctx.set_null_vectors(vecs)
            ctx.build_coarse()
            x = ctx.solve(bt, w.MG_GCR, 1e-10, raise_on_error=False)[0].cpu().numpy().reshape((nrhs,) + op.shape)
            for r in range(nrhs):
                e = e0[r].copy()
                e[odd] = 0.0
                res = b[r] - op.apply_Dr(e)
                y = []  # after every step, with the outer step's coefficient
                for _ in range(nu + 1):
                    Ae = op.apply_Dr(e)
                    y.append(e * (np.vdot(Ae, b[r]) / np.vdot(Ae, Ae)))
                    Ar = op.apply_Dr(res)
                    a = np.vdot(Ar, res) / np.vdot(Ar, Ar)
                    e, res = e + a * res, res - a * Ar
                got = op.apply_A(x[r])
                got[odd] = 0.0
                err = [np.linalg.norm(got - v) / np.linalg.norm(v) for v in y]
                print(prec, nu, r, err, flush=True)
                assert err[nu] < tol, (nu, r, err)
                assert all(v > 100 * tol for v in err[:nu]), (nu, r, err)

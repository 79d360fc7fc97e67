"""The paired steps of fixed-length GCR over long bases: three to nine groups of
eight vectors, up to the longest basis, odd lengths, lengths far beyond
the point where the residual has come down to rounding, and the other user of
the pairs, an unpreconditioned coarse solve of fixed length.

Result: the vector of smallest residual over the Krylov space, from an
orthonormal basis and a least-squares solve in FP64.

Tolerances.  A vector of smallest residual is compared up to FP64 rounding
times the growth over the basis, 1e-9, and in FP32 up to 30 stored vectors of
6e-8 each times the condition of the operator (about 10), 2e-5.  Where the
residual is at rounding it stays there: some units of the storage's rounding
times the square root of the 64 vectors, 1e-6 in FP32 and 1e-13 in FP64; the
direction updates of a residual taken to be orthogonal to the basis had
brought it back to 1e-5 and 1e-9.
"""
import numpy as np
import pytest
import torch

import inputs
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS = (6, 4, 4, 6)


def minimum(apply, v, m):
    """argmin ||v - A x|| over span{v, A v, .., A^(m-1) v}."""
    Z = [v / np.linalg.norm(v)]
    for _ in range(m - 1):
        z = apply(Z[-1])
        for _ in range(2):
            for u in Z:
                z = z - np.vdot(u, z) * u
        Z.append(z / np.linalg.norm(z))
    AZ = np.stack([apply(z) for z in Z], axis=1)
    return np.stack(Z, axis=1) @ np.linalg.lstsq(AZ, v, rcond=None)[0]


def setup_vector(ctx, prec, m):
    ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[1], seed=17, setup_relax=m, setup_max_steps=1,
                                       setup_prec=getattr(w, prec)))
    ctx.build_null_vectors()
    return ctx.get_null_vectors().cpu().numpy().ravel()


def operator(ctx, shape, op):
    def apply(z):
        return ctx.apply_D(torch.from_numpy(z.reshape(shape)).cuda(), op, w.F64).cpu().numpy().ravel()
    return apply


@pytest.mark.parametrize("prec,tol,lengths", [("F64", 1e-9, (16, 17, 24, 25, 30, 64)), ("F32", 2e-5, (17, 24, 30))])
def test_long_setup_vector_is_the_minimum(prec, tol, lengths):
    with w.Context(DIMS) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.4, 61)).cuda())
        ctx.set_clover(0.05, 1.0)
        v = ctx.setup_start_vectors(17, 1)
        apply = operator(ctx, v.shape, w.OP_DP)
        v0 = v.cpu().numpy().ravel()
        for m in lengths:
            got = setup_vector(ctx, prec, m)
            x = minimum(apply, v0, m)
            x /= np.linalg.norm(x)
            err = np.linalg.norm(got - x)
            print(prec, m, err, flush=True)
            assert err < tol, (m, err)


@pytest.mark.parametrize("prec,tol", [("F64", 1e-13), ("F32", 1e-6)])
@pytest.mark.parametrize("m0", [4.0, 9.0])
def test_residual_stays_at_rounding(m0, prec, tol):
    with w.Context(DIMS) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.4, 61)).cuda())
        ctx.set_clover(m0, 1.0)
        v = ctx.setup_start_vectors(17, 1)
        apply = operator(ctx, v.shape, w.OP_DP)
        v0 = v.cpu().numpy().ravel()
        for m in (40, 52, 63, 64):
            y = apply(setup_vector(ctx, prec, m))
            res = np.linalg.norm(v0 - y * (np.vdot(y, v0) / np.vdot(y, y))) / np.linalg.norm(v0)
            print(m0, prec, m, res, flush=True)
            assert res < tol, (m, res)


@pytest.mark.parametrize("m", [7, 24, 33])
def test_fixed_coarse_solve(m):
    """One outer step with the coarse correction alone: the solution is that of the coarse solve, prolonged."""
    dims, block, nvec, m0 = (12, 4, 4, 4), (4, 2, 2, 2), 4, 0.3
    links = inputs.gauge_field(dims, 0.3, 62)
    op = WilsonClover(dims, links, m0, 1.0)
    rng = np.random.default_rng(8)
    shape = tuple(reversed(dims)) + (4, 3)
    b = (rng.standard_normal(op.shape) + 1j * rng.standard_normal(op.shape))
    b[op.lat.odd] = 0.0
    with w.Context(dims) as ctx:
        ctx.set_gauge(torch.from_numpy(links).cuda())
        ctx.set_clover(m0, 1.0)
        ctx.set_mg_params(w.default_params(block=[block], nvec=[nvec], nu_post=0, smoother_prec=w.F64, cycle_mode=1,
                                           restart=[m], max_iter=[m], outer_max_iter=1))
        vecs = rng.standard_normal((nvec,) + shape) + 1j * rng.standard_normal((nvec,) + shape)
        ctx.set_null_vectors(torch.from_numpy(vecs).cuda())
        ctx.build_coarse()
        bt = torch.from_numpy(b.reshape((1,) + shape)).cuda()
        x = ctx.solve(bt, w.MG_GCR, 1e-10, raise_on_error=False)[0].cpu().numpy().reshape(op.shape)
        rhs = ctx.restrict(bt)
        cshape = rhs.shape

        def coarse(z):
            return ctx.apply_coarse(torch.from_numpy(z.reshape(cshape)).cuda(), 1, w.OP_FULL, w.F64).cpu().numpy().ravel()

        c = minimum(coarse, rhs.cpu().numpy().ravel(), m)
        z = ctx.prolong(torch.from_numpy(c.reshape(cshape)).cuda()).cpu().numpy().reshape(op.shape)
    z[op.lat.odd] = 0.0
    Az = op.apply_Dr(z)
    y = z * (np.vdot(Az, b) / np.vdot(Az, Az))
    err = np.linalg.norm((op.apply_A(x) - y)[op.lat.even]) / np.linalg.norm(y)
    print(m, err, flush=True)
    assert err < 1e-9

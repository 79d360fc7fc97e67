"""The several-vector kernels of the GCR solvers (multi-dot, step, solution
update) at the basis sizes where their grouping changes: one slot, the edges
of a group of eight vectors, more than sixteen, and the largest basis.

The library's plain FP64 GCR on D_r is the oracle's GCR in another order of
rounding, so both take the same number of steps (one more or less where the
last residual lands on the tolerance) and the solution's true residual, by
the oracle's D, meets the tolerance.  The null-vector setup runs the FP32
kernels with 1, 9 and 30 slots: its vectors come out orthonormal to FP32
rounding (24 vectors orthogonalised twice: 1e-5) and a batch of two solves
over it converges."""
import numpy as np
import pytest
import torch

import inputs
from oracle.dirac import WilsonClover
from oracle.krylov import SolveInfo, gcr

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS = (4, 4, 4, 6)


@pytest.fixture(scope="module")
def small():
    U = inputs.gauge_field(DIMS, 0.3, 1601)
    ctx = w.Context(DIMS)
    ctx.set_gauge(torch.from_numpy(U).cuda())
    ctx.set_clover(-0.1, 1.0)
    yield ctx, WilsonClover(DIMS, U, -0.1, 1.0)
    ctx.close()


def canon(v):
    return torch.from_numpy(np.ascontiguousarray(v).reshape((-1,) + tuple(reversed(DIMS)) + (4, 3))).cuda()


@pytest.mark.parametrize("restart", [1, 7, 8, 9, 17, 64])
def test_gcr_steps_match_oracle(small, restart):
    ctx, op = small
    print("restart", restart, flush=True)
    ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[4], outer_restart=restart))
    b = inputs.z2_source(DIMS, 2601).reshape(op.shape)
    tol = 1e-9
    x, st = ctx.solve(canon(b), w.GCR, tol)
    br = op.reduced_source(b)
    info = SolveInfo()
    gcr(op.apply_Dr, br, tol=tol, restart=restart, maxiter=1000, target_norm=np.linalg.norm(b), info=info)
    xr = x.cpu().numpy().reshape(op.shape)
    assert np.linalg.norm(b - op.apply_D(xr)) <= tol * 1.0000001 * np.linalg.norm(b)
    assert abs(st[0]["iters"] - info.iters) <= 1, (st[0]["iters"], info.iters)


@pytest.mark.parametrize("relax", [1, 9, 30])
def test_setup_vectors_orthonormal(small, relax):
    ctx, op = small
    print("relax", relax, flush=True)
    ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[24], setup_relax=relax, setup_max_steps=2,
                                       tol=[0.2], restart=[20], max_iter=[60], outer_max_iter=400))
    ctx.build_null_vectors()
    v = ctx.get_null_vectors().cpu().numpy().reshape(24, -1)
    assert np.abs(v.conj() @ v.T - np.eye(24)).max() < 1e-5
    ctx.build_coarse()
    b = np.stack([inputs.z2_source(DIMS, 2610 + r) for r in range(2)])
    x, _ = ctx.solve(canon(b), w.MG_GCR, 1e-10)
    for r in range(2):
        bb = b[r].reshape(op.shape)
        res = np.linalg.norm(bb - op.apply_D(x[r].cpu().numpy().reshape(op.shape))) / np.linalg.norm(bb)
        assert res <= 1.0000001e-10, (r, res)

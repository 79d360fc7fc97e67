"""The smoother's last step hands its result on in FP64 by itself: with one
step and several, FP32 and FP64 smoothers, one right-hand side and
batches, on a lattice whose half volume fills no workgroup, multigrid solves
reach 1e-10 (oracle D), and a batch takes as many outer iterations as its
vectors alone (within 1: the stopping vote of a batch's coarse solves is its
slowest member's).  A wrong or missing last step costs the preconditioner,
not the residual: the iteration counts show it, as more smoothing steps may
not take more iterations than fewer.
"""
import numpy as np
import pytest
import torch

import inputs
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS = (6, 4, 4, 10)


@pytest.mark.parametrize("prec", ["F64", "F32"])
def test_last_smoother_step(prec):
    U = inputs.gauge_field(DIMS, 0.3, 44)
    op = WilsonClover(DIMS, U, -0.1, 1.0)
    b = torch.from_numpy(np.stack([inputs.z2_source(DIMS, 900 + r) for r in range(3)]).reshape(
        (3,) + tuple(reversed(DIMS)) + (4, 3))).cuda()
    iters = {}
    for nu in (1, 2, 4):
        with w.Context(DIMS) as ctx:
            ctx.set_gauge(torch.from_numpy(U).cuda())
            ctx.set_clover(-0.1, 1.0)
            ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[8], nu_post=nu, seed=5,
                                               smoother_prec=getattr(w, prec)))
            ctx.build_null_vectors(0)
            ctx.build_coarse(0)
            alone = [ctx.solve(b[r:r + 1], w.MG_GCR, 1e-10) for r in range(3)]
            x, st = ctx.solve(b, w.MG_GCR, 1e-10)
        for r in range(3):
            bv = b[r].cpu().numpy().reshape(op.shape)
            for v in (x[r], alone[r][0][0]):
                res = np.linalg.norm(bv - op.apply_D(v.cpu().numpy().reshape(op.shape))) / np.linalg.norm(bv)
                assert res <= 1.0000001e-10, (nu, r, res)
            assert abs(st[r]["iters"] - alone[r][1][0]["iters"]) <= 1, (nu, r)
        iters[nu] = max(s["iters"] for s in st)
    assert iters[4] <= iters[2] <= iters[1], iters

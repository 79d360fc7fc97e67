"""Operator applies at the sizes where their launches change: a lattice of a few
wavefronts (small workgroups), a ragged last wavefront, batches of one and of
many right-hand sides per thread (two per thread and lattice tiles from 12
workgroups per compute unit on, odd batches, tiles that do not divide 4 x 8).

Every launch shape does the same arithmetic in the same order, so a batch must
equal its right-hand sides applied one at a time bit for bit, in every form,
precision and adjoint; one right-hand side is compared with the oracle (FP64,
1e-13 of the largest entry: sums of a few hundred terms)."""
import numpy as np
import pytest
import torch

import inputs
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

OPS = [w.OP_FULL, w.OP_SCHUR, w.OP_DP, w.OP_SCHUR_X]


@pytest.mark.parametrize("dims,nrhs", [((4, 4, 4, 4), 2), ((2, 6, 4, 10), 5), ((16, 16, 16, 48), 16),
                                       ((30, 18, 6, 10), 97)])
def test_batches_equal_single(dims, nrhs):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    shape = (nrhs,) + tuple(reversed(dims)) + (4, 3)
    v = torch.complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64),
                      torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))
    U = inputs.gauge_field_torch(dims, 0.3, 1801, device="cuda")
    with w.Context(dims) as ctx:
        ctx.set_gauge(U)
        ctx.set_clover(-0.1, 1.0)
        for op in OPS:
            for prec in (w.F64, w.F32, w.F16):
                for apply in (ctx.apply_D, ctx.apply_Ddag):
                    print(dims, nrhs, op, prec, apply.__name__, flush=True)
                    got = apply(v, op, prec)
                    for r in sorted({0, 1, nrhs // 2, nrhs - 1}):
                        assert torch.equal(got[r], apply(v[r:r + 1], op, prec)[0]), (op, prec, r)
        if np.prod(dims) <= 1024:
            o = WilsonClover(dims, U.cpu().numpy(), -0.1, 1.0)
            x = v[0].cpu().numpy().reshape(o.shape)
            for op, want in ((w.OP_FULL, o.apply_D(x)), (w.OP_SCHUR, o.apply_Dr(x)), (w.OP_DP, o.apply_Dp(x))):
                got = ctx.apply_D(v[:1], op, w.F64).cpu().numpy().reshape(o.shape)
                if op == w.OP_SCHUR:
                    assert np.abs(got[o.lat.odd]).max() == 0.0
                    got, want = got[o.lat.even], want[o.lat.even]
                assert np.abs(got - want).max() <= 1e-13 * np.abs(want).max(), op

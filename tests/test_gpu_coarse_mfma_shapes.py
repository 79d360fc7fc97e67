"""Matrix-core coarse stencil against the same stencil on the vector units
(one right-hand side at a time, FP32), for every tile count
of its rows (n = 16, 32, 48, 64), groups of sixteen right-hand sides that are
partly and wholly filled, and as few sites as one workgroup per parity.

Tolerance: entries and inputs are rounded to FP16 (2^-11 each, relative to
the largest of a block column), 8 n products of them: 2 * 2^-11 max-norm
relative to the result, with n-term sums of random signs; 4e-3 bounds it.
"""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 4, 4, 12)])
@pytest.mark.parametrize("nvec", [8, 16, 24, 32])
def test_batches_match_one_at_a_time(dims, nvec):
    rng = np.random.default_rng(12)
    shape = (nvec,) + tuple(reversed(dims)) + (4, 3)
    V = int(np.prod(dims)) // 16
    with w.Context(dims) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(dims, 0.3, 72)).cuda())
        ctx.set_clover(-0.1, 1.0)
        ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[nvec]))
        ctx.set_null_vectors(torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).cuda())
        ctx.build_coarse(0)
        b = rng.standard_normal((33, V, 2 * nvec)) + 1j * rng.standard_normal((33, V, 2 * nvec))
        b[:, : V // 2] *= 1e-3  # columns scaled by themselves
        b = torch.from_numpy(b).cuda()
        want = torch.cat([ctx.apply_coarse(b[r:r + 1], 1, w.OP_SCHUR, w.F32) for r in range(33)])
        for nrhs in (2, 15, 16, 17, 33):
            got = ctx.apply_coarse(b[:nrhs].contiguous(), 1, w.OP_SCHUR, w.F32)
            for r in range(nrhs):
                err = ((got[r] - want[r]).abs().max() / want[r].abs().max()).item()
                assert err < 4e-3, (nrhs, r, err)

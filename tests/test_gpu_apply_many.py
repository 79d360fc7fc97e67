"""An apply of more right-hand sides than the second extent of a grid holds
(65535): every one is done, also those on either side of the places where the
launches are split, and equals its apply alone bit for bit."""
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS, NRHS = (2, 2, 2, 2), 65539


@pytest.mark.parametrize("op", [w.OP_FULL, w.OP_SCHUR, w.OP_DP, w.OP_SCHUR_X])
def test_more_than_a_grid_extent(op):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    shape = (NRHS,) + tuple(reversed(DIMS)) + (4, 3)
    v = torch.complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64),
                      torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))
    with w.Context(DIMS) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.3, 82)).cuda())
        ctx.set_clover(-0.1, 1.0)
        for apply in (ctx.apply_D, ctx.apply_Ddag):
            for prec in (w.F64, w.F16):
                got = apply(v, op, prec)
                for r in (0, 1, 32767, 32768, 65534, 65535, 65536, NRHS - 1):
                    assert torch.equal(got[r], apply(v[r:r + 1], op, prec)[0]), (apply.__name__, prec, r)
                assert got.flatten(1).abs().amax(1).min() > 0.0

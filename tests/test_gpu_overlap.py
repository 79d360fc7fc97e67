"""Applies and transfers whose output shares memory with their input: the
input counts as read before the output is written, so the result is, bit for
bit, that of the same call on buffers apart.  Applies with the output one
spinor or a few components behind or before the input (out == in itself is
refused); transfers also in place.
"""
import ctypes

import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS, BLOCK, NVEC = (8, 8, 8, 8), (4, 2, 4, 4), 9
PRECS = [w.F64, w.F32, w.F16]


@pytest.fixture(scope="module")
def ctx():
    with w.Context(DIMS) as c:
        c.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.4, 81)).cuda())
        c.set_clover(-0.1, 1.0)
        c.set_mg_params(w.default_params(block=[BLOCK], nvec=[NVEC]))
        c.set_null_vectors(gauss(1, (NVEC,) + tuple(reversed(DIMS)) + (4, 3)))
        c.build_coarse()
        yield c


def gauss(seed, shape):
    rng = np.random.default_rng(seed)
    return torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).cuda()


def call(fn, head, n_in, n_out, shift, v, nrhs):
    """fn on one buffer, the output `shift` elements behind the input (before it if negative)"""
    i0 = max(0, -shift)
    buf = torch.zeros(i0 + max(n_in, n_out + shift), dtype=torch.complex128, device="cuda")
    buf[i0:i0 + n_in] = v.reshape(-1)
    o0 = i0 + shift
    assert o0 < i0 + n_in and i0 < o0 + n_out
    w.check(fn(*head, ctypes.c_void_p(buf[o0:].data_ptr()), ctypes.c_void_p(buf[i0:].data_ptr()), nrhs))
    return buf[o0:o0 + n_out]


@pytest.mark.parametrize("dag", [False, True])
@pytest.mark.parametrize("op", [w.OP_FULL, w.OP_SCHUR, w.OP_DP, w.OP_SCHUR_X])
def test_apply(ctx, op, dag):
    one = int(np.prod(DIMS)) * 12
    fn = w._lib.LIB.wcmg_apply_Ddag if dag else w._lib.LIB.wcmg_apply_D
    for prec in PRECS:
        for nrhs, shift in ((1, 5), (1, -12), (3, one), (3, -one), (2, one // 2)):
            v = gauss(7, (nrhs,) + tuple(reversed(DIMS)) + (4, 3))
            want = (ctx.apply_Ddag if dag else ctx.apply_D)(v, op, prec).reshape(-1)
            got = call(fn, (ctx.h, 0, op, prec), nrhs * one, nrhs * one, shift, v, nrhs)
            assert torch.equal(got, want), (prec, nrhs, shift)


@pytest.mark.parametrize("prec", PRECS)
def test_transfers(ctx, prec):
    one = int(np.prod(DIMS)) * 12
    cone = int(np.prod(ctx.coarse_dims())) * 2 * NVEC
    for nrhs in (1, 2, 17):
        f = gauss(8, (nrhs,) + tuple(reversed(DIMS)) + (4, 3))
        c = gauss(9, (nrhs, cone // (2 * NVEC), 2 * NVEC))
        down, up = ctx.restrict(f, prec=prec).reshape(-1), ctx.prolong(c, prec=prec).reshape(-1)
        for shift in (0, 3, nrhs * one - nrhs * cone):
            got = call(w._lib.LIB.wcmg_restrict, (ctx.h, 0, 0, prec), nrhs * one, nrhs * cone, shift, f, nrhs)
            assert torch.equal(got, down), (nrhs, shift)
        for shift in (0, 3, nrhs * cone - nrhs * one):
            got = call(w._lib.LIB.wcmg_prolong, (ctx.h, 0, 0, prec), nrhs * cone, nrhs * one, shift, c, nrhs)
            assert torch.equal(got, up), (nrhs, shift)

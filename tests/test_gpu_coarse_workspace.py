"""Coarse-level calls that share launches and work space.

* the persistent solve keeps one work space per context, cleared by every
  call: solves of different precision, launch form, restart length and
  right-hand side in one context, in turn, equal the same solves each in a
  context of its own, bit for bit (the launch sums in a fixed order);
* a batched stencil application converts all its right-hand sides in one
  launch: the same vectors in another order give the same results in that
  order, bit for bit (each is summed by itself, in the order the number of
  right-hand sides sets).
"""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

DIMS, BLOCK = (8, 8, 8, 8), (2, 2, 2, 4)


def build(nvec):
    ctx = w.Context(DIMS)
    ctx.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.3, 71)).cuda())
    ctx.set_clover(-0.1, 1.0)
    ctx.set_mg_params(w.default_params(block=[BLOCK], nvec=[nvec], coarse_fp16=1))
    rng = np.random.default_rng(4)
    shape = (nvec,) + tuple(reversed(DIMS)) + (4, 3)
    ctx.set_null_vectors(torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).cuda(), level=0)
    ctx.build_coarse(0)
    return ctx


def vectors(nvec, nrhs):
    rng = np.random.default_rng(9)
    shape = (nrhs, 4 * 4 * 4 * 2, 2 * nvec)
    return torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).cuda()


def test_solves_in_turn_equal_solves_alone():
    calls = [(w.F32, 0, 30, 1e-3), (w.F64, 0, 64, 1e-8), (w.F32, 3, 5, 1e-3), (w.F64, 2, 3, 1e-6), (w.F32, 4, 30, 0.2),
             (w.F32, 0, 1, 0.1)]
    b = vectors(6, len(calls))
    with build(6) as ctx:
        for i, (prec, launch, restart, tol) in enumerate(calls):
            print("call", i, prec, launch, restart, tol, flush=True)
            x, st = ctx.coarse_solve(b[i], prec=prec, tol=tol, max_iter=200, restart=restart, launch=launch)
            with build(6) as alone:
                y, sy = alone.coarse_solve(b[i], prec=prec, tol=tol, max_iter=200, restart=restart, launch=launch)
            assert torch.equal(x, y), i
            assert st["iters"] == sy["iters"] and st["true_rel_res"] == sy["true_rel_res"], i


@pytest.mark.parametrize("nvec,nrhs", [(6, 2), (5, 3), (24, 13)])
@pytest.mark.parametrize("prec", ["F64", "F32"])
def test_every_right_hand_side_of_a_batch(nvec, nrhs, prec):
    b = vectors(nvec, nrhs)
    with build(nvec) as ctx:
        perm = torch.from_numpy(np.random.default_rng(2).permutation(nrhs)).cuda()
        for op in (w.OP_FULL, w.OP_SCHUR):
            got = ctx.apply_coarse(b, 1, op, getattr(w, prec))
            assert got.abs().amax(dim=(1, 2)).min() > 0.1
            assert torch.equal(ctx.apply_coarse(b[perm].contiguous(), 1, op, getattr(w, prec)), got[perm])

"""Fixed-length GCR of the setup takes its steps in pairs on one pass over the
basis: its result is the vector of smallest residual over the Krylov space
whatever the pairing.  Against that minimum, from an orthonormal Krylov basis
and a least-squares solve in FP64 (the operator checked against the oracle
elsewhere): lengths of one step, one pair, pairs with a last single step, and
basis sizes around the eight vectors a group loads together.

Tolerances: FP64 rounding times the growth over the basis stays far below
1e-9.  FP32 rounds m stored vectors at 6e-8 each, amplified by the condition
of the pairs (about 10): 2e-5 for m <= 12.
"""
import numpy as np
import pytest
import torch

import inputs

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


@pytest.mark.parametrize("prec,tol", [("F64", 1e-9), ("F32", 2e-5)])
def test_setup_vector_is_the_minimum(prec, tol):
    with w.Context(DIMS) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(DIMS, 0.4, 61)).cuda())
        ctx.set_clover(0.05, 1.0)
        v = ctx.setup_start_vectors(17, 1)
        shape = v.shape

        def apply(z):
            return ctx.apply_D(torch.from_numpy(z.reshape(shape)).cuda(), w.OP_DP, w.F64).cpu().numpy().ravel()

        v0 = v.cpu().numpy().ravel()
        for m in (1, 2, 3, 7, 8, 9, 10, 12):
            ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[1], seed=17, setup_relax=m,
                                               setup_max_steps=1, setup_prec=getattr(w, prec)))
            ctx.build_null_vectors()
            got = ctx.get_null_vectors().cpu().numpy().ravel()
            x = minimum(apply, v0, m)
            x /= np.linalg.norm(x)
            err = np.linalg.norm(got - x)
            print(prec, m, err, flush=True)
            assert err < tol, (m, err)

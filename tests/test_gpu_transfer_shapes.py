"""Restriction and prolongation of the first level over the shapes where their
kernels change: batches of 1 (vector kernel), 2, 8, 9, 16 (one or two tiles of
the matrix instructions) and 17 (two launches); 1 to 64 null vectors (one to
four row tiles, with and without padding); blocks of 16 sites (fewer units
than lanes) to 1024 (the largest, with the largest LDS use), odd numbers of
blocks; FP64, FP32 and half precision.

Reference: NumPy QR of each block and chirality with a positive diagonal, and
its products.  Bounds, relative to the largest entry: FP64 1e-12 (sums of at
most 6144 terms); FP32 1e-5 (64 terms at 2^-24 each, or FP32-rounded inputs
under an FP64 sum); F16 5e-3 (components rounded to 2^-11 of their site's
largest, errors of independent terms)."""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")

TOL = {"F64": 1e-12, "F32": 1e-5, "F16": 5e-3}
SHAPES = [
    ((4, 4, 4, 4), (2, 2, 2, 2), 5),
    ((4, 4, 6, 4), (2, 2, 2, 2), 16),
    ((4, 8, 4, 8), (2, 4, 2, 4), 17),
    ((8, 4, 4, 12), (4, 4, 4, 4), 24),
    ((8, 4, 4, 8), (4, 4, 4, 4), 33),
    ((6, 8, 4, 4), (6, 4, 2, 4), 1),
    ((16, 8, 4, 4), (8, 8, 4, 4), 64),
]


def split(v, dims, block):
    """[n][Lt][Lz][Ly][Lx][4][3] -> [n][blocks][2][sites x 6]"""
    nb = [d // b for d, b in zip(dims, block)]
    n = v.shape[0]
    v = v.reshape(n, nb[3], block[3], nb[2], block[2], nb[1], block[1], nb[0], block[0], 2, 6)
    v = v.transpose(0, 1, 3, 5, 7, 9, 2, 4, 6, 8, 10)
    return v.reshape(n, int(np.prod(nb)), 2, -1)


def join(v, dims, block):
    nb = [d // b for d, b in zip(dims, block)]
    n = v.shape[0]
    v = v.reshape(n, nb[3], nb[2], nb[1], nb[0], 2, block[3], block[2], block[1], block[0], 6)
    v = v.transpose(0, 1, 6, 2, 7, 3, 8, 4, 9, 5, 10)
    return v.reshape((n,) + tuple(reversed(dims)) + (4, 3))


@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_transfer_shapes(shape):
    dims, block, nvec = SHAPES[shape]
    rng = np.random.default_rng(17 + shape)
    cplx = lambda s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    fine_shape = tuple(reversed(dims)) + (4, 3)
    with w.Context(dims) as ctx:
        ctx.set_gauge(torch.from_numpy(inputs.gauge_field(dims, 0.3, 1701)).cuda())
        ctx.set_clover(0.1, 1.0)
        ctx.set_mg_params(w.default_params(block=[block], nvec=[nvec]))
        v = cplx((nvec,) + fine_shape)
        ctx.set_null_vectors(torch.from_numpy(v).cuda())
        ctx.build_coarse()
        vb = split(v, dims, block).transpose(1, 2, 3, 0)  # [block][chi][K][k]
        q, r = np.linalg.qr(vb)
        d = np.einsum("bsii->bsi", r)
        q = q * (d / np.abs(d))[:, :, None, :]
        nc = q.shape[0]
        for nrhs in (1, 2, 8, 9, 16, 17):
            f, c = cplx((nrhs,) + fine_shape), cplx((nrhs, nc, 2 * nvec))
            down = np.einsum("bsik,nbsi->nbsk", q.conj(), split(f, dims, block))
            down[:, :, 1] *= -1
            down = down.reshape(nrhs, nc, 2 * nvec)
            up = join(np.einsum("bsik,nbsk->nbsi", q, c.reshape(nrhs, nc, 2, nvec)), dims, block)
            for prec, tol in TOL.items():
                print(dims, block, nvec, nrhs, prec, flush=True)
                got = ctx.restrict(torch.from_numpy(f).cuda(), prec=getattr(w, prec)).cpu().numpy()
                assert np.abs(got - down).max() <= tol * np.abs(down).max(), ("restrict", nrhs, prec)
                got = ctx.prolong(torch.from_numpy(c).cuda(), prec=getattr(w, prec)).cpu().numpy()
                assert np.abs(got - up).max() <= tol * np.abs(up).max(), ("prolong", nrhs, prec)

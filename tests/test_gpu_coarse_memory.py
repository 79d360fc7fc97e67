"""A context keeps no more than 32 MiB of work space for coarse solves: a solve
that needs more (here 130 MiB) gives it back, and solves of either size afterwards
repeat their results bit for bit."""
import numpy as np
import pytest
import torch

import inputs

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")


def test_large_work_space_is_given_back():
    dims, nvec = (16, 16, 16, 16), 8
    with w.Context(dims) as ctx:
        ctx.set_gauge(inputs.gauge_field_torch(dims, 0.3, 86, device="cuda"))
        ctx.set_clover(0.1, 1.0)
        ctx.set_mg_params(w.default_params(block=[(2, 2, 2, 2)], nvec=[nvec]))
        gen = torch.Generator(device="cuda")
        gen.manual_seed(3)

        def gauss(*shape):
            return torch.complex(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64),
                                 torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64))

        ctx.set_null_vectors(gauss(nvec, *reversed(dims), 4, 3))
        ctx.build_coarse()
        b = gauss(int(np.prod(ctx.coarse_dims())), 2 * nvec)

        def solve(restart):
            x, st = ctx.coarse_solve(b, prec=w.F64, tol=1e-6, max_iter=64, restart=restart)
            torch.cuda.synchronize()
            return x, st["iters"]

        small, n_small = solve(1)  # what every solve needs once is allocated here
        free = torch.cuda.mem_get_info()[0]
        large, n_large = solve(64)
        kept = free - torch.cuda.mem_get_info()[0]
        print("kept", kept >> 20, "MiB", flush=True)
        assert kept <= 40 << 20
        for restart, x, n in ((1, small, n_small), (64, large, n_large)):
            y, k = solve(restart)
            assert torch.equal(x, y) and n == k

"""Link force at the edges of its launch: one pair of spinors (its spinors are
read once for all planes) and several, lattices whose sites do not fill the
last wavefront or workgroup group, and extents of two, against the oracle.

Tolerance: FP64 sums of at most a few hundred terms per entry, far below the
1e-12 (max-norm relative) the other force tests use.
"""
import numpy as np
import pytest
import torch

import inputs
from oracle import force as F
from oracle.dirac import WilsonClover

pytestmark = pytest.mark.gpu

w = pytest.importorskip("paper_1011_2775_amd")


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((4, 4, 4, 4), 1), ((6, 2, 4, 6), 1), ((6, 2, 4, 6), 3),
                                       ((4, 6, 10, 2), 2)])
def test_force_launch_edges(dims, nrhs):
    V = int(np.prod(dims))
    U = inputs.gauge_field(dims, 0.4, 31)
    op = WilsonClover(dims, U, -0.1, 1.2, -1)
    rng = np.random.default_rng(5)
    x, lam = (rng.standard_normal((nrhs, V, 4, 3)) + 1j * rng.standard_normal((nrhs, V, 4, 3)) for _ in range(2))
    with w.Context([(dims, -1)]) as ctx:
        ctx.set_gauge(torch.from_numpy(U).cuda())
        ctx.set_clover(-0.1, 1.2)
        shape = (nrhs,) + tuple(reversed(dims)) + (4, 3)
        for include_clover in (True, False):
            got = ctx.force(torch.from_numpy(x.reshape(shape)).cuda(), torch.from_numpy(lam.reshape(shape)).cuda(),
                            include_clover).cpu().numpy().reshape(V, 4, 3, 3)
            want = sum(F.force(op, x[r], lam[r], include_clover) for r in range(nrhs))
            err = np.abs(got - want).max() / np.abs(want).max()
            assert err < 1e-12, (include_clover, err)

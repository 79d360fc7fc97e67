"""Link force without its clover part on either side of the lattice size at
which it changes from a wavefront per direction to a thread per site (16384
sites), with a ragged last workgroup, periodic and antiperiodic time and an
anisotropic hop, against the oracle.

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


@pytest.mark.parametrize("dims,nrhs,t_bc,hop_s", [((16, 16, 8, 6), 2, -1, 1.0), ((16, 16, 8, 8), 1, -1, 1.0),
                                                  ((12, 10, 14, 10), 3, 1, 0.35)])
def test_hop_force(dims, nrhs, t_bc, hop_s):
    V = int(np.prod(dims))
    U = inputs.gauge_field(dims, 0.4, 83)
    op = WilsonClover(dims, U, -0.1, 1.0, t_bc, hop_s=hop_s)
    rng = np.random.default_rng(6)
    x, lam = (rng.standard_normal((nrhs, V, 4, 3)) + 1j * rng.standard_normal((nrhs, V, 4, 3)) for _ in range(2))
    with w.Context([(dims, t_bc)]) as ctx:
        ctx.set_gauge(torch.from_numpy(U).cuda())
        ctx.set_clover_aniso(-0.1, hop_s, 1.0, 1.0)
        shape = (nrhs,) + tuple(reversed(dims)) + (4, 3)
        got = ctx.force(torch.from_numpy(x.reshape(shape)).cuda(), torch.from_numpy(lam.reshape(shape)).cuda(),
                        False).cpu().numpy().reshape(V, 4, 3, 3)
    want = sum(F.force(op, x[r], lam[r], False) for r in range(nrhs))
    err = np.abs(got - want).max() / np.abs(want).max()
    print(dims, err, flush=True)
    assert err < 1e-12

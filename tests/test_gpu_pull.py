"""The pull of the Schwarz apply: block outputs found from lattice indices
against the node-to-block map, bit for bit."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

# (shape, cells, degree): one cell, a single round's 512 unknowns not reached
# and passed, ragged remainders, scalar and vector problems
CASES = [("disk", 1, 1), ("disk", 2, 4), ("disk", 11, 2), ("disk", 37, 3), ("porous", 1, 3),
         ("porous", 5, 1), ("porous", 7, 2), ("porous", 4, 4), ("elastic", 1, 2),
         ("elastic", 6, 1), ("elastic", 5, 2), ("elastic", 3, 3)]


def _desc(shape, n, p):
    if shape == "disk":
        return fcgen.disk_poisson_2d(3, n=n, p=p)
    make = fcgen.porous_poisson_3d if shape == "porous" else fcgen.porous_elasticity_3d
    return make(3, n=n, p=p, n_voids=3, rmin=0.08, rmax=0.16)


@pytest.mark.parametrize("shape,n,p", CASES)
def test_lattice_pull_is_the_mapped_pull(monkeypatch, shape, n, p):
    """z = S r and 8 steps of CG with the lattice pull and with the map
    (FC_PULL_LATTICE=0 at the build): the same block outputs summed in the same
    order, so every bit is the same.  (Timing mode keeps tiny problems in separate
    launches.)"""
    torch = require_gpu()
    pb = fc.Problem.setup(_desc(shape, n, p))
    out = []
    for lattice in ("0", "1"):
        monkeypatch.setenv("FC_PULL_LATTICE", lattice)
        pc = fc.Precond(pb)
        r = torch.as_tensor(np.random.default_rng(4).standard_normal(pb.n), device="cuda")
        z, b, x = (torch.empty_like(r) for _ in range(3))
        pc.apply_M(r, z)
        pb.rhs(b)
        b += 1e-3 * b.abs().max() * r
        fc.pcg_solve(pb, pc, b, x, tol=0.0, maxit=8, stop="residual", timing=1)
        out.append((z.cpu().numpy(), x.cpu().numpy()))
    assert np.all(np.isfinite(out[0][0]))
    for a, c in zip(*out):
        assert a.tobytes() == c.tobytes()

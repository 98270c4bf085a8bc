"""Sizes and forms of problems that take a kernel of their own and that the other
tests of these kernels leave out (test_routes.py holds that the sizes here take
them)."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
import tests.test_gpu_sliced as sliced
import tests.test_gpu_tiny as tiny
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


# several cells at p = 2 in 3-D, and the largest size of every degree
@pytest.mark.parametrize("dim,n,p", [(3, 2, 2), (3, 3, 2), (3, 4, 2), (2, 47, 1), (2, 26, 2),
                                     (2, 16, 3), (2, 10, 4), (3, 11, 1)])
def test_tiny_steps(dim, n, p):
    tiny.test_tiny_steps_match_separate_launches(dim, n, p)


# enough long rows for the sliced product
@pytest.mark.parametrize("dim,n,p", [(3, 14, 3), (3, 13, 4), (2, 21, 3)])
def test_sliced_product(dim, n, p):
    sliced.test_sliced_product(dim, n, p)


def _plane(pde, n, p):
    """A disk in the plane; vector problems with two components per node, and
    degrees above those of the sliced copy."""
    return fcgen.custom(2, n, p, pde, 1e-3, shapes=[{"centre": [0.48, 0.53], "semi": [0.37, 0.3]}],
                        domain="inclusions", clamp_zmin=pde == "elasticity", seed=p)


PLANE = [("elasticity", 1, 1), ("elasticity", 9, 1), ("elasticity", 8, 2), ("elasticity", 5, 3),
         ("elasticity", 6, 4), ("elasticity", 4, 5), ("elasticity", 3, 8), ("poisson", 5, 5),
         ("poisson", 4, 6), ("poisson", 3, 7), ("poisson", 3, 8)]


@pytest.mark.parametrize("pde,n,p", PLANE)
def test_plane_lattice_forms_are_the_general_ones(monkeypatch, pde, n, p):
    """The pull from lattice indices and from the node-to-block map, and blocks
    read from the lattice and found in the matrix: the same bits."""
    torch = require_gpu()
    hs = fc.HostSystem(_plane(pde, n, p))
    pb = hs.upload()
    r = torch.as_tensor(np.random.default_rng(4).standard_normal(pb.n), device="cuda")
    out = []
    for lattice in ("0", "1"):
        monkeypatch.setenv("FC_PULL_LATTICE", lattice)
        pc = fc.Precond(pb)
        z, x = torch.empty_like(r), torch.empty_like(r)
        pc.apply_M(r, z)
        fc.pcg_solve(pb, pc, r, x, tol=0.0, maxit=8, stop="residual", timing=1)
        out.append((z, x))
    assert torch.isfinite(out[0][0]).all()
    for a, c in zip(*out):
        assert torch.equal(a, c)
    e = hs.export()
    pm = fc.Precond(fc.Problem.from_matrix(e["n_dofs"], e["bsr_dim"], e["rowptr"], e["col"],
                                           e["val"], e["rhs"], e["elem_dofs"], e["eta"]))
    assert pc.info() == pm.info()
    for k in range(pc.info()["n_blocks"]):
        assert pc.block_inverse(k).tobytes() == pm.block_inverse(k).tobytes(), k


def test_plane_members_of_a_batch():
    """A batch of these forms against their single solves: 6 steps, equal up to
    rounding (1e-10 of x, as in test_gpu_cg_paths)."""
    torch = require_gpu()
    pbs = [fc.Problem.setup(_plane(*c)) for c in PLANE]
    pcs = [fc.Precond(p) for p in pbs]
    bs = [torch.as_tensor(np.random.default_rng(k).standard_normal(p.n), device="cuda")
          for k, p in enumerate(pbs)]
    xs, ys = [torch.empty_like(b) for b in bs], [torch.empty_like(b) for b in bs]
    kw = dict(tol=0.0, maxit=6, stop="residual")
    fc.Batch(pbs, pcs).solve(bs, xs, **kw)
    for p, c, b, x, y in zip(pbs, pcs, bs, xs, ys):
        fc.pcg_solve(p, c, b, y, **kw)
        assert float((x - y).norm()) <= 1e-10 * float(y.norm())

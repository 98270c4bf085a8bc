"""CG steps in one workgroup: every degree and dimension it takes, problems of one
cell, of a wave's and a workgroup's edge and of its largest size, against the same
solve in timing mode, which takes the separate launches."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

CASES = [(2, 1, 1), (2, 7, 1), (2, 31, 1), (2, 44, 1), (2, 1, 2), (2, 16, 2), (2, 25, 2), (2, 5, 3),
         (2, 13, 3), (2, 1, 4), (2, 9, 4), (3, 1, 1), (3, 9, 1), (3, 1, 2), (3, 5, 2)]


@pytest.mark.parametrize("dim,n,p", CASES)
def test_tiny_steps_match_separate_launches(dim, n, p):
    torch = require_gpu()
    shapes = [{"centre": [0.45] * dim, "semi": [0.3] * dim}]
    pb = fc.Problem.setup(fcgen.custom(dim, n, p, "poisson", 1e-3, shapes=shapes,
                                       domain="inclusions", seed=n + p))
    pc = fc.Precond(pb)
    b = torch.as_tensor(np.random.default_rng(n).standard_normal(pb.n), device="cuda")
    for kw in (dict(tol=1e-11), dict(tol=0.0, maxit=5, check_every=2),
               dict(tol=1e-9, stop="residual", check_every=1)):
        x, y, z = (torch.full_like(b, float("nan")) for _ in range(3))
        one = fc.pcg_solve(pb, pc, b, x, **kw)
        ref = fc.pcg_solve(pb, pc, b, y, timing=1, **kw)
        fc.pcg_solve_noalloc(pb, pc, b, z, **kw)
        assert one["status"] == ref["status"]
        assert abs(one["iters"] - ref["iters"]) <= (0 if "maxit" in kw else 1)
        assert torch.equal(x, z)
        # equal steps up to rounding: a few hundred units in the last place times
        # the condition number of S A (below 1e3 at alpha = 1e-3); a step more or
        # less changes x by the tolerance
        bound = 1e-10 if one["iters"] == ref["iters"] else 1e-7
        assert float((x - y).norm()) <= bound * float(y.norm())

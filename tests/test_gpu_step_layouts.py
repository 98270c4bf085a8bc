"""CG steps of 3-D scalar problems on either side of the rules that pick their
product's layout (test_routes.py checks on which side each size lies), against the
recurrences written with the public products."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu
from tests.test_gpu_cg_paths import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(5, 2), (8, 2), (9, 2),    # sliced, the p update joined
                                 (10, 2), (12, 2),          # rows
                                 (16, 2)])                  # sliced, joined
def test_steps_match_the_recurrences(n, p):
    """Bounds as in test_gpu_cg_paths: rounding only, at alpha = 1e-2."""
    torch = require_gpu()
    pb = fc.Problem.setup(fcgen.porous_poisson_3d(1, n=n, p=p, n_voids=3, rmin=0.08, rmax=0.16,
                                                  alpha=1e-2))
    pc = fc.Precond(pb)
    b = torch.as_tensor(np.random.default_rng(9).standard_normal(pb.n), device="cuda")
    its = 8
    ref, href = _reference(torch, pb, pc, b, its)
    xs = []
    for solve, kw in ((fc.pcg_solve, {}), (fc.pcg_solve_noalloc, {}),
                      (fc.pcg_solve, {"check_every": 3}), (fc.pcg_solve, {"timing": 1})):
        x = torch.full_like(b, 7.0)
        h = torch.zeros(its + 1, dtype=torch.float64, device="cuda")
        solve(pb, pc, b, x, tol=0.0, maxit=its, stop="residual", history=h, **kw)
        assert float((x - ref).norm() / ref.norm()) < 1e-10
        assert np.abs(h.cpu().numpy() - href).max() < 1e-10 * max(1.0, href.max())
        xs.append(x)
    # the same product in every step, however the steps are launched
    for x in xs[1:]:
        assert torch.equal(x, xs[0])

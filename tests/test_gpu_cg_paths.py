"""Every way a CG step can take (where the dots of a step are summed depends on
the problem's size and blocks) against the same recurrences written with the
public products y = A x and z = S r."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

# (name, description, eta_bar).  alpha = 1e-2 keeps every block's condition
# number below 1e4, so the two differ by rounding only: 8 steps of sums over up
# to 6e5 terms, each within 1e-16 * sqrt(6e5) of its size, through blocks of
# condition 1e4: below 1e-8 of x at the very worst, and 1e-10 is asked.
CASES = {
    # one workgroup; (p, q) from the product's workgroups, beta with p
    "smallest": (lambda: fcgen.disk_poisson_2d(1, n=2, p=1, alpha=1e-2), 1.0),
    # slices and boundary rows in one launch, a few hundred workgroups
    "sliced": (lambda: fcgen.disk_poisson_2d(1, n=60, p=3, alpha=1e-2), 1.0),
    # above 1,024 product workgroups: a pass over p and q
    "pass": (lambda: fcgen.porous_elasticity_3d(1, n=10, p=2, alpha=1e-2), 1.0),
    # no block: the step length in a launch of its own
    "no_block": (lambda: fcgen.porous_poisson_3d(1, n=6, p=2, alpha=1e-2), -1.0),
    # blocks on cut cells only: the node-to-block map, with diagonal scaling
    "some_blocks": (lambda: fcgen.porous_elasticity_3d(1, n=5, p=2, alpha=1e-2), 0.8),
    # above 1,024 partial sets of the pull: beta in a launch of its own
    "large": (lambda: fcgen.porous_poisson_3d(1, n=81, p=1, alpha=1e-2), 1.0),
}


def _reference(torch, pb, pc, b, its):
    x, q, z = torch.zeros_like(b), torch.empty_like(b), torch.empty_like(b)
    r = b.clone()
    pc.apply_M(r, z)
    p, rz, hist = z.clone(), torch.dot(r, z), [1.0]
    for _ in range(its):
        pb.apply_A(p, q)
        a = rz / torch.dot(p, q)
        x += a * p
        r -= a * q
        pc.apply_M(r, z)
        rz, old = torch.dot(r, z), rz
        p = z + (rz / old) * p
        hist.append(float(r.norm() / b.norm()))
    return x, np.array(hist)


@pytest.mark.parametrize("name", CASES)
def test_steps_match_the_recurrences(name):
    torch = require_gpu()
    make, eta_bar = CASES[name]
    pb = fc.Problem.setup(make())
    pc = fc.Precond(pb, eta_bar=eta_bar)
    rng = np.random.default_rng(9)
    b = torch.as_tensor(rng.standard_normal(pb.n), device="cuda")
    its = 8 if pb.n > 30 else 2
    ref, href = _reference(torch, pb, pc, b, its)
    for solve in (fc.pcg_solve, fc.pcg_solve_noalloc):
        if solve is fc.pcg_solve_noalloc and pb.n > 2 ** 19:
            continue
        x = torch.full_like(b, 7.0)
        h = torch.zeros(its + 1, dtype=torch.float64, device="cuda")
        info = solve(pb, pc, b, x, tol=0.0, maxit=its, stop="residual", history=h, check_every=3)
        assert info["iters"] == its and info["status"] == "E_NOTCONV"
        assert float((x - ref).norm() / ref.norm()) < 1e-10
        assert np.abs(h.cpu().numpy() - href).max() < 1e-10 * max(1.0, href.max())
        t = torch.empty_like(b)
        pb.apply_A(x, t)
        assert abs(info["rel_res_true"] - float((b - t).norm() / b.norm())) < 1e-12 * href.max()

"""Where a run stops: the iterate, the count and the status do not depend on how many
steps are launched at a time, on every way a step can be launched, whether the
stop comes from the criterion (beta) or from a breakdown (alpha)."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

# (description, eta_bar, mode)
CASES = {
    "tiny": (lambda: fcgen.disk_poisson_2d(1, n=16, p=2, alpha=1e-3), 1.0, "f64"),
    "joined": (lambda: fcgen.disk_poisson_2d(1, n=60, p=3, alpha=1e-3), 1.0, "f64"),
    "rows": (lambda: fcgen.porous_poisson_3d(1, n=12, p=2, alpha=1e-3), 1.0, "f64"),
    "no_block": (lambda: fcgen.porous_poisson_3d(1, n=6, p=2, alpha=1e-1), -1.0, "f64"),
    "staged": (lambda: fcgen.porous_elasticity_3d(1, n=6, p=2, alpha=1e-3), 1.0, "f64"),
    "single_precision": (lambda: fcgen.porous_elasticity_3d(1, n=6, p=2, alpha=1e-3), 1.0, "s_f32"),
    "bf16": (lambda: fcgen.porous_elasticity_3d(1, n=6, p=2, alpha=1e-3), 1.0, "s_bf16"),
    "large": (lambda: fcgen.porous_poisson_3d(1, n=81, p=1, alpha=1e-2), 1.0, "f64"),
}


def _bits(solve, b, **kw):
    torch = require_gpu()
    x = torch.full_like(b, float("nan"))
    info = solve(b, x, **kw)
    torch.cuda.synchronize()
    return x.cpu().numpy().tobytes(), info["iters"], info["status"]


@pytest.mark.parametrize("name", CASES)
def test_stop_does_not_depend_on_the_launches(name):
    torch = require_gpu()
    make, eta_bar, mode = CASES[name]
    pb = fc.Problem.setup(make())
    store = fc.STORE_F64 | {"f64": 0, "s_f32": fc.STORE_F32, "s_bf16": fc.STORE_BF16}[mode]
    pc = fc.Precond(pb, eta_bar=eta_bar, store=store)
    b = torch.as_tensor(np.random.default_rng(3).standard_normal(pb.n), device="cuda")

    def solve(b, x, **kw):
        return fc.pcg_solve(pb, pc, b, x, tol=1e-3, stop="residual", mode=mode, **kw)

    one = _bits(solve, b, check_every=1)
    assert one[2] == "OK" and one[1] > 1
    for k in (2, 7, 64):
        assert _bits(solve, b, check_every=k) == one
    if mode == "f64" and pb.n <= 2 ** 19:
        def noalloc(b, x, **kw):
            return fc.pcg_solve_noalloc(pb, pc, b, x, tol=1e-3, stop="residual", **kw)

        assert _bits(noalloc, b, check_every=7) == one


def _indefinite(n, m):
    """2 n identity blocks of m, blocks 2 k and 2 k + 1 coupled entry by entry by 2: S
    is the identity, and (p, A p) < 0 for b of opposite sign in the two."""
    size = 2 * n * m
    rows = np.arange(size)
    own = (rows // m * m)[:, None] + np.arange(m)
    other = np.where(rows // m % 2 == 0, rows + m, rows - m)
    col = np.concatenate([own, other[:, None]], 1)
    val = np.concatenate([(own == rows[:, None]) * 1.0, np.full((size, 1), 2.0)], 1)
    order = np.argsort(col, 1)
    col, val = np.take_along_axis(col, order, 1), np.take_along_axis(val, order, 1)
    return fc.Problem.from_matrix(size, 1, np.arange(size + 1) * (m + 1), col.ravel(),
                                  val.ravel(), np.zeros(size), rows.reshape(2 * n, m),
                                  np.ones(2 * n))


@pytest.mark.parametrize("m", [9, 100])   # block products of both kinds
def test_breakdown_leaves_the_iterate(m):
    """The step that breaks down is not taken: x stays the iterate before it."""
    torch = require_gpu()
    pbs = [_indefinite(350, m) for _ in range(2)]
    pcs = [fc.Precond(p) for p in pbs]
    bs = []
    for k, p in enumerate(pbs):
        v = np.random.default_rng(k).standard_normal((350, 1, m)) * [[[1.0], [-1.0]]]
        bs.append(torch.as_tensor(v.reshape(p.n), device="cuda"))
    for p, c, b in zip(pbs, pcs, bs):
        for solve in (fc.pcg_solve, fc.pcg_solve_noalloc):
            for k in (1, 16):
                x = torch.full_like(b, 7.0)
                info = solve(p, c, b, x, tol=1e-12, check_every=k)
                assert info["status"] == "E_BREAKDOWN" and info["iters"] == 1
                assert not x.any()
    xs = [torch.full_like(b, 7.0) for b in bs]
    for info, x in zip(fc.Batch(pbs, pcs).solve(bs, xs, tol=1e-12), xs):
        assert info["status"] == "E_BREAKDOWN" and info["iters"] == 1
        assert not x.any()

"""Every class of tiles a batch can hold: sliced and row-layout products, block
sizes with and without a kernel of their own, lattice and listed blocks, members
of one and of many tiles."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def _member(dim, n, p, pde="poisson", alpha=1e-3):
    shapes = [{"centre": [0.45] * dim, "semi": [0.3] * dim}]
    return fcgen.custom(dim, n, p, pde, alpha, shapes=shapes, domain="inclusions", seed=n + p,
                        clamp_zmin=pde == "elasticity")


GROUPS = {
    "degrees_2d": [((2, 20, p), 1.0) for p in (1, 2, 3, 4, 5)],
    "degrees_3d": [((3, 5, p), 1.0) for p in (1, 2, 3, 4)],
    "vector": [((3, 5, 1, "elasticity"), 1.0), ((3, 4, 2, "elasticity"), 1.0),
               ((3, 3, 3, "elasticity"), 1.0), ((2, 12, 3), 1.0)],
    "listed_blocks": [((2, 24, 2), 0.5), ((3, 7, 2), 0.9), ((3, 5, 4), 0.9), ((2, 16, 1), 0.7)],
    "one_and_many_tiles": [((2, 1, 1), 1.0), ((2, 150, 2), 1.0), ((3, 20, 2), 1.0)],
}


@pytest.mark.parametrize("name", list(GROUPS))
def test_batch_classes_match_single_solves(name):
    torch = require_gpu()
    pbs = [fc.Problem.setup(_member(*m)) for m, _ in GROUPS[name]]
    pcs = [fc.Precond(pb, eta_bar=e) for pb, (_, e) in zip(pbs, GROUPS[name])]
    bs, xs = [], []
    for pb in pbs:
        b = torch.as_tensor(np.random.default_rng(pb.n).standard_normal(pb.n), device="cuda")
        bs.append(b)
        xs.append(torch.full_like(b, float("nan")))
    batch = fc.Batch(pbs, pcs, autotune=False)
    for _ in range(2):   # graph replay
        res = batch.solve(bs, xs, tol=1e-10)
        torch.cuda.synchronize()
        for k, (pb, pc) in enumerate(zip(pbs, pcs)):
            x1 = torch.zeros_like(bs[k])
            single = fc.pcg_solve(pb, pc, bs[k], x1, tol=1e-10)
            assert res[k]["status"] == single["status"] == "OK", (k, res[k], single)
            assert abs(res[k]["iters"] - single["iters"]) <= 1, (k, res[k], single)
            d, e1, e2 = x1 - xs[k], torch.empty_like(x1), torch.empty_like(x1)
            pb.apply_A(d, e1)
            pb.apply_A(x1, e2)
            # both stop at 1e-10: the bound of the oracle-checked batch test
            assert float(torch.dot(d, e1)) <= 1e-16 * float(torch.dot(x1, e2)), k

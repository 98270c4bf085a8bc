"""Product with the sliced copy of a scalar lattice matrix: single cells, classes
of rows that end on, just before and just after a slice of 64, every degree."""
import numpy as np
import pytest
import scipy.sparse as sp

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

CASES = ([(2, n, p) for n, p in ((1, 1), (1, 4), (2, 3), (7, 1), (8, 2), (9, 1), (31, 2), (13, 4))] +
         [(3, n, p) for n, p in ((1, 1), (1, 4), (2, 2), (4, 1), (5, 3), (7, 2), (6, 4), (17, 1),
                             (15, 2), (16, 2))])   # either side of the few-long-rows rule


@pytest.mark.parametrize("dim,n,p", CASES)
def test_sliced_product(dim, n, p):
    torch = require_gpu()
    shapes = [{"centre": [0.5] * dim, "semi": [0.3] * dim}]
    desc = fcgen.custom(dim, n, p, "poisson", 1e-3, shapes=shapes, domain="inclusions",
                        seed=n + p)
    pb = fc.Problem.setup(desc)
    assert pb.info()["sliced"]
    S = pb.export()
    A = sp.csr_matrix((S["val"].ravel(), S["col"], S["rowptr"]), shape=(pb.n, pb.n))
    x = np.random.default_rng(p).standard_normal(pb.n)
    xd = torch.as_tensor(x, device="cuda")
    yd = torch.full_like(xd, float("nan"))
    pb.apply_A(xd, yd)
    # two sums of at most (2p + 1)^dim products, each within its length of units
    # in the last place of the sum of moduli
    bound = 2 * (2 * p + 1) ** dim * 2.0 ** -52 * (abs(A) @ abs(x))
    assert np.all(np.abs(yd.cpu().numpy() - A @ x) <= bound)

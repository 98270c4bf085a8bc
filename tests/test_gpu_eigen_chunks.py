"""Eigen-decompositions of more blocks than one launch takes: the inverses on
either side of its end."""
import numpy as np
import pytest
import scipy.sparse as sp

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def test_unstabilised_inverses_across_launches():
    """9,261 blocks of 64 (a launch takes 8,192), the plain inverse.  alpha = 1 makes
    every block the same well-conditioned matrix up to the boundary (below 1e3 in
    the scaling with a unit diagonal), so P A = I to m eps times that."""
    require_gpu()
    d = fcgen.custom(3, 21, 3, "poisson", 1.0, shapes=[{"centre": [0.5] * 3, "semi": [0.2] * 3}])
    hs = fc.HostSystem(d)
    e = hs.export()
    A = sp.csr_matrix((e["val"].ravel(), e["col"], e["rowptr"]), shape=(e["n_dofs"],) * 2)
    pc = fc.Precond(hs.upload(), stabilize=False)
    assert pc.info()["n_blocks"] == pc.info()["n_eig_blocks"] == 9261
    for k in (0, 4630, 8191, 8192, 9260):
        g = e["elem_dofs"][k]
        a = A[g][:, g].toarray()
        s = np.sqrt(np.diag(a))
        r = (pc.block_inverse(k) * s[:, None] * s) @ (a / s[:, None] / s) - np.eye(64)
        assert np.abs(r).max() <= 64 * 2.0 ** -52 * 1e3 * 64

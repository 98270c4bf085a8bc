"""Block products with more than 64 rows in every size of chunk: few blocks and many,
sizes on either side of the limits, in FP64 and FP32, alone and in a batch."""
import numpy as np
import pytest

import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu
from tests.test_gpu_local_inverse import _problem

pytestmark = pytest.mark.gpu

# (m, blocks): 5 and 1,100 lie on either side of every limit
SIZES = [(m, 5) for m in (65, 72, 95, 96, 97, 125, 128, 129, 162, 176, 177, 192)] + \
        [(m, 1100) for m in (72, 96, 97, 128, 162, 192)]


def _blocks(m, nb, rng):
    """nb copies of a few SPD blocks of condition 10, each scaled by its own power of
    two (exact), and their inverses."""
    base = []
    for _ in range(4):
        q = np.linalg.qr(rng.standard_normal((m, m)))[0]
        a = (q * np.geomspace(1.0, 0.1, m)) @ q.T
        base.append(0.5 * (a + a.T))
    base, scale = np.array(base), 2.0 ** rng.integers(-3, 4, nb)
    k = np.arange(nb) % 4
    return base[k] * scale[:, None, None], np.linalg.inv(base)[k] / scale[:, None, None]


@pytest.mark.parametrize("m,nb", SIZES)
def test_block_products(m, nb):
    torch = require_gpu()
    rng = np.random.default_rng(m)
    blocks, inv = _blocks(m, nb, rng)
    pb = _problem(blocks)
    pc = fc.Precond(pb, store=fc.STORE_F64 | fc.STORE_F32)
    assert pc.info()["n_f32_blocks"] == nb
    b = rng.standard_normal((nb, m))
    ref = np.einsum("kij,kj->ki", inv, b).ravel()
    bd = torch.as_tensor(b.ravel(), device="cuda")
    z = torch.full_like(bd, float("nan"))
    pc.apply_M(bd, z)
    # the inverse (condition 10) and a sum of m products, both within m units in the
    # last place of the sum of moduli
    bound = np.einsum("kij,kj->ki", np.abs(inv), np.abs(b)).ravel()
    assert np.all(np.abs(z.cpu().numpy() - ref) <= 2 * 10 * m * 2.0 ** -52 * bound)
    # S is the inverse of A: one step of CG is the solution, in FP32 up to the
    # rounding of the inverses and sums (m units of the condition number)
    for mode, eps in (("f64", 2.0 ** -52), ("s_f32", 2.0 ** -24)):
        x = torch.full_like(bd, float("nan"))
        fc.pcg_solve(pb, pc, bd, x, tol=0.0, maxit=1, stop="residual", mode=mode)
        assert np.linalg.norm(x.cpu().numpy() - ref) <= 10 * m * eps * np.linalg.norm(ref)
    y = torch.full_like(bd, float("nan"))
    fc.Batch([pb], [pc], autotune=False).solve([bd], [y], tol=0.0, maxit=1, stop="residual")
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 10 * m * 2.0 ** -52 * np.linalg.norm(ref)

"""Local inverses at every block size where the kernels change: one, two and
four blocks per wave, exact and padded sizes up to 64, tile edges up to 192;
blocks read from a matrix and from the lattice; a singular block among them."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 7, 8, 9, 10, 15, 16, 17, 24, 25, 26, 27, 28, 31, 32, 33, 48, 63, 64, 65, 80, 81, 95,
         96, 97, 112, 125, 128, 129, 144, 160, 161, 176, 191, 192]


def _block_diagonal(m, nb, rng):
    """nb dense SPD blocks of size m with rows scaled over six decades (1e3 once
    scaled to a unit diagonal; a few scaled ones pass the threshold of the
    pseudo-inverse, which is not what is tested here); the third has an exact
    null vector where m > 1."""
    blocks = []
    for k in range(nb):
        q = np.linalg.qr(rng.standard_normal((m, m)))[0]
        a = (q * np.geomspace(1.0, 1e-3, m)) @ q.T
        if k == 2:
            if m > 1:
                v = np.ones(m) / np.sqrt(m)
                p = np.eye(m) - np.outer(v, v)
                a = p @ a @ p
        else:
            s = 10.0 ** rng.uniform(-3, 3, m)
            a = a * s[:, None] * s[None]
        blocks.append(0.5 * (a + a.T))
    return np.array(blocks)


def _problem(blocks):
    nb, m, _ = blocks.shape
    n = nb * m
    rows = np.arange(n + 1) * m
    col = (np.arange(n) // m * m)[:, None] + np.arange(m)
    dofs = np.arange(n).reshape(nb, m)
    return fc.Problem.from_matrix(n, 1, rows, col.ravel(), blocks.reshape(-1), np.zeros(n), dofs,
                                  np.ones(nb))


@pytest.mark.parametrize("m", SIZES)
def test_inverse_of_given_blocks(m):
    torch = require_gpu()
    blocks = _block_diagonal(m, 5, np.random.default_rng(m))
    pb = _problem(blocks)
    pc = fc.Precond(pb)
    info = pc.info()
    assert info["n_blocks"] == 5
    drop = pc.block_dropped()
    P = np.array([pc.block_inverse(k) for k in range(5)])
    for k, a in enumerate(blocks):
        lam, v = np.linalg.eigh(a)
        keep = lam > 1e-13 * lam.max()
        if k == 2 and m > 1:
            assert drop[k] == m - keep.sum() == 1
            ref = (v[:, keep] / lam[keep]) @ v[:, keep].T
            tol = 1e-15 * m * (lam[keep].max() / lam[keep].min()) + 1e-13
            assert np.linalg.norm(P[k] - ref) <= 10 * tol * np.linalg.norm(ref)
        elif lam.min() > 1e-12 * lam.max():
            # in the scaling with a unit diagonal (elimination does not depend
            # on it): P A = I there to m eps times the scaled condition (1e3,
            # and a factor of the dimension for the scaling not being optimal)
            s = np.sqrt(np.diag(a))
            r = (P[k] * s[:, None] * s[None]) @ (a / s[:, None] / s[None]) - np.eye(m)
            assert drop[k] == 0
            assert np.abs(r).max() <= 1e-15 * m * 1e3 * m + 1e-13
    # z = S r reads the same inverses
    x = torch.as_tensor(np.random.default_rng(1).standard_normal(5 * m), device="cuda")
    z = torch.empty_like(x)
    pc.apply_M(x, z)
    xb = x.cpu().numpy().reshape(5, m)
    ref = np.einsum("kij,kj->ki", P, xb)
    bound = np.einsum("kij,kj->ki", np.abs(P), np.abs(xb))
    assert np.all(np.abs(z.cpu().numpy().reshape(5, m) - ref) <= 1e-15 * m * bound + 1e-300)


@pytest.mark.parametrize("shape,n,p", [("disk", 9, 1), ("disk", 9, 2), ("disk", 6, 3), ("disk", 5, 4),
                                       ("porous", 6, 1), ("porous", 5, 2), ("porous", 3, 3),
                                       ("porous", 3, 4), ("elastic", 5, 1), ("elastic", 4, 2),
                                       ("elastic", 3, 3)])
@pytest.mark.parametrize("eta_bar", [1.0, 0.9])
def test_lattice_blocks_are_the_matrix_blocks(shape, n, p, eta_bar):
    """The same system from its description (blocks read from lattice rows)
    and as a matrix (blocks found in its columns): the same inverses, bit for
    bit, and the same apply to rounding."""
    torch = require_gpu()
    if shape == "disk":
        d = fcgen.disk_poisson_2d(3, n=n, p=p)
    else:
        make = fcgen.porous_poisson_3d if shape == "porous" else fcgen.porous_elasticity_3d
        d = make(3, n=n, p=p, n_voids=3, rmin=0.08, rmax=0.16)
    hs = fc.HostSystem(d)
    e = hs.export()
    a = hs.upload()
    b = fc.Problem.from_matrix(e["n_dofs"], e["bsr_dim"], e["rowptr"], e["col"], e["val"], e["rhs"],
                               e["elem_dofs"], e["eta"])
    pa, pm = fc.Precond(a, eta_bar=eta_bar), fc.Precond(b, eta_bar=eta_bar)
    nb = pa.info()["n_blocks"]
    assert pa.info() == pm.info() and (pa.block_dropped() == pm.block_dropped()).all()
    for k in range(nb):
        assert pa.block_inverse(k).tobytes() == pm.block_inverse(k).tobytes(), k
    r = torch.as_tensor(np.random.default_rng(2).standard_normal(a.n), device="cuda")
    z, y = torch.empty_like(r), torch.empty_like(r)
    pa.apply_M(r, z)
    pm.apply_M(r, y)
    assert float((z - y).norm()) <= 1e-13 * float(y.norm())

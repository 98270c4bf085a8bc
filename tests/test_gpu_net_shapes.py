"""The network at the sizes where its kernels can go wrong: bricks cut by the
grid, coarse levels of one voxel, widths below, at and above a tile of channels,
batches that leave the chip idle and batches that fill it."""
import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from oracle import learned as L
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

CASES = [((8, 16, 32, 32), 2, 1, 2), ((8, 16, 32, 32), 2, 3, 5), ((3, 5, 17, 33), 1, 2, 9),
         ((8, 16, 32, 32), 2, 2, 33), ((16, 8, 48, 20), 5, 1, 12), ((4, 4, 4, 4), 3, 12, 17)]


@pytest.mark.parametrize("ch,in_ch,B,g", CASES)
def test_network_matches_oracle(ch, in_ch, B, g):
    torch = require_gpu()
    rng = np.random.default_rng(g)
    theta = fcgen.unet_init(ch, in_ch, seed=B)
    ref_theta = theta.astype(np.float64)
    off = 0
    for ci, co in L.layer_shapes(ch, in_ch).values():
        n = co * ci * 27
        # the GPU rounds weights (not biases) to BF16, nearest even
        u = theta[off: off + n].view(np.uint32).astype(np.uint64)
        ref_theta[off: off + n] = (((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000)
                                   .astype(np.uint32).view(np.float32))
        theta[off + n: off + n + co] = rng.standard_normal(co).astype(np.float32) * 0.1
        ref_theta[off + n: off + n + co] = theta[off + n: off + n + co]
        off += n + co
    x = rng.standard_normal((B, in_ch, g, g, g)).astype(np.float32)
    t = rng.standard_normal((B, 1, g, g, g)).astype(np.float32)
    m = fc.Model(theta, ch, in_ch)
    xd, td = torch.as_tensor(x, device="cuda"), torch.as_tensor(t, device="cuda")
    y = torch.full((B, 1, g, g, g), float("nan"), dtype=torch.float32, device="cuda")
    m.forward(xd, y)
    ref = L.forward(ref_theta, x.astype(np.float64), ch, in_ch)
    # FP32 accumulation; BF16 pairs in the weight gradient (2^-16 a product)
    assert np.abs(y.cpu().numpy() - ref).max() <= 2e-5 * np.abs(ref).max()
    loss, grad = m.loss_grad(xd, td)
    lo, go = L.loss_and_grad(ref_theta, x.astype(np.float64), t.astype(np.float64), ch, in_ch)
    assert abs(loss - lo) <= 1e-5 * abs(lo)
    off = 0
    for name, (ci, co) in L.layer_shapes(ch, in_ch).items():
        n = co * ci * 27 + co
        gg, gr = grad[off: off + n], go[off: off + n]
        off += n
        assert np.abs(gg - gr).max() <= 2e-4 * np.abs(gr).max(), name

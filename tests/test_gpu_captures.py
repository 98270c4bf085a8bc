"""Calls of this library while a graph is being captured elsewhere in the program:
they do their work, and the capture goes on and replays what it recorded.  Each
case in a process of its own, which a broken capture would leave unusable."""
import os
import subprocess
import sys
from pathlib import Path

import pytest

from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

_SCRIPT = """
import sys
import threading

import torch

import fcgen
import paper_1809_00828_amd as fc

what, mode = sys.argv[1:]
hs = fc.HostSystem(fcgen.disk_poisson_2d(1, n=20, p=2))
pb = hs.upload()
b = torch.ones(pb.n, dtype=torch.float64, device="cuda")
x, z = torch.empty_like(b), torch.empty_like(b)
side = torch.cuda.Stream()


def solved():
    pc = fc.Precond(pb)
    fc.pcg_solve(pb, pc, b, x, tol=0.0, maxit=40, timing=1)
    return pc


def problem():
    p = hs.upload(stream=side)
    pc = fc.Precond(p, stream=side)
    assert fc.pcg_solve(p, pc, b, x, tol=1e-9, check_every=4, stream=side)["status"] == "OK"
    assert (p.export()["val"] == hs.export()["val"]).all()
    assert pc.block_inverse(0).any()


def members():
    ps = [pb, fc.Problem.setup(fcgen.disk_poisson_2d(2, n=40, p=3))]
    bs = [torch.ones(p.n, dtype=torch.float64, device="cuda") for p in ps]
    return ps, [fc.Precond(p) for p in ps], bs, [torch.empty_like(v) for v in bs]


def batch(ps, pcs, bs, xs):
    bt = fc.Batch(ps, pcs, stream=side)
    for _ in range(2):
        infos = bt.solve(bs, xs, tol=1e-9, check_every=4, stream=side)
        assert all(i["status"] == "OK" for i in infos)


CH = (4, 4, 4, 4)
params = fcgen.unet_init(CH, 2, seed=1)


def model():
    return [torch.randn(2, c, 5, 5, 5, device="cuda") for c in (2, 1)]


def network(u, t):
    m = fc.Model(params, CH)
    m.set_params(2 * params)
    assert (m.params() == 2 * params).all()
    assert m.loss_grad(u, t, stream=side)[1].any()


def coarse():
    p = fc.Problem.setup(fcgen.porous_poisson_3d(1, n=4, p=1, n_voids=2, rmin=0.1, rmax=0.15))
    v = torch.ones(p.n, dtype=torch.float64, device="cuda")
    return p, fc.Precond(p), v, torch.empty_like(v), torch.empty(27, device="cuda")


def learned(p, pc, v, w, eta):
    m = fc.Model(params, CH)
    pc.attach(m)
    pc.coarse_channels(eta, eta)
    assert fc.pcg_solve(p, pc, v, w, tol=1e-8, mode="learned", stream=side)["status"] == "OK"
    assert pc.learned_stats()["applied"] > 0


ACTIONS = {  # name: (what is there before, the call)
    "destroy_precond": (lambda: [solved()], lambda have: have.clear()),
    "destroy_problem": (lambda: [hs.upload()], lambda have: have.clear()),
    "rebuild": (lambda: [solved()],
                lambda have: (have.clear(),
                              fc.Precond(pb, stream=side).apply_M(b, z, stream=side))),
    # a new problem, its first solve (the library's own capture), what it exports
    "problem": (lambda: None, lambda have: problem()),
    # members that stop at different steps: the lists are cut down in between
    "batch": (members, lambda have: batch(*have)),
    "model": (model, lambda have: network(*have)),
    "learned": (coarse, lambda have: learned(*have)),
}
make, act = ACTIONS[what]
have = make()
a, c = torch.ones(64, device="cuda"), torch.zeros(64, device="cuda")
torch.cuda.synchronize()
failed = []


def call():
    try:
        act(have)
    except Exception as e:
        failed.append(e)


g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, stream=torch.cuda.Stream(), capture_error_mode=mode):
    c.add_(a)
    if mode == "relaxed":
        call()
    else:
        t = threading.Thread(target=call)
        t.start()
        t.join()
    c.add_(a)
assert not failed, failed
for k in range(3):
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(c, 2.0 * (k + 1) * a)
"""


@pytest.mark.parametrize("what", ["destroy_precond", "destroy_problem", "rebuild", "problem", "batch",
                                  "model", "learned"])
@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_capture_goes_on(what, mode):
    """thread_local: the call comes from another thread than the capture's;
    relaxed: from the same one."""
    require_gpu()
    root = Path(__file__).resolve().parents[1]
    r = subprocess.run([sys.executable, "-c", _SCRIPT, what, mode], timeout=100, cwd=root,
                       env=dict(os.environ, PYTHONPATH=str(root)), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

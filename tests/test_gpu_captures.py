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


ACTIONS = {  # name: (what is there before, the call)
    "destroy_precond": (lambda: [solved()], lambda have: have.clear()),
    "destroy_problem": (lambda: [hs.upload()], lambda have: have.clear()),
    "rebuild": (lambda: [solved()],
                lambda have: (have.clear(),
                              fc.Precond(pb, stream=side).apply_M(b, z, stream=side))),
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


@pytest.mark.parametrize("what", ["destroy_precond", "destroy_problem", "rebuild"])
@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_capture_goes_on(what, mode):
    """thread_local: the call comes from another thread than the capture's;
    relaxed: from the same one."""
    require_gpu()
    root = Path(__file__).resolve().parents[1]
    r = subprocess.run([sys.executable, "-c", _SCRIPT, what, mode], timeout=100, cwd=root,
                       env=dict(os.environ, PYTHONPATH=str(root)), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

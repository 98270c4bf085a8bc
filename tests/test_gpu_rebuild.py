"""Buffers kept from one preconditioner to the next: rebuilds in several
threads on streams of their own give what a single build gives, and the memory
is given back with the last problem."""
import os
import subprocess
import sys
import threading
from pathlib import Path

import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def test_rebuilds_in_threads_equal_one_build():
    torch = require_gpu()
    descs = [fcgen.porous_elasticity_3d(1, n=4, p=2), fcgen.porous_poisson_3d(2, n=8, p=2),
             fcgen.disk_poisson_2d(3, n=20, p=3)]
    pbs = [fc.Problem.setup(d) for d in descs]
    rs = [torch.as_tensor(np.random.default_rng(k).standard_normal(p.n), device="cuda")
          for k, p in enumerate(pbs)]

    def once(k, eta_bar, stream):
        pc = fc.Precond(pbs[k], eta_bar=eta_bar, stream=stream)
        z, x = torch.empty_like(rs[k]), torch.empty_like(rs[k])
        pc.apply_M(rs[k], z, stream=stream)
        fc.pcg_solve(pbs[k], pc, rs[k], x, tol=0.0, maxit=4, stop="residual", stream=stream)
        stream.synchronize()
        return z.cpu().numpy(), x.cpu().numpy()

    jobs = [(k, e) for k in range(3) for e in (1.0, 0.9, -1.0)]
    ref = {j: once(*j, torch.cuda.current_stream()) for j in jobs}
    bad = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for rep in range(4):
                    for j in jobs[t % 3:] + jobs[:t % 3]:
                        for a, b in zip(once(*j, stream), ref[j]):
                            if a.tobytes() != b.tobytes():
                                bad.append((t, rep, j))
        except Exception as e:   # pytest only warns of a thread's exception
            bad.append((t, repr(e)))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


_GIVEN_BACK = """
import torch
import fcgen
import paper_1809_00828_amd as fc

torch.cuda.init()
fc.Precond(fc.Problem.setup(fcgen.disk_poisson_2d(0)))   # the library's own set-up is done
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
pb = fc.Problem.setup(fcgen.porous_elasticity_3d(1, n=8, p=3))   # 76 MB of inverses
for _ in range(3):
    fc.Precond(pb)
del pb
torch.cuda.synchronize()
assert torch.cuda.mem_get_info()[0] > before - (32 << 20)
"""


def test_memory_is_given_back_with_the_last_problem():
    # in a process of its own: here, other tests' problems may be alive
    require_gpu()
    root = Path(__file__).resolve().parents[1]
    subprocess.run([sys.executable, "-c", _GIVEN_BACK], check=True, timeout=100, cwd=root,
                   env=dict(os.environ, PYTHONPATH=str(root)))

"""Calls of several threads at once, each on a stream of its own: first solves (which
capture their steps) beside set-ups, batches that cut their lists, and networks; and
a preconditioner destroyed while work on it is still queued."""
import threading

import numpy as np
import pytest

import fcgen
import paper_1809_00828_amd as fc
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def test_threads_of_different_calls():
    torch = require_gpu()
    systems = [fc.HostSystem(fcgen.disk_poisson_2d(1, n=40, p=2)),
               fc.HostSystem(fcgen.porous_poisson_3d(2, n=8, p=2))]
    bs = [torch.as_tensor(np.random.default_rng(k).standard_normal(s.info()["n_dofs"]),
                          device="cuda") for k, s in enumerate(systems)]
    ch = (4, 4, 4, 4)
    params = fcgen.unet_init(ch, 2, seed=1)
    grids = [torch.ones(2, c, 9, 9, 9, device="cuda") for c in (2, 1)]
    shared = [s.upload() for s in systems]

    def solve(stream):   # a new problem, its first solve
        out = []
        for s, b in zip(systems, bs):
            p = s.upload(stream=stream)
            x = torch.empty_like(b)
            fc.pcg_solve(p, fc.Precond(p, stream=stream), b, x, tol=1e-9, check_every=4,
                         stream=stream)
            out.append(x)
        return out

    def batch(stream):   # members that stop at different steps
        pcs = [fc.Precond(p, stream=stream) for p in shared]
        xs = [torch.empty_like(b) for b in bs]
        fc.Batch(shared, pcs, stream=stream).solve(bs, xs, tol=1e-9, check_every=4, stream=stream)
        return xs

    def network(stream):
        m = fc.Model(params, ch)
        m.set_params(0.5 * params)
        return [torch.as_tensor(m.loss_grad(*grids, stream=stream)[1]),
                torch.as_tensor(m.params())]

    jobs = (solve, batch, network)
    ref = [[t.cpu() for t in j(torch.cuda.current_stream())] for j in jobs]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for rep in range(6):
                    out = jobs[k](stream)
                    stream.synchronize()
                    bad.extend((k, rep) for a, r in zip(out, ref[k]) if not torch.equal(a.cpu(), r))
        except Exception as e:   # pytest only warns of a thread's exception
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k % 3,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_destroying_waits_for_queued_work():
    """Work queued on a stream behind a pause of some 40 ms still finds the
    preconditioner's buffers as they were, although it is destroyed and one of the
    same sizes built at once."""
    torch = require_gpu()
    pbs = [fc.Problem.setup(fcgen.porous_elasticity_3d(k, n=4, p=2)) for k in (1, 2)]
    r = torch.as_tensor(np.random.default_rng(0).standard_normal(pbs[0].n), device="cuda")
    z, ref = torch.empty_like(r), torch.empty_like(r)
    fc.Precond(pbs[0]).apply_M(r, ref)
    torch.cuda.synchronize()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        pc = fc.Precond(pbs[0], stream=other)
        with torch.cuda.stream(side):
            torch.cuda._sleep(100_000_000)
            pc.apply_M(r, z)
        del pc
        fc.Precond(pbs[1], stream=other)
        torch.cuda.synchronize()
        assert torch.equal(z, ref)

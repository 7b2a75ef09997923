"""Members of a batch that have stopped cost nothing: the preconditioner by modes
leaves their slices alone, and the members still running are reduced over as
many blocks as if they ran alone."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dim,nx,nt,kw", [
    (2, 127, 40, {}), (2, 127, 40, {"mass": "q1"}), (2, 255, 9, {}), (3, 15, 6, {}), (3, 127, 3, {}),
    (2, 127, 40, {"precond": "ideal", "precision": "mixed", "side": "flexible"}), (2, 31, 40, {}), (3, 63, 80, {})])
def test_slices_of_stopped_members_stay(dim, nx, nt, kw):
    """The part of the workspace that an apply writes for member 0 is what
    changes with member 0's input; a solve in which member 0 stops at once
    (b = 0) does not touch it."""
    print(f"stopped members {dim} {nx} {nt} {kw}", flush=True)
    s = Solver(dim, nx, nt, [1e-3, 1e-5], restart=2, maxit=4, rtol=1e-14, device=DEV, **kw)
    words = s.workspace[: s.workspace.numel() // 4 * 4].view(torch.int32)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    v = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
    out = torch.empty_like(v)
    s.precond_apply(v, out=out)
    first = words.clone()
    v[0] = torch.randn(v[0].shape, dtype=torch.float64, device=DEV, generator=gen)
    s.precond_apply(v, out=out)
    before = words.clone()
    own = first != before
    assert int(own.sum()) >= (s.n * s.m if kw.get("precision") == "mixed" else 2 * s.n * s.m)
    b = v.clone()
    b[0] = 0
    s.solve(b)
    assert bool((words[own] == before[own]).all())


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("dim,nx,nt,batch", [(2, 15, 12, 9), (2, 63, 40, 20), (3, 7, 30, 5)])
def test_last_member_running(dim, nx, nt, batch, graph):
    """All members but one stop at once: the one left reaches its solution, in
    the steps that it takes alone."""
    print(f"one member of {batch}: {dim} {nx} {nt} graph {graph}", flush=True)
    gammas = [1e-4] * batch
    f = W.random_fields(dim, nx, nt, seed=41)
    pb = D.make_problem(dim, nx, nt, 1e-4)
    bo = D.rhs_scaled(pb, *f)
    kw = dict(graph=True, stream=torch.cuda.Stream()) if graph else {}
    for last in (0, batch - 1):
        s = Solver(dim, nx, nt, gammas, rtol=1e-10, device=DEV, **kw)
        b = s.new_vector()
        b[last] = torch.tensor(bo.reshape(b[last].shape), device=DEV)
        torch.cuda.synchronize()
        x, infos, _ = s.solve(b)
        one = Solver(dim, nx, nt, 1e-4, rtol=1e-10, device=DEV)
        x1, i1, _ = one.solve(b[last:last + 1].contiguous())
        assert infos[last].converged and infos[last].iters == i1[0].iters
        assert all(i.iters == 0 for k, i in enumerate(infos) if k != last)
        # two orders of summation of the same steps
        assert float((x[last] - x1[0]).norm()) <= 1e-12 * float(x1[0].norm())
        r = bo - D.kkt_scaled(pb) @ x[last].cpu().numpy().ravel()
        assert np.linalg.norm(r) <= 1.05e-10 * np.linalg.norm(bo)


def test_last_member_fills_the_chip():
    """Reductions and updates of the last of 64 members take about as long as
    alone (the same bytes over the same number of blocks); over a 64th of the
    blocks the updates took 33 times as long."""
    nx, nt, batch = 127, 64, 64
    ms = []
    for members in (1, batch):
        s = Solver(2, nx, nt, [1e-4] * members, restart=20, device=DEV)
        b = s.new_vector()
        gen = torch.Generator(device=DEV)
        gen.manual_seed(5)
        b[-1] = torch.randn(b[-1].shape, dtype=torch.float64, device=DEV, generator=gen)
        s.solve(b)
        runs = []
        for _ in range(3):
            s.timing_enable(True)
            _, infos, _ = s.solve(b)
            stats = s.timing_read()
            s.timing_enable(False)
            assert infos[-1].converged
            # (the first of the multi-dots is the norm of b, over every member)
            runs.append(stats["gs_update"]["ms"])
        ms.append(min(runs))
        del s, b
    print(f"updates alone {ms[0]:.3f} ms, as the last of {batch} {ms[1]:.3f} ms", flush=True)
    assert ms[1] <= 3.0 * ms[0]

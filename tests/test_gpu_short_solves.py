"""Solves that end after a few steps apply the operator hardly more often than
they take steps: blocks of Arnoldi steps start short where the tolerance is loose
and follow the rate of the last two steps.

One apply of the KKT operator per step, one for the initial and one for the final
residual; at most one step past the end."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("nx,nt", [(31, 32), (63, 20)])
@pytest.mark.parametrize("side", ["right", "left", "flexible"])
@pytest.mark.parametrize("gamma", [1e-8, 1e-4, 1.0])
@pytest.mark.parametrize("rtol", [0.5, 0.1, 1e-2, 1e-3])
def test_few_steps_few_applies(nx, nt, side, gamma, rtol):
    print(f"short solve {nx} {nt} {side} gamma {gamma} rtol {rtol}", flush=True)
    g, f, y0 = W.smooth_fields(2, nx, nt)
    s = Solver(2, nx, nt, gamma, side=side, rtol=rtol, device=DEV)
    b = s.rhs(*(torch.tensor(t[None], device=DEV) for t in (g, f, y0)))
    s.timing_enable(True)
    x, infos, _ = s.solve(b)
    stats = s.timing_read()
    s.timing_enable(False)
    steps = stats["kkt_apply"]["launches"] - 2
    print(f"  iterations {infos[0].iters} steps {steps}", flush=True)
    assert infos[0].converged and infos[0].iters <= steps <= infos[0].iters + 1
    if side != "left":
        pb = D.make_problem(2, nx, nt, gamma)
        bo = b.cpu().numpy().ravel()
        assert np.linalg.norm(bo - D.kkt_scaled(pb) @ x.cpu().numpy().ravel()) <= 1.05 * rtol * np.linalg.norm(bo)


def test_residual_that_falls_late():
    """Three steps to 1e-3, the third of which brings most: the rate of the
    first two says many more are left, and the next block has two steps at
    most."""
    nx, nt = 255, 256
    g, f, y0 = W.smooth_fields(2, nx, nt)
    s = Solver(2, nx, nt, 1e-4, rtol=1e-3, restart=20, device=DEV)
    b = s.rhs(*(torch.tensor(t[None], device=DEV) for t in (g, f, y0)))
    s.timing_enable(True)
    _, infos, hist = s.solve(b, history=True)
    steps = s.timing_read()["kkt_apply"]["launches"] - 2
    s.timing_enable(False)
    print(f"iterations {infos[0].iters} steps {steps} residuals {hist[0, :5]}", flush=True)
    assert infos[0].converged and steps <= infos[0].iters + 1

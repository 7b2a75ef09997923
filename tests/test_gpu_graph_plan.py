"""Graph solves where graphs and plain launches alternate: short first blocks of
loose tolerances, last blocks shorter than a graph, members that have stopped,
restarts, and a block that is cut.  Several right-hand sides on one context,
each solved again after eager work, against the eager solver.

The same kernels in the same order; only the blocks of a reduction may differ
once members have stopped: 1e-13 of the solution."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def right_hand_sides(s, dim, nx, nt, batch):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    smooth = [torch.tensor(np.repeat(t[None], batch, 0), device=DEV) for t in W.smooth_fields(dim, nx, nt)]
    noise = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
    stopped = noise.clone()
    stopped[: (batch + 1) // 2] = 0
    return [s.rhs(*smooth), noise, stopped]


def agree(sg, se, b):
    xe, ie, he = se.solve(b, history=True)
    for _ in range(2):
        xg, ig, hg = sg.solve(b, history=True)
        assert [i.iters for i in ig] == [i.iters for i in ie]
        assert [i.converged for i in ig] == [i.converged for i in ie]
        for k in range(sg.batch):
            assert float((xg[k] - xe[k]).norm()) <= 1e-13 * float(xe[k].norm())
        np.testing.assert_allclose(np.nan_to_num(hg), np.nan_to_num(he), rtol=1e-6, atol=1e-13)
        sg.kkt_apply(b)
        torch.cuda.synchronize()


@pytest.mark.parametrize("rtol,restart,chunk", [(0.5, 30, 4), (0.1, 30, 4), (1e-3, 5, 4), (1e-3, 30, 9), (1e-8, 30, 1),
                                                (1e-8, 30, 8), (1e-8, 7, 4), (1e-8, 3, 4), (1e-8, 1, 4)])
@pytest.mark.parametrize("kw", [{}, {"side": "left"}, {"precision": "mixed", "side": "flexible"}])
def test_graph_solves_match_eager(rtol, restart, chunk, kw):
    dim, nx, nt, batch = 2, 15, 24, 3
    print(f"graph plan rtol {rtol} restart {restart} chunk {chunk} {kw}", flush=True)
    args = dict(rtol=rtol, restart=restart, maxit=40, device=DEV, **kw)
    gammas = [1e-2, 1e-7, 1e-4]
    se = Solver(dim, nx, nt, gammas, **args)
    sg = Solver(dim, nx, nt, gammas, graph=True, graph_chunk=chunk, **args)
    for b in right_hand_sides(se, dim, nx, nt, batch):
        agree(sg, se, b)


@pytest.mark.parametrize("side", ["right", "left", "flexible"])
@pytest.mark.parametrize("graph,chunk", [(False, 4), (True, 4), (True, 8)])
def test_block_cut_for_one_member(side, graph, chunk):
    """One level and a right-hand side of a single sine mode: that member's
    Krylov space ends with its second vector, inside the first block, while the
    other member goes on."""
    dim, nx, nt, gammas = 2, 7, 2, [1e-3, 1e-6]
    print(f"block cut {side} graph {graph} chunk {chunk}", flush=True)
    s = Solver(dim, nx, nt, gammas, side=side, rtol=1e-11, graph=graph, graph_chunk=chunk, device=DEV)
    rng = np.random.default_rng(8)
    mode = W.sine_product(W.mesh(dim, nx))
    b = np.stack([np.stack([0.7 * mode, -0.4 * mode]), rng.standard_normal((2, nx * nx))]).reshape(s.vec_shape)
    tb = torch.tensor(b, device=DEV)
    for _ in range(3):
        x, infos, _ = s.solve(tb)
        assert infos[0].converged and infos[0].iters <= 2
        assert infos[1].converged and infos[1].iters > 2
        for k, gm in enumerate(gammas):
            A = D.kkt_scaled(D.make_problem(dim, nx, nt, gm)).toarray()
            xs = np.linalg.solve(A, b[k].ravel())
            # ||A^-1|| ||A|| is below 1e4 on this grid
            assert np.linalg.norm(x[k].cpu().numpy().ravel() - xs) <= 1e-7 * np.linalg.norm(xs)
        s.kkt_apply(tb)
        torch.cuda.synchronize()

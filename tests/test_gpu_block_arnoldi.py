"""Block Gram-Schmidt (2 to 4 Arnoldi steps orthogonalised together) against
the oracle's step-by-step modified Gram-Schmidt GMRES.

Restart lengths and step counts around the block length give every block size
and first and last blocks of a cycle, one long cycle every basis size; the
shapes give vectors of one partial chunk of 128 values, of whole chunks and of
many; the degenerate ones exhaust the Krylov space inside a block.

Both compute the same iterate in exact arithmetic.  A step's column carries an
error of about 1e-16 over the share of the vector that the pass leaves, 1e-3 at
worst over four steps, times the condition of the small least-squares problem
(at most about 1e3 here): 1e-10 in the iterate.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D, krylov as KR, precond as P
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV)


def rel(a, b):
    return np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b))


@pytest.mark.parametrize("side", ["right", "left", "flexible"])
@pytest.mark.parametrize("restart,k", [(1, 2), (2, 5), (3, 7), (4, 8), (5, 9), (6, 6), (7, 13)])
def test_block_steps_match_oracle(side, restart, k):
    dim, nx, nt, gamma, eps, T = 2, 7, 24, 1e-3, 0.99, 0.005
    print(f"block {side} restart={restart} k={k}", flush=True)
    g, f, y0 = W.random_fields(dim, nx, nt, seed=5)
    pb = D.make_problem(dim, nx, nt, gamma, eps=eps, T=T)
    A = D.kkt_scaled(pb)
    bo = D.rhs_scaled(pb, g, f, y0)
    s = Solver(dim, nx, nt, gamma, T=T, eps=eps, side=side, restart=restart, maxit=k, rtol=1e-12, device=DEV)
    x, infos, hist = s.solve(s.rhs(dev(g[None]), dev(f[None]), dev(y0[None])), history=True)
    res = KR.gmres(lambda v: A @ v, bo, P.EpsCirculantRBD(pb).apply, side=side, restart=restart, maxit=k, rtol=1e-12)
    assert infos[0].iters == res.iters
    assert rel(x.cpu().numpy(), res.x) < 1e-10
    n = res.iters + 1
    np.testing.assert_allclose(hist[0, :n], res.history[:n], rtol=1e-8, atol=1e-12)


@pytest.mark.parametrize("side", ["right", "left", "flexible"])
@pytest.mark.parametrize("k", [39, 40])
def test_block_steps_up_to_the_largest_basis(side, k):
    """The iterate after 39 or 40 steps without a restart is an ill-conditioned
    function of b (step-by-step classical and modified Gram-Schmidt already
    differ by 1e-10 in it): the bound is the change of the oracle's iterate
    under a relative change of 1e-15 in b, over the share of 1e-3."""
    dim, nx, nt, gamma, eps, T = 2, 7, 24, 1e-3, 0.99, 0.005
    print(f"block {side} restart=40 k={k}", flush=True)
    g, f, y0 = W.random_fields(dim, nx, nt, seed=5)
    pb = D.make_problem(dim, nx, nt, gamma, eps=eps, T=T)
    A = D.kkt_scaled(pb)
    bo = D.rhs_scaled(pb, g, f, y0)
    pc = P.EpsCirculantRBD(pb)
    s = Solver(dim, nx, nt, gamma, T=T, eps=eps, side=side, restart=40, maxit=k, rtol=1e-12, device=DEV)
    x, infos, _ = s.solve(s.rhs(dev(g[None]), dev(f[None]), dev(y0[None])))
    run = lambda v: KR.gmres(lambda u: A @ u, v, pc.apply, side=side, restart=40, maxit=k, rtol=1e-12)
    res = run(bo)
    moved = run(bo * (1.0 + 1e-15 * np.random.default_rng(0).standard_normal(bo.size)))
    assert infos[0].iters == res.iters == k
    assert rel(x.cpu().numpy(), res.x) < 1e3 * rel(moved.x, res.x) + 1e-10


@pytest.mark.parametrize("dim,nx,nt", [(2, 3, 2), (2, 3, 8), (2, 15, 4), (3, 3, 3), (2, 31, 40), (3, 7, 33)])
def test_block_solves_over_vector_lengths(dim, nx, nt):
    """Two members of different gamma, converged; (2, 3, 2) has 18 unknowns,
    fewer than a solve to 1e-12 would take steps."""
    gammas = (1e-2, 1e-6)
    print(f"block lengths {dim} {nx} {nt}", flush=True)
    fl = [W.random_fields(dim, nx, nt, seed=70 + b) for b in range(2)]
    s = Solver(dim, nx, nt, list(gammas), rtol=1e-12, device=DEV)
    x, infos, _ = s.solve(s.rhs(*(dev(np.stack([q[i] for q in fl])) for i in range(3))))
    xs = x.cpu().numpy()
    for b, gm in enumerate(gammas):
        assert infos[b].converged and infos[b].relres_true < 1e-11
        pb = D.make_problem(dim, nx, nt, gm)
        A = D.kkt_scaled(pb)
        r = D.rhs_scaled(pb, *fl[b]) - A @ xs[b].ravel()
        assert np.linalg.norm(r) <= 1e-11 * np.linalg.norm(D.rhs_scaled(pb, *fl[b]))


@pytest.mark.parametrize("graph", [False, True])
def test_block_mg_fp32_matches_fp64_solution(graph):
    """FP32 V-cycles run shifted blocks: the solution agrees with the FP64
    solve to the residual tolerance."""
    dim, nx, nt, gammas = 2, 15, 20, (1e-3, 1e-6)
    fl = [W.random_fields(dim, nx, nt, seed=90 + b) for b in range(2)]
    xs = []
    for precision in ("fp64", "mixed"):
        s = Solver(dim, nx, nt, list(gammas), coeff=W.coeff_sines3d, spatial="mg", side="flexible", rtol=1e-11,
                   precision=precision, graph=graph, stream=torch.cuda.Stream() if graph else None, device=DEV)
        x, infos, _ = s.solve(s.rhs(*(dev(np.stack([q[i] for q in fl])) for i in range(3))))
        assert all(i.converged and i.relres_true <= 1.1e-11 for i in infos)
        xs.append(x.cpu().numpy())
    # ||x - x'|| <= ||A^-1|| (two residuals of 1e-11 ||b||), ||A^-1|| ||b|| / ||x|| below 1e4 here
    assert rel(xs[1], xs[0]) < 1e-6


def test_zero_and_exhausted_right_hand_sides():
    """b = 0 returns x = 0; a right-hand side P e, whose Krylov space is
    small, ends inside a block."""
    dim, nx, nt = 2, 3, 6
    s = Solver(dim, nx, nt, [1e-3, 1e-3], device=DEV)
    b = s.new_vector()
    b[1, 0, 0, 4] = 1.0
    x, infos, _ = s.solve(b)
    assert infos[0].converged and infos[0].iters == 0 and float(x[0].abs().max()) == 0.0
    assert infos[1].converged and infos[1].relres_true <= 1.05e-8

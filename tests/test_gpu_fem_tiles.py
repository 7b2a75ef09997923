"""Finite-element matvec over the grids where its tiles and level chunks end:
3-D tiles of 16 x 16 x 4 points (nx = 15, 31, 63 leave a part of the last, 7
takes the kernel without tiles), chunks of 1 to 16 levels with a remainder, the
residual form through the true residual of an unconverged solve.

A 27-point sum of products against the sparse matrix product: 1e-14 of the
whole vector (a few ulps of the largest products)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHAPES = [(3, 7, 40, 2), (3, 15, 2, 1), (3, 15, 30, 2), (3, 15, 400, 1), (3, 31, 18, 1), (3, 31, 70, 3), (3, 63, 20, 1),
          (2, 15, 2, 1), (2, 31, 70, 2), (2, 63, 600, 1)]


@pytest.mark.parametrize("dim,nx,nt,batch", SHAPES)
def test_fem_matvec_tiles(dim, nx, nt, batch):
    gammas = [10.0 ** (-1 - 3 * b) for b in range(batch)]
    print(f"fem tiles {dim} {nx} {nt} {batch}", flush=True)
    s = Solver(dim, nx, nt, gammas, mass="q1", restart=1, maxit=1, device=DEV)
    x = W.random_vector(dim, nx, nt, seed=8, batch=batch)
    dx = torch.tensor(x, device=DEV)
    for transpose in (False, True):
        y = s.kkt_apply(dx, transpose=transpose).cpu().numpy()
        for b, gm in enumerate(gammas):
            yo = D.kkt_apply_blocks(D.make_problem(dim, nx, nt, gm, mass="q1"), x[b].ravel(), transpose)
            d = y[b].ravel() - yo
            assert np.linalg.norm(d) <= 1e-14 * np.linalg.norm(yo)
            assert np.abs(d).max() <= 1e-13 * np.abs(yo).max()


@pytest.mark.parametrize("dim,nx,nt", [(3, 15, 9), (3, 31, 20), (2, 31, 40)])
def test_fem_residual_form(dim, nx, nt):
    gammas = [1e-2, 1e-6]
    s = Solver(dim, nx, nt, gammas, mass="q1", maxit=3, rtol=1e-14, device=DEV)
    b = torch.tensor(W.random_vector(dim, nx, nt, seed=9, batch=2), device=DEV)
    x0 = torch.tensor(W.random_vector(dim, nx, nt, seed=10, batch=2), device=DEV)
    x, infos, _ = s.solve(b, x0=x0)
    for k, gm in enumerate(gammas):
        pb = D.make_problem(dim, nx, nt, gm, mass="q1")
        r = b[k].cpu().numpy().ravel() - D.kkt_apply_blocks(pb, x[k].cpu().numpy().ravel(), False)
        want = np.linalg.norm(r) / np.linalg.norm(b[k].cpu().numpy())
        assert abs(infos[k].relres_true - want) <= 1e-11 * want

"""KKT matvec over the grids where the 3-D blocks (a column of four planes per
thread) end: planes of one ragged tile (nx = 3, 7, 15), several (31, 63), the
larger halo (127); automatic level chunks of 1 to 8 with a remainder; the
residual form through the true residual of an unconverged solve, in 2-D as
well.

At most eleven products per element against the sparse product: 1e-14 of the
whole vector, the bound of the other matvec tests."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHAPES = [(3, 3, 5, 2, None), (3, 7, 9, 1, None), (3, 15, 50, 2, None), (3, 31, 70, 1, None), (3, 63, 9, 1, None),
          (3, 127, 3, 1, None), (3, 15, 100, 3, W.coeff_sines3d), (3, 31, 9, 1, W.coeff_sines3d),
          (3, 127, 2, 1, W.coeff_sines3d)]


@pytest.mark.parametrize("dim,nx,nt,batch,coeff", SHAPES)
def test_kkt_tiles(dim, nx, nt, batch, coeff):
    gammas = [10.0 ** (-1 - 3 * b) for b in range(batch)]
    print(f"kkt tiles {dim} {nx} {nt} {batch} {coeff is not None}", flush=True)
    s = Solver(dim, nx, nt, gammas, coeff=coeff, spatial="dst" if coeff is None else "mg", restart=1, maxit=1, device=DEV)
    x = W.random_vector(dim, nx, nt, seed=8, batch=batch)
    dx = torch.tensor(x, device=DEV)
    for transpose in (False, True):
        y = s.kkt_apply(dx, transpose=transpose).cpu().numpy()
        for b, gm in enumerate(gammas):
            yo = D.kkt_apply(D.make_problem(dim, nx, nt, gm, coeff=coeff), x[b].ravel(), transpose=transpose)
            d = y[b].ravel() - np.asarray(yo).ravel()
            assert np.linalg.norm(d) <= 1e-14 * np.linalg.norm(yo)


@pytest.mark.parametrize("dim,nx,nt", [(3, 7, 9), (3, 31, 40), (3, 63, 6), (3, 127, 2), (2, 15, 20), (2, 63, 50), (2, 255, 9)])
def test_kkt_residual_form(dim, nx, nt):
    gammas = [1e-2, 1e-6]
    s = Solver(dim, nx, nt, gammas, maxit=3, rtol=1e-14, device=DEV)
    b = torch.tensor(W.random_vector(dim, nx, nt, seed=9, batch=2), device=DEV)
    x0 = torch.tensor(W.random_vector(dim, nx, nt, seed=10, batch=2), device=DEV)
    x, infos, _ = s.solve(b, x0=x0)
    for k, gm in enumerate(gammas):
        pb = D.make_problem(dim, nx, nt, gm)
        r = b[k].cpu().numpy().ravel() - np.asarray(D.kkt_apply(pb, x[k].cpu().numpy().ravel())).ravel()
        want = np.linalg.norm(r) / np.linalg.norm(b[k].cpu().numpy())
        assert abs(infos[k].relres_true - want) <= 1e-11 * want

"""The V-cycle's one-launch coarse end and the one-wave lexicographic sweeps
against the oracle's V-cycle, for each smoother: hierarchies that are all coarse
end (2-D nx <= 63, 3-D nx <= 15, one point), that have levels above it, one and
two and four columns per lane, and members switched off.

One cycle is a few sweeps of multiplications by at most 1 and divisions by
diagonals of modulus at least 1: 1e-12 of the vector in FP64 with D_eps's
conditioning (as the other cycle tests), 1e-5 in FP32."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D, precond as P
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dim,nx,nt,batch", [(2, 1, 4, 2), (2, 3, 5, 1), (2, 7, 6, 3), (2, 63, 4, 2), (2, 127, 4, 1), (2, 255, 3, 1),
                                             (3, 1, 3, 1), (3, 3, 5, 2), (3, 15, 4, 1), (3, 31, 3, 1)])
@pytest.mark.parametrize("smoother", ["rb", "lex", "sym"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_cycle_matches_oracle(dim, nx, nt, batch, smoother, precision):
    gammas = [10.0 ** (-2 - 2 * b) for b in range(batch)]
    print(f"mg tail {precision} {smoother} {dim} {nx} {nt} {batch}", flush=True)
    s = Solver(dim, nx, nt, gammas, coeff=W.coeff_sines3d, spatial="mg", side="flexible", precision=precision,
               mg_smoother=smoother, restart=1, device=DEV)
    v = W.random_vector(dim, nx, nt, seed=4, batch=batch)
    w = s.precond_apply(torch.tensor(v, device=DEV)).cpu().numpy()
    tol = 1e-5 if precision == "mixed" else 1e-11
    for b, gm in enumerate(gammas):
        pb = D.make_problem(dim, nx, nt, gm, coeff=W.coeff_sines3d)
        wo = P.EpsCirculantRBD(pb, spatial="mg", coeff=W.coeff_sines3d, smoother=smoother).apply(v[b].ravel())
        d = w[b].ravel() - wo
        assert np.linalg.norm(d) <= tol * np.linalg.norm(wo)
        assert np.abs(d).max() <= 10 * tol * np.abs(wo).max()


@pytest.mark.parametrize("smoother", ["rb", "sym"])
@pytest.mark.parametrize("nx", [15, 127])
def test_members_that_stop_early(smoother, nx):
    """Members of very different gamma: later cycles skip the converged ones."""
    gammas = [1e-8, 1e-1, 1e-4]
    fl = [W.random_fields(2, nx, 6, seed=20 + b) for b in range(3)]
    s = Solver(2, nx, 6, gammas, coeff=W.coeff_sines3d, spatial="mg", side="flexible", mg_smoother=smoother, device=DEV)
    x, infos, _ = s.solve(s.rhs(*(torch.tensor(np.stack([q[i] for q in fl]), device=DEV) for i in range(3))))
    assert len({i.iters for i in infos}) > 1
    for b, gm in enumerate(gammas):
        pb = D.make_problem(2, nx, 6, gm, coeff=W.coeff_sines3d)
        bo = D.rhs_scaled(pb, *fl[b])
        r = bo - D.kkt_scaled(pb) @ x[b].cpu().numpy().ravel()
        assert np.linalg.norm(r) <= 1.05e-8 * np.linalg.norm(bo)

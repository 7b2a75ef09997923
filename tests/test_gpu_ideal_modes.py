"""The ideal preconditioner by modes (sine transforms of all steps, scalar
recurrences along time) against the oracle's sequential substitution: step
counts below, at and past the 16 time chunks of a block and past the 8 loads of
a thread, mode counts that leave a part of a block, and grids large enough for
one chunk.

Both orders of summation are backward stable solves of the same systems
(condition at most 1 + tau ||K||, 1e3 here, every recurrence contracting):
1e-12, and 1e-5 with FP32 transforms."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D, precond as P
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dim,nx,nt,batch", [(2, 7, 3, 1), (2, 7, 17, 2), (2, 15, 18, 1), (2, 31, 40, 1), (2, 7, 150, 1),
                                             (3, 7, 34, 2), (2, 255, 3, 2), (2, 255, 12, 2)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_ideal_by_modes(dim, nx, nt, batch, precision):
    gammas = [10.0 ** (-2 - 3 * b) for b in range(batch)]
    print(f"ideal modes {precision} {dim} {nx} {nt} {batch}", flush=True)
    s = Solver(dim, nx, nt, gammas, precision=precision, side="flexible" if precision == "mixed" else "right",
               precond="ideal", restart=2, device=DEV)
    v = W.random_vector(dim, nx, nt, seed=3, batch=batch)
    dv = torch.tensor(v, device=DEV)
    w = s.precond_apply(dv).cpu().numpy()
    for b, gm in enumerate(gammas):
        wo = P.IdealRBD(D.make_problem(dim, nx, nt, gm)).apply(v[b]).reshape(w[b].shape)
        tol = 1e-5 if precision == "mixed" else 1e-12
        assert np.linalg.norm(w[b] - wo) <= tol * np.linalg.norm(wo)
        # every level, so that a lost chunk shows
        lev = np.abs(w[b] - wo).max(axis=2)
        assert lev.max() <= 10 * tol * np.abs(wo).max()
    s.precond_apply(dv, out=dv)  # in place
    assert np.array_equal(dv.cpu().numpy(), w)

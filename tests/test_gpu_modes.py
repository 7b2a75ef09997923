"""The preconditioner by modes (FP64 sine transforms, automatic kernels) against
the oracle's four steps and against the library's own time-transform path.

Shapes: one and two steps, odd and even step counts, the smallest lines, every
line length, Q1 elements, and both ways of running the recurrences -- scans
inside a block (with 16 chunks or one) and marching chunks, with a remainder in
the last chunk and tiles that leave a part.

Both are exact solves of systems with condition 1 + tau ||K|| up to rounding;
the time transforms add the conditioning 1/eps = sqrt(n) of D_eps: 1e-11
against the oracle (which has it too), 1e-12 between the two paths at up to
some 500 steps."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import discretize as D, precond as P
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dim,nx,nt,batch", [(2, 7, 2, 1), (2, 7, 3, 2), (2, 15, 18, 2), (2, 31, 9, 1), (3, 7, 20, 2), (3, 15, 4, 1),
                                             (2, 7, 130, 1), (2, 63, 6, 1)])
@pytest.mark.parametrize("mass", ["identity", "q1"])
def test_modes_match_oracle(dim, nx, nt, batch, mass):
    gammas = [10.0 ** (-1 - 4 * b) for b in range(batch)]
    print(f"modes oracle {mass} {dim} {nx} {nt} {batch}", flush=True)
    s = Solver(dim, nx, nt, gammas, mass=mass, restart=1, device=DEV)
    v = W.random_vector(dim, nx, nt, seed=12, batch=batch)
    dv = torch.tensor(v, device=DEV)
    s.timing_enable(True)
    w = s.precond_apply(dv).cpu().numpy()
    assert "time_fwd" not in s.timing_read() and "modes" in s.timing_read()
    s.timing_enable(False)
    for b, gm in enumerate(gammas):
        wo = P.EpsCirculantRBD(D.make_problem(dim, nx, nt, gm, mass=mass)).apply(v[b].ravel()).reshape(w[b].shape)
        assert np.linalg.norm(w[b] - wo) <= 1e-11 * np.linalg.norm(wo)
        assert np.abs(w[b] - wo).max() <= 1e-10 * np.abs(wo).max()
    s.precond_apply(dv, out=dv)  # in place
    assert np.array_equal(dv.cpu().numpy(), w)


@pytest.mark.parametrize("dim,nx,nt,batch,mass", [
    (2, 15, 200, 3, "identity"), (2, 31, 140, 64, "identity"), (2, 31, 141, 70, "q1"), (2, 63, 70, 40, "identity"),
    (2, 127, 70, 16, "identity"), (2, 127, 360, 1, "identity"), (2, 255, 100, 2, "q1"), (2, 255, 256, 1, "identity"),
    (2, 511, 70, 1, "identity"), (2, 511, 75, 1, "q1"), (3, 15, 115, 40, "identity"), (3, 31, 130, 2, "q1"),
    (3, 63, 70, 1, "identity"), (3, 63, 73, 1, "q1"), (3, 7, 500, 4, "identity")])
def test_modes_match_time_transforms(dim, nx, nt, batch, mass):
    gammas = list(10.0 ** np.linspace(-9, 0, batch)) if batch > 1 else [1e-4]
    print(f"modes path {mass} {dim} {nx} {nt} {batch}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    out = []
    for tc in (0, -1):
        s = Solver(dim, nx, nt, gammas, mass=mass, restart=1, time_cols=tc, device=DEV)
        if not out:
            v = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
        out.append(s.precond_apply(v))
        del s
    d = out[0] - out[1]
    for b in range(batch):
        assert float(d[b].norm()) <= 1e-12 * float(out[1][b].norm())
        # every level of both blocks
        assert float(d[b].abs().amax(dim=2).max()) <= 1e-11 * float(out[1][b].abs().max())


@pytest.mark.parametrize("side", ["right", "left", "flexible"])
@pytest.mark.parametrize("nx,nt,batch", [(15, 20, 3), (31, 140, 64)])
def test_modes_in_solves(side, nx, nt, batch):
    """Masked members and the accumulating last pass: the solves agree with
    those through the time transforms."""
    gammas = list(10.0 ** np.linspace(-8, -1, batch))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    xs, its = [], []
    for tc in (0, -1):
        s = Solver(2, nx, nt, gammas, side=side, time_cols=tc, device=DEV)
        if not xs:
            b = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
        x, infos, _ = s.solve(b)
        assert all(i.converged for i in infos)
        xs.append(x)
        its.append([i.iters for i in infos])
        del s
    assert its[0] == its[1] and len(set(its[0])) > 1
    for k in range(batch):
        assert float((xs[0][k] - xs[1][k]).norm()) <= 1e-10 * float(xs[1][k].norm())

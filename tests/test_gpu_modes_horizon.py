"""The preconditioner by modes where 1 - eps d^{-n} nearly cancels: eps at or
near 1 (the circulant preconditioner) and a short horizon, d = 1 + alpha + tau mu
just above 1.  Reference: the scalar systems of the sine modes in long double.

Shapes: scans in 16 chunks and in one, marching chunks, Q1 elements.

Each of the n steps of a recurrence rounds its value once or twice (1.1e-16
each), the transforms some forty times, delta and the closing factor a few
times: (2 n + 60) 1.1e-16 of the member bounds the sum of all."""
import numpy as np
import pytest
import torch

from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
LD = np.longdouble


def sine_matrix(nx):
    k = np.arange(1, nx + 1, dtype=LD)
    pi = np.arccos(LD(-1))
    return np.sqrt(LD(2) / (nx + 1)) * np.sin(pi * np.outer(k, k) / (nx + 1)), pi


def transform(v, S, dim, nx):
    v = v.reshape(v.shape[0], *([nx] * dim))
    for ax in range(1, dim + 1):
        v = np.moveaxis(np.tensordot(v, S, axes=([ax], [0])), -1, ax)
    return v.reshape(v.shape[0], -1)


def exact(v, dim, nx, T, nt, gamma, eps, mass):
    """P_eps^{-1} v of one member, v [2][n][m]."""
    n, tau, h = nt - 1, LD(T) / nt, LD(1) / (nx + 1)
    S, pi = sine_matrix(nx)
    k = np.arange(1, nx + 1, dtype=LD)
    mu1 = 4 / (h * h) * np.sin(pi * k * h / 2) ** 2
    im1 = np.ones(nx, dtype=LD)
    if mass == "q1":
        mk = h / 3 * (2 + np.cos(pi * k * h))
        mu1 = 4 / h * np.sin(pi * k * h / 2) ** 2 / mk
        im1 = 1 / mk
    mu, im = np.zeros((nx,) * dim, dtype=LD), np.ones((nx,) * dim, dtype=LD)
    for ax in range(dim):
        shape = [1] * dim
        shape[ax] = nx
        mu, im = mu + mu1.reshape(shape), im * im1.reshape(shape)
    delta = tau / np.sqrt(LD(gamma)) + tau * mu.ravel()
    eps = LD(eps)

    def solve(y):
        d = 1 + delta
        z = np.zeros_like(delta)
        for s in range(n):
            z = (y[s] + z) / d
        z = eps * z / ((1 - eps) - eps * np.expm1(-n * np.log1p(delta)))
        out = np.empty_like(y)
        for s in range(n):
            z = (y[s] + z) / d
            out[s] = z
        return out

    y1, y2 = (transform(v[b].astype(LD), S, dim, nx) * im.ravel() for b in (0, 1))
    z2, z1 = solve(y2), solve(y1[::-1])[::-1]
    z1, z2 = transform(z1, S, dim, nx), transform(z2, S, dim, nx)
    return np.stack([z1 - z2, z1 + z2])


@pytest.mark.parametrize("eps,T", [(1.0, 1e-6), (1.0, 1e-4), (0.99, 1e-3), (1.0 - 1e-6, 1e-2), (None, 1.0)])
@pytest.mark.parametrize("dim,nx,nt,batch,mass", [(2, 7, 3, 1, "identity"), (2, 15, 128, 1, "identity"), (2, 15, 60, 2, "q1"),
                                                  (2, 63, 20, 17, "identity"), (3, 15, 130, 40, "identity"),
                                                  (3, 15, 131, 40, "q1")])
def test_short_horizons(dim, nx, nt, batch, mass, eps, T):
    gammas = list(10.0 ** np.linspace(-2, 6, batch)) if batch > 1 else [1e2]
    print(f"short horizon {mass} {dim} {nx} {nt} {batch} eps {eps} T {T}", flush=True)
    s = Solver(dim, nx, nt, gammas, T=T, eps=eps, mass=mass, restart=1, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    v = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen) + 1.0
    w = s.precond_apply(v)
    for b in sorted({0, batch - 1}):
        ex = exact(v[b].cpu().numpy(), dim, nx, T, nt, gammas[b], s.eps, mass)
        err = float(np.linalg.norm(w[b].cpu().numpy() - ex) / np.linalg.norm(ex))
        assert err <= (2 * (nt - 1) + 60) * 1.1e-16, (b, err)

"""Whole (x1, x2) planes of the preconditioner by modes (nx <= 63) against the
library's own time-transform path: blocks with one, two and eight planes of which
the last holds a part, odd step counts (a middle slice that is its own partner),
one step, several planes per slice (3-D), masked members, and the FP32 planes of
the ideal preconditioner against its FP64 ones.

FP64: 1e-12 of the member, the bound between the two paths.  FP32: a transform of
63 x 63 points sums some 2 x 6 stages of rounding 6e-8 twice: 5e-6."""
import numpy as np
import pytest
import torch

from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHAPES = [(2, 7, 2, 1), (2, 7, 6, 3), (2, 7, 8, 5), (2, 15, 2, 1), (2, 15, 8, 3), (2, 31, 2, 1), (2, 31, 38, 3), (2, 63, 2, 1),
          (2, 63, 34, 2), (2, 63, 300, 17), (3, 7, 4, 1), (3, 15, 8, 3), (3, 31, 10, 1), (3, 63, 4, 1)]


def _vector(s, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)


@pytest.mark.parametrize("dim,nx,nt,batch", SHAPES)
@pytest.mark.parametrize("odd", [0, 1])
def test_planes_match_time_transforms(dim, nx, nt, batch, odd):
    nt += odd
    print(f"planes {dim} {nx} {nt} {batch}", flush=True)
    gammas = list(10.0 ** np.linspace(-9, 0, batch)) if batch > 1 else [1e-4]
    out, v = [], None
    for tc in (0, -1):
        s = Solver(dim, nx, nt, gammas, restart=1, time_cols=tc, device=DEV)
        v = _vector(s, 21) if v is None else v
        out.append(s.precond_apply(v))
    for b in range(batch):
        d = out[0][b] - out[1][b]
        assert float(d.norm()) <= 1e-12 * float(out[1][b].norm())
        assert float(d.abs().max()) <= 1e-11 * float(out[1][b].abs().max())


@pytest.mark.parametrize("dim,nx,nt,batch", [(2, 7, 9, 3), (2, 31, 20, 2), (2, 63, 33, 2), (3, 15, 6, 2), (3, 63, 3, 1)])
def test_planes_fp32(dim, nx, nt, batch):
    gammas = [10.0 ** (-2 - 3 * b) for b in range(batch)]
    out, v = [], None
    for kw in ({}, {"precision": "mixed", "side": "flexible"}):
        s = Solver(dim, nx, nt, gammas, restart=1, precond="ideal", device=DEV, **kw)
        v = _vector(s, 22) if v is None else v
        out.append(s.precond_apply(v))
    for b in range(batch):
        assert float((out[1][b] - out[0][b]).norm()) <= 5e-6 * float(out[0][b].norm())

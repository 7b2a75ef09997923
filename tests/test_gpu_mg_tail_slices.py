"""The V-cycle's one-launch coarse end with few and with many slices, where it
starts a level lower and runs smaller blocks: each member of a large batch gets
what it gets alone.

Both run the same operations per point; only FP32 pairs of points may round
differently (1e-6 of the member, as a few 6e-8)."""
import pytest
import torch

import workloads as W
from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# slices per member 2 (n/2 + 1); the rules change at 256 and 1024 slices
SHAPES = [(2, 3, 33, 40), (2, 7, 33, 40), (2, 15, 33, 40), (2, 31, 33, 40), (2, 63, 33, 40), (2, 127, 33, 40),
          (3, 3, 33, 12), (3, 7, 33, 12), (3, 15, 33, 12), (3, 31, 33, 12)]


@pytest.mark.parametrize("dim,nx,nt,batch", SHAPES)
@pytest.mark.parametrize("smoother", ["rb", "lex", "sym"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_members_of_a_batch_match_single_members(dim, nx, nt, batch, smoother, precision):
    print(f"mg slices {precision} {smoother} {dim} {nx} {nt} {batch}", flush=True)
    kw = dict(coeff=W.coeff_sines3d, spatial="mg", side="flexible", precision=precision, mg_smoother=smoother, restart=1,
              device=DEV)
    many = Solver(dim, nx, nt, [10.0 ** (-1 - b % 7) for b in range(batch)], **kw)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(17)
    v = torch.randn(many.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
    w = many.precond_apply(v)
    for b in (0, batch - 1):
        one = Solver(dim, nx, nt, 10.0 ** (-1 - b % 7), **kw)
        w1 = one.precond_apply(v[b:b + 1].contiguous())
        tol = 1e-6 if precision == "mixed" else 1e-14
        assert float((w[b] - w1[0]).norm()) <= tol * float(w1.norm())


@pytest.mark.parametrize("dim,nx,batch,smoother,own", [
    (3, 15, 1, "lex", False), (3, 15, 9, "lex", True), (2, 63, 9, "sym", False), (2, 63, 31, "sym", True),
    (3, 15, 1, "rb", True), (2, 63, 1, "rb", True), (2, 31, 40, "rb", False)])
def test_large_level_by_itself(dim, nx, batch, smoother, own):
    """One block per CU in FP64: red-black, and from one round (3-D) or four (2-D)
    of slices on also lexicographic, the level is smoothed in launches of its
    own."""
    s = Solver(dim, nx, 33, [1e-3] * batch, coeff=W.coeff_sines3d, spatial="mg", side="flexible", mg_smoother=smoother,
               restart=1, device=DEV)
    s.timing_enable(True)
    s.precond_apply(torch.randn(s.vec_shape, dtype=torch.float64, device=DEV))
    launches = s.timing_read()["mg_smooth"]["launches"]
    s.timing_enable(False)
    assert launches == (2 if own else 1)

"""Members of a batch that have stopped cost nothing: the preconditioner by modes
leaves their slices alone."""
import pytest
import torch

from paper_2410_22686_amd import Solver

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dim,nx,nt,kw", [
    (2, 127, 40, {}), (2, 127, 40, {"mass": "q1"}), (2, 255, 9, {}), (3, 15, 6, {}), (3, 127, 3, {}),
    (2, 127, 40, {"precond": "ideal", "precision": "mixed", "side": "flexible"}), (2, 31, 40, {}), (3, 63, 80, {})])
def test_slices_of_stopped_members_stay(dim, nx, nt, kw):
    """The part of the workspace that an apply writes for member 0 is what
    changes with member 0's input; a solve in which member 0 stops at once
    (b = 0) does not touch it."""
    print(f"stopped members {dim} {nx} {nt} {kw}", flush=True)
    s = Solver(dim, nx, nt, [1e-3, 1e-5], restart=2, maxit=4, rtol=1e-14, device=DEV, **kw)
    words = s.workspace[: s.workspace.numel() // 4 * 4].view(torch.int32)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    v = torch.randn(s.vec_shape, dtype=torch.float64, device=DEV, generator=gen)
    out = torch.empty_like(v)
    s.precond_apply(v, out=out)
    first = words.clone()
    v[0] = torch.randn(v[0].shape, dtype=torch.float64, device=DEV, generator=gen)
    s.precond_apply(v, out=out)
    before = words.clone()
    own = first != before
    assert int(own.sum()) >= (s.n * s.m if kw.get("precision") == "mixed" else 2 * s.n * s.m)
    b = v.clone()
    b[0] = 0
    s.solve(b)
    assert bool((words[own] == before[own]).all())

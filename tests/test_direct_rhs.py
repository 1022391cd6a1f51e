"""Stand-alone solves whose first product reads the caller's array instead of a
padded copy (direct_rhs in csrc/qn_api.cpp): one quasi-Newton step from U = 0
has R = -F exactly and goes through the padded tensor, so it gives the same
bits."""

import pytest
import torch

import synth
from paper_2502_03611_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,problem,shape,kw", [
    ("fp32", "cubic", (7, 9), {}),
    ("fp32", "system", (63, 200), {}),               # deep 32 x 32 tiles, padding in x and y
    ("fp32", "cubic", (255, 511), {}),
    ("fp32", "cubic", (33, 40, 45), {}),             # padding planes
    ("fp32", "system", (31, 65, 127), {}),
    ("fp64", "cubic", (100, 106), {}),               # no axis factors
    ("fp64", "cubic", (106, 63), {}),                # factored y between two dense passes' x
    ("fp64", "cubic", (41, 29, 65), {"discretization": "sem", "sem_order": 2}),
    ("fp64", "cubic", (255, 255), {"discretization": "sem", "sem_order": 4}),
    ("fp64", "cubic", (83, 48), {"boundary": "neumann", "lin": 1.0}),
])
def test_direct_solve_gives_the_step_from_zero(prec, problem, shape, kw):
    print(f"direct rhs {prec} {problem} {shape} {kw}", flush=True)
    ncomp = 2 if problem == "system" else 1
    f = torch.from_numpy(synth.random_field((ncomp,) + shape, 17, scale=20.0))
    pool = torch.empty(f.numel() + 1, dtype=torch.float64, device="cuda")
    F = pool[1:].view(f.shape)  # 8-byte but not 16-byte aligned
    F.copy_(f)
    s = Solver(shape, problem, beta=0.75, precision=prec, **kw)
    x = s.fdm_solve(F, 1.0, 0.75)
    u = torch.zeros_like(F)
    s.iterate(u, F, rtol=0.0, max_iter=1)
    assert torch.isfinite(x).all() and torch.equal(x, u)
    y = F.clone()
    s.fdm_solve(y, 1.0, 0.75, X=y)  # in place
    assert torch.equal(x, y)

"""Strip form of the folded mode products (csrc/qn_gemm_strip.h), taken by
grids of 2^20 or more values whose padded tiles waste a quarter of their work:
its contraction runs in the tile form's order, so its results are the tile
form's bits (which test_gpu_parity.py holds to the oracle)."""

import numpy as np
import pytest
import torch

import synth
from paper_2502_03611_amd import Solver
from paper_2502_03611_amd.batched import BatchedSolver

pytestmark = pytest.mark.gpu


def _pinned(s):
    """Pin the first dense launch to its own default tile: every dense launch
    of the solver then runs tiled."""
    s.set_tile(0, s.tiles()[0])
    return s


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("problem,shape,kw", [
    ("cubic", (100, 110, 106), {}),               # one block count per axis, even extents
    ("system", (75, 69, 137), {}),                # odd extents, a last strip of 4 lanes
    ("quasilinear", (35, 260, 133), {}),          # several block tiles along y
    ("cubic", (102, 63, 201), {}),                # FP64: y factored between two dense axes
    ("cubic", (63, 137, 138), {}),                # FP64: z factored (pass with the divide)
    ("cubic", (137, 138, 63), {}),                # FP64: x factored
    ("cubic", (200, 66, 90), {"boundary": "neumann", "lin": 1.0}),
    ("cubic", (133, 89, 101), {"discretization": "sem", "sem_order": 2}),
    ("cubic", (66, 66, 66), {}),                  # below 2^20 values: padding of 128 about 66
    ("system", (34, 37, 130), {}),
    ("cubic", (31, 82, 127), {}),                 # FP64: z and x factored
])
def test_strips_give_the_tiles_bits(problem, shape, kw, prec):
    if kw.get("discretization") == "sem":
        shape = tuple(2 * (n // 2) - 1 for n in shape)
    print(f"strips {problem} {shape} {prec} {kw}", flush=True)
    ncomp = 2 if problem == "system" else 1
    f = torch.from_numpy(synth.random_field((ncomp,) + shape, 81, scale=20.0)).cuda()
    beta = 0.0 if problem == "quasilinear" else 1.0
    a = Solver(shape, problem, beta=beta, precision=prec, **kw)
    b = _pinned(Solver(shape, problem, beta=beta, precision=prec, **kw))
    xa, xb = a.fdm_solve(f, 1.5, 0.25), b.fdm_solve(f, 1.5, 0.25)
    assert torch.isfinite(xa).all()
    ua, ub = torch.zeros_like(f), torch.zeros_like(f)
    sa, sb = a.iterate(ua, f, rtol=0.0, max_iter=2), b.iterate(ub, f, rtol=0.0, max_iter=2)
    b.autotune()  # drops the pinned tile
    xc = b.fdm_solve(f, 1.5, 0.25)
    # (factored axes beside them see the same inputs in both forms)
    assert torch.equal(xa, xb) and torch.equal(xa, xc)
    # the residual's partial sums are grouped by extents, the shift rules by them
    assert sa["iters"] == sb["iters"] == 2
    assert float((ua - ub).abs().max()) <= 1e-13 * float(ub.abs().max())


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-6)])
def test_batched_strips_match_the_single_solver(prec, tol):
    """A class of 70^2 instances large enough for strips (and one of 33^2 that
    is not): instances equal the single-problem solver's; stopped instances are
    left alone."""
    n, count = 70, 240
    sizes, ncomp = [n] * count + [33, 33], [1] * count + [1, 2]
    b = BatchedSolver(sizes, ncomp, precision=prec, beta_mode="midpoint")
    F, U = b.pool(), b.pool()
    fs = [synth.random_field((c, m, m), 900 + i, scale=30.0) for i, (m, c) in enumerate(zip(sizes, ncomp))]
    for i, f in enumerate(fs):
        b.fill(F, i, f)
    X = b.fdm_solve(F, 1.2, 0.4)
    status, res = b.iterate(U, F, rtol=1e-10, max_iter=60)
    assert status == 0
    for i in (0, 1, count // 2, count - 1, count, count + 1):
        s = Solver((sizes[i],) * 2, "system" if ncomp[i] == 2 else "cubic", beta_mode="midpoint", precision=prec)
        f = torch.from_numpy(fs[i]).cuda()
        x = s.fdm_solve(f, 1.2, 0.4)
        assert float((b.view(X, i) - x).norm() / x.norm()) <= tol
        u = torch.zeros_like(f)
        st = s.iterate(u, f, rtol=1e-10, max_iter=60)
        assert abs(st["iters"] - res[i]["iters"]) <= 1
        assert float((b.view(U, i) - u).norm() / u.norm()) <= max(tol * 1e-2, 1e-9)

"""Numerics of the solves per form of the mode products: strips, tiles, factored
transforms and their mixtures.  Which form a case takes is read from its launches
(launch_trace.py) and asserted, so that no case compares a form with itself."""

import os

import numpy as np
import pytest
import torch

import synth
from launch_trace import CLANG, forms, trace
from oracle import neumann as onm
from oracle import tensor as otensor
from paper_2502_03611_amd import QNError, Solver

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm host compiler")]


def _rows(shape, do=("solve",), **kw):
    return trace([dict(kw, shape=shape, do=list(do))])[0]


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("problem,shape,prec,sem,want", [
    ("cubic", (100, 110, 106), "fp64", 0, "SSSSSS"),
    ("system", (34, 37, 130), "fp64", 0, "SFFFS"),
    ("cubic", (102, 63, 201), "fp64", 0, "SFSSFS"),
    ("quasilinear", (138, 36, 262), "fp64", 0, "SSSSSS"),
    ("cubic", (133, 89, 101), "fp64", 2, "SSSSSS"),
    ("cubic", (66, 134, 229), "fp32", 0, "SSSSSS"),
    ("system", (96, 66, 31), "fp32", 0, "SSSSSS"),
    ("cubic", (275, 44, 175), "fp32", 0, "SSSSSS"),      # several block tiles along z
    ("cubic", (89, 133, 101), "fp32", 2, "SSSSSS"),
])
def test_strips_and_pinned_tiles_give_the_same_bits(problem, shape, prec, sem, want):
    print(f"strips {problem} {shape} {prec} {sem}", flush=True)
    kw = {"precision": prec, "problem": problem, "sem_order": sem}
    assert forms(_rows(shape, **kw)) == want
    assert forms(_rows(shape, (["pin", 0], "solve"), **kw)) == want.replace("S", "T")
    ncomp = 2 if problem == "system" else 1
    f = torch.from_numpy(synth.random_field((ncomp,) + shape, 83, scale=20.0)).cuda()
    opt = dict(beta=0.0 if problem == "quasilinear" else 1.0, precision=prec)
    if sem:
        opt.update(discretization="sem", sem_order=sem)
    a, b = Solver(shape, problem, **opt), Solver(shape, problem, **opt)
    first = torch.zeros_like(f)
    b.iterate(first, f, rtol=0.0, max_iter=1)  # the padding holds strip values from here on
    b.set_tile(0, b.tiles()[0])
    assert torch.equal(a.fdm_solve(f, 1.5, 0.25), b.fdm_solve(f, 1.5, 0.25))
    ua, ub = torch.zeros_like(f), torch.zeros_like(f)
    a.iterate(ua, f, rtol=0.0, max_iter=3)
    b.iterate(ub, f, rtol=0.0, max_iter=3)
    assert torch.isfinite(ua).all() and torch.equal(ua, ub)


@pytest.mark.parametrize("shape,bc,want", [
    ((40, 127, 127), "dirichlet", "FFTTFF"),             # padded layout: x and y factored, z tiled
    ((66, 127, 95), "dirichlet", "FFSSFF"),
    ((127, 100), "dirichlet", "TFT"),
    ((100, 255), "dirichlet", "FTTF"),
    ((61, 511), "dirichlet", "FFF"),                     # odd stages: 4 x 31, 4 x 29
    ((57, 95, 129), "dirichlet", "FFFFF"),
    ((61, 58, 58), "dirichlet", "TTFTT"),
    ((61, 61), "dirichlet", "TTTT"),
    ((61, 60, 63), "neumann", "TTTTTT"),
    ((129, 63, 99), "neumann", "FFFFF"),
    ((15, 799, 63), "dirichlet", "FFFFF"),               # stages of 40: y, x, z
    ((15, 31, 799), "dirichlet", "FFFFF"),
    ((799, 17, 31), "dirichlet", "FFFFF"),
    ((17, 2047), "dirichlet", "FFF"),                    # stages of 64
    ((2047, 17), "dirichlet", "FFF"),
    ((33, 801), "neumann", "FFF"),
])
def test_factored_and_mixed_solves_match_the_oracle(shape, bc, want):
    print(f"routes {shape} {bc}", flush=True)
    rows = _rows(shape, boundary=bc)
    assert forms(rows) == want
    long = {(15, 799, 63): "k_fast_lines<2, 0>", (15, 31, 799): "k_fast_rows<2, 0>", (17, 2047): "k_fast_rows<2, 1>",
            (799, 17, 31): "k_fast_lines<2, 1>", (2047, 17): "k_fast_lines<2, 1>"}.get(shape, "")
    assert any(long in r["name"] for r in rows)
    r = synth.random_field((1,) + shape, 73)
    s = Solver(shape, "cubic", beta=1.0, boundary=bc)
    x = s.fdm_solve(torch.from_numpy(r).cuda(), 1.0, 0.9)
    s.fdm_solve(torch.from_numpy(r).cuda(), 1.0, 0.9)  # second use of the workspace
    ref = (otensor.fdm_solve(r[0], 0.9, 1.0) if bc == "dirichlet"
           else onm.fdm_solve(r[0], onm.spacing(shape, 2.0), 0.9))
    assert _rel(x.cpu().numpy()[0], ref) <= 1e-12


def test_direct_solve_beside_a_factored_axis():
    """The tiled x product reads the caller's array, y is factored."""
    shape = (63, 106)
    rows = _rows(shape)
    assert forms(rows) == "TFT" and not any("pad_copy" in r["name"] for r in rows)
    F = torch.from_numpy(synth.random_field((1,) + shape, 17, scale=20.0)).cuda()
    s = Solver(shape, "cubic", beta=0.75)
    x = s.fdm_solve(F, 1.0, 0.75)
    u = torch.zeros_like(F)
    s.iterate(u, F, rtol=0.0, max_iter=1)
    assert torch.isfinite(x).all() and torch.equal(x, u)


@pytest.mark.parametrize("shape,sem", [((255, 255), 2), ((63, 255, 255), 4), ((66, 36), 0)])
def test_every_fp64_tile_of_dense_axes_gives_the_same_bits(shape, sem):
    """Blocks of 128 modes (the 128-wide tiles) on axes that do not factor."""
    print(f"tiles {shape} {sem}", flush=True)
    assert set(forms(_rows(shape, sem_order=sem))) == {"T"}
    opt = dict(discretization="sem", sem_order=sem) if sem else {}
    f = torch.from_numpy(synth.random_field((1,) + shape, 302, scale=20.0)).cuda()
    s = Solver(shape, "cubic", beta=1.0, **opt)
    want = s.fdm_solve(f, 1.5, 0.25)
    default = s.tiles()
    tried = 0
    for i, (kind, axis, _, _) in enumerate(default):
        base = kind & 3
        for flags in (0, 4, 32, 36, 64):
            for tm in (32, 64, 128):
                for tn in (32, 64, 128):
                    try:
                        s.set_tile(i, (base + flags, axis, tm, tn))
                    except QNError:
                        continue
                    tried += 1
                    assert torch.equal(s.fdm_solve(f, 1.5, 0.25), want), (i, base + flags, tm, tn)
        s.set_tile(i, default[i])
    assert tried > len(default)
    u, v = torch.zeros_like(f), torch.zeros_like(f)
    s.autotune()
    s.iterate(u, f, rtol=0.0, max_iter=3)
    Solver(shape, "cubic", beta=1.0, **opt).iterate(v, f, rtol=0.0, max_iter=3)
    assert torch.equal(u, v) and torch.equal(s.fdm_solve(f, 1.5, 0.25), want)


@pytest.mark.parametrize("shape,prec", [
    ((95, 1023), "fp64"), ((15, 1023, 31), "fp64"), ((511, 511, 31), "fp64"),  # more than 64 KB of LDS
    ((66, 134, 229), "fp32"), ((63, 106), "fp64"), ((63, 63, 63), "bf16x3"),
])
def test_a_first_solve_can_be_captured(shape, prec):
    """A solver's first solve, in a graph: the limits that its kernels need are
    raised outside the stream; replays on new inputs equal eager solves."""
    print(f"capture {shape} {prec}", flush=True)
    s, e = (Solver(shape, "cubic", beta=1.0, precision=prec) for _ in range(2))
    R = torch.from_numpy(synth.random_field((1,) + shape, 5)).cuda()
    X = torch.empty_like(R)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        s.fdm_solve(R, 1.1, 0.7, X=X)
    torch.cuda.synchronize()
    for i in range(3):
        R.mul_(0.5 - i)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(X, e.fdm_solve(R, 1.1, 0.7)), i
        torch.cuda.synchronize()

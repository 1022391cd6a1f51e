"""Factored eigen-transforms (csrc/qn_fast.hip).  On the CPU the stages and the
index rule are compiled for the host (fast_host.cpp) and compared with the
defining sine / cosine sums for every accepted interval count, with every
element access checked.  On the GPU the solves are held to the oracle where
the route changes: all axes factored, mixed with dense axes in every position,
odd and prime-free lengths, the longest stages, Neumann data, aliasing."""

import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import synth
from oracle import neumann as onm
from oracle import tensor as otensor
from paper_2502_03611_amd import Solver

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_03611_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_stages_match_the_defining_sums(tmp_path):
    """Errors are printed in units of 136 roundings of ||x||, the worst case of
    two stages of at most 64 terms and the twiddle."""
    exe = tmp_path / "fast_host"
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", CSRC,
                    os.path.join(HERE, "fast_host.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), "2", "520"], check=True, capture_output=True, text=True).stdout
    out += subprocess.run([str(exe), "1024", "1024"], check=True, capture_output=True, text=True).stdout
    out += subprocess.run([str(exe), "2048", "2048"], check=True, capture_output=True, text=True).stdout
    rows = [ln.split() for ln in out.splitlines()]
    assert len(rows) > 300
    seen = {int(r[0]) for r in rows}
    assert {32, 64, 128, 256, 512, 1024, 2048} <= seen  # nested grids of 2^k - 1 points
    for r in rows:
        assert float(r[4]) <= 1.0, r


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [
    (63, 63), (31, 17), (64, 79), (255, 127), (1023, 33),        # 2D; stages of 64, odd stages
    (63, 63, 63), (49, 59, 95), (15, 127, 99), (97, 64, 143),    # 3D, uneven factorisations
    (40, 63, 70), (63, 40, 70), (70, 40, 63), (40, 63, 63), (63, 40, 63), (63, 63, 40),  # mixed axes
])
def test_solve_matches_the_oracle(shape):
    print(f"factored solve {shape}", flush=True)
    r = synth.random_field((2,) + shape, 71)
    s = Solver(shape, "system", beta=1.0)
    R = torch.from_numpy(r).cuda()
    x = s.fdm_solve(R, 1.3, 0.7)
    s.fdm_solve(R, 1.3, 0.7, X=R)  # in place, second use of the workspace
    assert torch.equal(x, R)
    x = x.cpu().numpy()
    for c in range(2):
        assert _rel(x[c], otensor.fdm_solve(r[c], 0.7, 1.3)) <= 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(65, 129), (33, 17, 61), (33, 40, 65), (40, 31, 36), (101, 200)])
def test_neumann_solve_matches_the_oracle(shape):
    print(f"factored Neumann solve {shape}", flush=True)
    r = synth.random_field((1,) + shape, 72)
    s = Solver(shape, "cubic", beta=1.0, boundary="neumann")
    x = s.fdm_solve(torch.from_numpy(r).cuda(), 1.0, 0.9).cpu().numpy()
    assert _rel(x[0], onm.fdm_solve(r[0], onm.spacing(shape, 2.0), 0.9)) <= 1e-12

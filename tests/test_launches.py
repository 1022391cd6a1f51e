"""Launches read on the CPU (launch_trace.py): which form each mode product
takes and whether its launch is one that the device accepts."""

import os
import re
import shutil
import subprocess

import pytest

from launch_trace import CLANG, argument_bytes, forms, trace
from paper_2502_03611_amd import LIB_PATH

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm host compiler")

KB64, KB160 = 64 * 1024, 160 * 1024


def test_every_launch_fits_the_device():
    """Kernels of more than 64 KB of dynamic LDS have had their limit raised, each
    of them and on each device; the limits of a workgroup and of a launch hold;
    a factored pass keeps a workgroup's rows within its 32-bit byte offsets."""
    long_axes = [(511, 511, 511), (639, 33), (33, 639), (1023, 95), (2047, 17), (17, 2047), (15, 799, 63),
                 (799, 15, 31), (31, 15, 799), (399, 399, 399), (95, 95, 95), (255, 255)]
    calls = [{"shape": s, "do": ["solve", "iterate", ["device", 3], "solve", "iterate"]} for s in long_axes]
    calls += [{"shape": [n + 2 for n in s], "boundary": "neumann", "do": ["solve"]} for s in long_axes]
    # the widest gap between the components of a padded tensor
    calls += [{"shape": (65, 4093, 2047), "problem": "system", "do": ["solve", "iterate"]}]
    calls += [{"sizes": [255] * 8 + [1023] * 2 + [799, 63], "ncomp": [1] * 11 + [2], "precision": "fp64"}]
    raised, large = set(), set()
    for rows in trace(calls):
        for r in rows:
            if r["kind"] == "raise":
                raised.add((r["device"], r["name"]))
                continue
            assert 0 < r["block"] <= 1024 and r["lds"] <= KB160, r
            assert 0 < r["grid"] and r["grid"] * r["block"] < 2 ** 32, r
            assert 0 <= r["span"] < 2 ** 32 - 8 * 4096, r
            if r["lds"] > KB64:
                assert (r["device"], r["name"]) in raised, r
                large.add(r["name"])
    assert len(large) >= 4, large


@pytest.mark.parametrize("shape,launch,want", [
    ((102, 63, 201), 0, "TFTTFT"),   # x of a grid in strips with y factored: the dense axes run tiled
    ((102, 63, 201), 1, "SFSSFS"),   # its y launches are not issued
    ((102, 63, 201), 4, "SFSSFS"),
    ((63, 137, 138), 2, "SFFFS"),    # z, in a grid with y and z factored
    ((255, 255), 0, "FFF"),
    ((255, 255), 2, "FFF"),
    ((40, 127, 127), 3, "FFTTFF"),   # tiled beside factored axes already
])
def test_pinning_a_tile_moves_issued_launches_only(shape, launch, want):
    rows, = trace([{"shape": shape, "do": [["pin", launch], "solve"]}])
    assert forms(rows) == want
    rows, = trace([{"shape": shape, "do": [["pin", launch], "autotune", "solve"]}])
    before, = trace([{"shape": shape, "do": ["solve"]}])
    assert forms(rows) == forms(before)  # autotune drops it


@pytest.mark.parametrize("call", [
    {"shape": (100, 110, 106)}, {"shape": (66, 134, 229), "precision": "fp32"},
    {"shape": (34, 37, 130), "problem": "system"}, {"shape": (102, 63, 201)},
    {"shape": (133, 89, 101), "sem_order": 2},
])
def test_pinned_tiles_keep_the_residual_launch(call):
    """The residual's workgroups, and so the grouping of its partial sums, are the
    same beside strips and beside pinned tiles."""
    free, pinned = trace([dict(call, do=["iterate"]), dict(call, do=[["pin", 0], "iterate"])])
    assert "S" in forms(free) and "S" not in forms(pinned)

    def residual(rows):
        return [(r["name"], r["grid"], r["block"]) for r in rows if "residual" in r.get("name", "")]
    assert residual(free) and residual(free) == residual(pinned)


@pytest.mark.parametrize("shape,kw,want", [
    # prime-like stage lengths (chains of many multiply-adds) on grids of few tiles: dense
    ((61, 61), {}, "TTTT"), ((57, 57), {}, "TTTT"), ((45, 45), {}, "TTTT"), ((61, 58), {}, "TTTT"),
    ((59, 59), {"boundary": "neumann"}, "TTTT"), ((100, 123), {}, "TTTT"),
    ((57, 57, 57), {}, "TTTTTT"), ((64, 64, 64), {}, "TTTTTT"), ((61, 63, 63), {}, "TTTTTT"),
    ((61, 61, 58), {}, "TTTTTT"), ((127, 61, 61), {}, "TTTTTT"), ((64, 64, 64), {"problem": "system"}, "TTTTTT"),
    # short chains, longer axes or a second field: factored
    ((63, 63), {}, "FFF"), ((51, 51), {}, "FFF"), ((57, 63), {}, "FFF"), ((92, 92), {}, "FFF"), ((123, 123), {}, "FFF"),
    ((61, 511), {}, "FFF"), ((31, 17), {}, "FFF"), ((1023, 33), {}, "FFF"),
    ((63, 58), {}, "TFT"), ((127, 100), {}, "TFT"), ((100, 127), {}, "FTTF"), ((100, 255), {}, "FTTF"),
    ((63, 63, 63), {}, "FFFFF"), ((15, 15, 15), {}, "FFFFF"), ((51, 51, 51), {}, "FFFFF"),
    ((45, 45, 45), {"problem": "system"}, "FFFFF"),
    ((61, 58, 58), {}, "TTFTT"), ((31, 31, 123), {}, "FFFFF"), ((61, 127, 127), {}, "FFFFF"), ((61, 255, 255), {}, "FFFFF"),
])
def test_factored_axes_of_small_grids(shape, kw, want):
    rows, = trace([dict(kw, shape=shape, do=["solve"])])
    assert forms(rows) == want


def test_factored_classes_of_batches():
    for n, count, want in ((61, 300, "TTTT"), (61, 100, "FFF"), (57, 160, "TTTT"), (64, 112, "FFF"), (64, 113, "TTTT"),
                           (56, 1024, "TTTT"), (54, 1024, "FFF"), (63, 700, "FFF"), (127, 40, "FFF")):
        rows, = trace([{"sizes": [n] * count, "ncomp": [1] * count, "precision": "fp64"}])
        assert forms(rows) == want, (n, count)


@pytest.mark.parametrize("shape,problem,want", [
    # too little tile work, or too little padding, for strips to gain in FP32: tiles
    ((164, 31, 63), "cubic", "T"), ((60, 35, 66), "system", "T"), ((62, 108, 31), "system", "T"),
    ((217, 63, 31), "cubic", "T"), ((274, 63, 31), "cubic", "T"), ((63, 214, 72), "system", "T"),
    ((127, 198, 89), "cubic", "T"), ((31, 31, 31), "cubic", "T"),
    ((254, 254, 66), "cubic", "T"), ((127, 254, 66), "system", "T"), ((254, 200, 254), "cubic", "T"),
    ((196, 63, 254), "system", "T"), ((127, 313, 130), "cubic", "T"),
    ((66, 66, 66), "cubic", "S"), ((66, 36, 127), "cubic", "S"), ((96, 66, 31), "system", "S"),
    ((66, 109, 63), "system", "S"), ((44, 240, 153), "cubic", "S"), ((275, 44, 175), "cubic", "S"),
    ((150, 203, 176), "system", "S"), ((254, 130, 127), "system", "S"), ((280, 63, 277), "cubic", "S"),
    ((270, 270, 510), "cubic", "S"),
])
def test_strips_of_small_fp32_grids(shape, problem, want):
    rows, = trace([{"shape": shape, "problem": problem, "precision": "fp32", "do": ["solve"]}])
    assert forms(rows) == 6 * want


def test_strips_of_fp32_batches():
    for n, count, want in ((95, 132, "S"), (72, 231, "S"), (140, 61, "S"), (210, 136, "S"), (222, 121, "T")):
        rows, = trace([{"sizes": [n] * count, "ncomp": [1] * count, "precision": "fp32"}])
        assert forms(rows) == 4 * want, n


def test_launch_arguments_stay_small():
    """Launches bound by the host slow down with the bytes they copy."""
    dense, lines, rows = argument_bytes()
    assert dense <= 120 and lines <= 168 and rows <= 136


def test_mode_products_use_no_scratch_memory(tmp_path):
    """The library's own code objects: no mode product spills (a selection between
    two forms of the coefficients has made the strips do so)."""
    so = shutil.copy(LIB_PATH, tmp_path)
    tool = os.path.join(os.path.dirname(CLANG), "llvm-objdump")
    subprocess.run([tool, "--offloading", so], check=True, capture_output=True, cwd=tmp_path)
    seen = 0
    for f in tmp_path.glob("*gfx950"):
        notes = subprocess.run([os.path.join(os.path.dirname(CLANG), "llvm-readelf"), "--notes", str(f)],
                               check=True, capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", notes):
            if re.search(r"k_(strip|fold|fast|gemm)_", name):
                seen += 1
                assert size == "0", name
    assert seen > 200

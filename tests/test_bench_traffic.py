"""Counted HBM bytes are reported only while the sources that issue the kernel's
loads and stores are those that were counted."""

import os
import shutil

import pytest

bench = pytest.importorskip("bench")


@pytest.mark.parametrize("kernel,files", [
    ("k_fast_lines<0,0>", ("qn_fast.hip", "qn_fast.h")),
    ("k_residual<QUASILIN,double>", ("qn_pointwise.hip",)),
    ("k_gemm_left_bf<2,128,128,EPI_STORE,true,0>", ("qn_gemm_bf16.hip",)),
])
def test_counts_lapse_with_their_sources(kernel, files, tmp_path, monkeypatch):
    csrc = os.path.join("paper_2502_03611_amd", "csrc")
    shutil.copytree(os.path.join(bench.ROOT, csrc), tmp_path / csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.traffic_if_current(kernel, 511) > 1e9
    assert bench.traffic_if_current(kernel, 255) is None
    for name in files:
        path = tmp_path / csrc / name
        text = path.read_text()
        path.write_text(text + "\n")
        assert bench.traffic_if_current(kernel, 511) is None, name
        path.write_text(text)

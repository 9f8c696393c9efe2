"""LDS of the FP64 contraction's workgroups, checked on the host (no device):
two share a CU at every number of terms per class that two grids reach up to 2.5
times the band limit (64) and well past it, and the largest class fits at all."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "paper_1504_04653_amd/csrc/geometry.hpp"
using namespace sympix;
int main() {
    const int per_cu = 160 * 1024, granule = 1280, reduction = 256;   // LDS of a workgroup's vote beside the dynamic part
    for (int terms = 1; terms <= 128; ++terms) {
        const int one = (f64_lds_bytes(terms, f64_tile_rows(terms)) + reduction + granule - 1) / granule * granule;
        if (one * (terms <= 121 ? 2 : 1) > per_cu || f64_lds_bytes(terms, 64) + reduction > per_cu) {
            std::printf("terms %d: %d bytes\n", terms, one);
            return 1;
        }
    }
    std::puts("f64_lds OK");
}
"""


def test_two_workgroups_share_a_cu(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "check.cpp", str(tmp_path / "check")
    src.write_text(PROGRAM)
    res = subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", exe, str(src)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert "f64_lds OK" in res.stdout, res.stdout

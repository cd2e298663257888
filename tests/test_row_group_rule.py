"""When the many-right-hand-side products take row groups, on the CPU: csrc's
own header compiled with the host compiler.  Not for products too small to
be bound by their gathers (1100 of 64 values a compute unit in FP64, 2800 in
FP32), nor where rows share few columns,
nor where their copies would take more than 48 GiB."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2509_19267_amd", "csrc")
DRIVER = r"""
#include "repgroups.h"
extern "C" int takes(int64_t rep, int64_t cols, int64_t nnz, int64_t f64) {
  return rg::rep_rg_fits(rep, nnz, 256, f64 != 0) && rg::rep_rg_pays(cols, nnz);
}
"""


@pytest.mark.parametrize("rows,rep,per_row,share,f64,f32", [
    (65536, 64, 225, 0.30, 1, 1), (25600, 128, 25, 0.40, 1, 1),
    (12544, 64, 81, 0.33, 1, 1), (12544, 64, 25, 0.40, 1, 0),
    (6400, 64, 225, 0.30, 1, 1), (6400, 64, 81, 0.33, 1, 0),
    (6400, 65, 81, 0.33, 1, 1), (6400, 64, 25, 0.40, 0, 0),
    (1600, 256, 225, 0.30, 1, 1), (1600, 64, 25, 0.40, 0, 0),
    (100, 128, 81, 0.33, 0, 0), (500000, 64, 3, 0.50, 0, 0),
    (500000, 64, 5, 0.70, 0, 0), (10 ** 8, 64, 20, 0.30, 0, 0)])
def test_rule(tmp_path, rows, rep, per_row, share, f64, f32):
    (tmp_path / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC,
                    str(tmp_path / "d.cpp"), "-o", str(tmp_path / "d.so")],
                   check=True)
    so = ctypes.CDLL(str(tmp_path / "d.so"))
    so.takes.argtypes = [ctypes.c_int64] * 4
    nnz = rows * per_row
    assert so.takes(rep, int(share * nnz), nnz, 1) == f64
    assert so.takes(rep, int(share * nnz), nnz, 0) == f32

"""The chunk plan of the nonzero-balanced residual pass, on the CPU: csrc's own
header compiled with the host compiler.  Every row belongs to the chunk of its
first nonzero, and what a lane loads ahead lies inside the row pointers, also
where the last row runs through chunks that own no rows."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2509_19267_amd", "csrc")
DRIVER = r"""
#include "mergeplan.h"
extern "C" int64_t plan(const int64_t *rp, int64_t rows, int32_t *rs) {
  const rg::MergeRows p = rg::merge_rows(rp, rows);
  for (size_t c = 0; c < p.rs.size(); ++c) rs[c] = p.rs[c];
  return p.nchunk;
}
extern "C" int64_t longest(const int64_t *rp, int64_t rows) {
  return rg::merge_rows(rp, rows).maxlen;
}
extern "C" int64_t first_row(int64_t rs, int64_t re, int64_t lane, int64_t rows) {
  return rg::mp_first_row(rs, re, lane, rows);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC,
                    str(d / "d.cpp"), "-o", str(d / "d.so")], check=True)
    so = ctypes.CDLL(str(d / "d.so"))
    so.plan.restype = so.first_row.restype = so.longest.restype = ctypes.c_int64
    so.first_row.argtypes = [ctypes.c_int64] * 4
    return so


LENS = {"one_long_row": [1000], "last_row_over_a_boundary": [200, 100],
        "last_row_over_three_chunks": [3] * 509 + [700],
        "ends_on_a_boundary": [100, 412], "empty_rows_after": [5, 900, 0, 0],
        "empty": [0, 0, 0], "first_row_long": [800, 1, 0, 2],
        "many": list(np.random.default_rng(0).geometric(0.1, 3000)) + [257]}


@pytest.mark.parametrize("name", LENS)
def test_rows_loaded_ahead_exist(lib, name):
    rp = np.concatenate([[0], np.cumsum(LENS[name])]).astype(np.int64)
    rows, nnz = len(rp) - 1, int(rp[-1])
    rs = np.full(max(1, (nnz + 255) // 256) + 1, -1, np.int32)
    nchunk = lib.plan(ctypes.c_void_p(rp.ctypes.data), ctypes.c_int64(rows),
                      ctypes.c_void_p(rs.ctypes.data))
    assert lib.longest(ctypes.c_void_p(rp.ctypes.data),
                       ctypes.c_int64(rows)) == max(LENS[name])
    assert nchunk == len(rs) - 1 and rs[0] == 0 and rs[-1] == rows
    for c in range(nchunk):
        for r in range(rs[c], rs[c + 1]):
            assert rp[r] // 256 == c or (rp[r] == nnz and c == nchunk - 1)
        for lane in range(64):
            f = lib.first_row(int(rs[c]), int(rs[c + 1]), lane, rows)
            assert 0 <= f < rows                  # ptr[f], ptr[f + 1] exist
            if rs[c] + lane < rs[c + 1]:
                assert f == rs[c] + lane

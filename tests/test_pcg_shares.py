"""The persistent PCG's shares, on the CPU: csrc's own header compiled with
the host compiler.  A workgroup that takes part in the exchange of a step has a
row, because its published entries are what the others wait for before they
empty the buffer of the step before; the shares cover every row and every
entry of a buffer once."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2509_19267_amd", "csrc")
DRIVER = r"""
#include "pcgshare.h"
extern "C" void share(int c, int cap, int p, int *out) {
  const rg::PqShare s = rg::pq_share(c, cap, p);
  out[0] = s.rpw; out[1] = s.active; out[2] = s.per;
}
"""


@pytest.fixture(scope="module")
def share(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    (d / "d.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC,
                    str(d / "d.cpp"), "-o", str(d / "d.so")], check=True)
    so = ctypes.CDLL(str(d / "d.so"))

    def f(c, cap, p):
        out = (ctypes.c_int * 3)()
        so.share(c, cap, p, out)
        return tuple(out)
    return f


@pytest.mark.parametrize("cap", [1, 7, 8, 9, 257, 2050, 4000, 4096, 4500, 8192])
@pytest.mark.parametrize("p", [1, 3, 38, 250, 255, 256])
def test_every_exchanging_workgroup_has_rows(share, cap, p):
    for c in {0, 1, 2, p - 1, p, p + 1, cap // 3, cap - 1, cap}:
        if not 0 <= c <= cap:
            continue
        rpw, active, per = share(c, cap, p)
        assert 1 <= active <= p
        rows = [(w * rpw, min(c, (w + 1) * rpw)) for w in range(active)]
        if c > 0:
            assert all(a < b for a, b in rows), (c, cap, p)
        assert [i for a, b in rows for i in range(a, b)] == list(range(c))
        clears = [i for w in range(active)
                  for i in range(w * per, min(cap, (w + 1) * per))]
        assert clears == list(range(cap))

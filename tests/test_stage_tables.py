"""The twiddle table of the grouped kernels: the natural table's entries in the
order the stages read them, for every length those kernels take (lines up to
1024, convolutions of Bluestein's algorithm up to 8192).  A kernel of two or
more stages reads exactly sum (R_s - 1) Ns_s entries, so an empty or short
table would be read out of range."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_04896_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

WRAP = r"""
#include <algorithm>
#include "croft_internal.h"
extern "C" {
int t_stage_count(int n) { return (int)(croft::stage_twiddles_fp64(n).size() / 2); }
void t_stage(int n, double *out) { auto v = croft::stage_twiddles_fp64(n); std::copy(v.begin(), v.end(), out); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("stages")
    (d / "wrap.cpp").write_text(WRAP)
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "-fPIC", "-shared", f"-I{CSRC}", str(d / "wrap.cpp"),
                        os.path.join(CSRC, "croft_plan.cpp"), "-o", str(d / "lib.so")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    L = ctypes.CDLL(str(d / "lib.so"))
    L.t_stage.argtypes = [ctypes.c_int, np.ctypeslib.ndpointer(np.float64, flags="C_CONTIGUOUS")]
    return L


def radices(n):
    """The 5s, the 3s, then 8s with one 4, 16 or 2 for the remainder."""
    out = []
    for p in (5, 3):
        while n % p == 0:
            out.append(p)
            n //= p
    a = n.bit_length() - 1
    assert n == 1 << a
    if a % 3 == 1 and a > 1:
        return out + [8] * (a // 3 - 1) + [16]
    return out + [8] * (a // 3) + {0: [], 1: [2], 2: [4]}[a % 3]


@pytest.mark.parametrize("n", [16, 18, 32, 50, 243, 360, 512, 720, 960, 1000, 1024, 2048, 4096, 8192])
def test_stage_table_is_complete_and_in_order(lib, n):
    want, ns = [], 1
    for s, r in enumerate(radices(n)):
        if s:
            want += [np.exp(-2j * np.pi * (q * k) / (ns * r)) for q in range(1, r) for k in range(ns)]
        ns *= r
    assert ns == n and lib.t_stage_count(n) == len(want)
    if not want:
        return
    got = np.empty(2 * len(want))
    lib.t_stage(n, got)
    # a few ulp of the unit circle for numpy's own argument rounding
    np.testing.assert_allclose(got[0::2] + 1j * got[1::2], want, rtol=0, atol=4e-15)

"""The candidates the autotuner times, against those a wisdom line can name: the
numbers of a length need not be consecutive (a contiguous length whose only
alternative is the streaming tile has 0 and 3)."""
import ctypes
import os
import shutil
import subprocess

import pytest

import paper_2002_04896_amd as croft
from test_abi_cpu import parse_describe

PKG = os.path.dirname(os.path.abspath(croft.__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

WRAP = r"""
#include <algorithm>
#include "croft_internal.h"
extern "C" int t_candidates(int n, int kind, int dtype, int *out) {
    const auto c = croft::kernel_candidates(n, kind, dtype);
    std::copy(c.begin(), c.end(), out);
    return (int)c.size();
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("candidates")
    (d / "wrap.cpp").write_text(WRAP)
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "-fPIC", "-shared", f"-I{PKG}/csrc", str(d / "wrap.cpp"),
                        f"-L{PKG}", "-lcroft", f"-Wl,-rpath,{PKG}", "-o", str(d / "lib.so")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return ctypes.CDLL(str(d / "lib.so"))


# (dims, kind): whole tiles and whole 128-byte lines in every storage, so that
# no candidate gives way to a plainer twin
@pytest.mark.parametrize("n,kind", [(400, 0), (576, 0), (640, 0), (960, 0), (512, 0), (96, 1), (384, 1), (512, 1), (1024, 1)])
@pytest.mark.parametrize("dtype", range(4))
def test_the_autotuner_visits_every_candidate(lib, tmp_path, monkeypatch, n, kind, dtype):
    w = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    dims = (n, 64, 2) if kind == 0 else (64, n, 2)
    named = []
    for cand in range(40):
        w.write_text(f"{n} {kind} {dtype} {cand} 0\n")
        if parse_describe(croft.croft_plan_describe(*dims, dtype))[1][kind]["candidate"] == str(cand):
            named.append(cand)
    out = (ctypes.c_int * 64)()
    assert list(out[:lib.t_candidates(n, kind, dtype, out)]) == named

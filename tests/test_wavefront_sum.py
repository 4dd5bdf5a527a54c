"""The fused multiply pass's energy sum over a wavefront, run on the CPU with the
lanes that a block does not have holding NaN: for every block size the first
lane's sum takes each existing lane once and none of the others."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_04896_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include "croft_internal.h"

int main() {
    int bad = 0;
    for (int block = 1; block <= 1024; ++block)
        for (int base = 0; base < block; base += 64) {
            double v[64], want = 0;
            for (int l = 0; l < 64; ++l) {
                const bool exists = base + l < block;
                v[l] = exists ? (double)(1 + (base + l) % 97) : std::nan("");
                if (exists) want += v[l];
            }
            for (int h = 32; h > 0; h /= 2) {
                double w[64];
                for (int l = 0; l < 64; ++l)
                    w[l] = v[l] + (croft::butterfly_peer_exists(block, base + l, h) ? v[l ^ h] : 0.0);
                for (int l = 0; l < 64; ++l) v[l] = w[l];
            }
            if (!(v[0] == want)) ++bad, std::printf("block %d wavefront %d: %g, not %g\n", block, base / 64, v[0], want);
        }
    return bad != 0;
}
"""


def test_lanes_past_the_end_of_the_block_add_nothing(tmp_path):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    (tmp_path / "t.cpp").write_text(PROGRAM)
    exe = tmp_path / "t"
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", f"-I{CSRC}", str(tmp_path / "t.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]

"""What the autotuner picks where the candidates are far apart."""
import pytest

import paper_2002_04896_amd as croft

pytestmark = pytest.mark.gpu

C64, F16 = croft.CROFT_C64, croft.CROFT_C16F


def recorded(tmp_path, monkeypatch, dims, dtype):
    w = tmp_path / "w.txt"
    w.write_text("")
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    croft.croft_plan_destroy(croft.croft_plan_create_ex(*dims, dtype, croft.CROFT_FORWARD, croft.CROFT_MEASURE, 1))
    return {(int(l[0]), int(l[1])): int(l[3]) for l in (l.split() for l in w.read_text().splitlines())}


def test_one_kernel_for_both_directions_is_not_taken_for_twice_as_fast(tmp_path, monkeypatch):
    # few tiles of 960 points: 8.8 us on the stage-by-stage tile (1, a kernel per
    # direction) against 13.8 on the grouped stages (0, one kernel for both)
    assert recorded(tmp_path, monkeypatch, (64, 960, 4), C64)[960, 1] == 1

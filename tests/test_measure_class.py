"""A choice that the autotuner made serves the passes it was timed on: grids of
the same size to a factor of two with rows of the same alignment, in the same
place of the plan (dry runs on the CPU; the autotuner itself on the GPU)."""
import pytest

import paper_2002_04896_amd as croft
from test_abi_cpu import parse_describe

C64, C128 = croft.CROFT_C64, croft.CROFT_C128


def line(n, kind, dtype, mib, partial, first, choice, axis=None):
    """The file's line for a class: the third number is dtype + 4 class."""
    step = max(0, (mib - 1).bit_length())
    cls = 1 + partial + 2 * first + 4 * step
    return f"{n} {kind} {dtype + 4 * cls} {choice[0]} {choice[1]}" + (f" {axis}" if axis else "") + "\n"


def choices(describe, *args):
    return {p["axis"]: (p["candidate"], p["waves"]) for p in parse_describe(describe(*args))[1]}


@pytest.mark.parametrize("text,inside,outside", [
    # 180 x 256 x 64 rows of 96 (whole) in 16 .. 32 MiB against 97 (partial) and other sizes
    (line(180, 1, C64, 32, 0, 0, (1, 3), 1), [(96, 180, 200), (192, 180, 100)],
     [(97, 180, 200), (96, 180, 32), (96, 180, 500)]),
    (line(180, 1, C64, 32, 1, 0, (0, 3), 1), [(97, 180, 200)], [(96, 180, 200), (97, 180, 20)]),
    (line(300, 0, C64, 64, 0, 0, (0, 3)), [(300, 128, 200)], [(300, 128, 300), (300, 64, 30)])])
def test_a_measured_line_serves_its_class(tmp_path, monkeypatch, text, inside, outside):
    w = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    axis = "x" if text.split()[1] == "0" else "y"
    want = tuple(text.split()[3:5])
    for dims, hit in [(d, True) for d in inside] + [(d, False) for d in outside]:
        w.write_text("")
        before = choices(croft.croft_plan_describe, *dims)[axis]
        assert before != want
        w.write_text(text)
        assert choices(croft.croft_plan_describe, *dims)[axis] == (want if hit else before), dims


def test_a_measured_first_z_pass_is_not_the_last_one(tmp_path, monkeypatch):
    w = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    dims = (256, 128, 256)  # 129 x 128 elements a row of z: whole lines, 32.25 MiB
    w.write_text(line(256, 1, C64, 33, 0, 1, (4, 3), 2))
    assert choices(croft.croft_plan_describe_real, *dims, C64, 1)["z"] == ("4", "3")
    assert choices(croft.croft_plan_describe_real, *dims, C64, -1)["z"] != ("4", "3")


def test_a_plain_line_serves_every_class_but_after_a_line_of_the_class(tmp_path, monkeypatch):
    w = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    w.write_text(line(180, 1, C64, 32, 0, 0, (1, 3), 1) + "180 1 0 0 5 1\n")
    assert choices(croft.croft_plan_describe, 96, 180, 200)["y"] == ("1", "3")
    assert choices(croft.croft_plan_describe, 97, 180, 200)["y"] == ("0", "5")


@pytest.mark.gpu
def test_measuring_one_grid_leaves_the_other_classes_alone(tmp_path, monkeypatch):
    w = tmp_path / "w.txt"
    w.write_text("")
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    others = [(97, 180, 64), (96, 180, 20), (96, 180, 300)]
    before = [choices(croft.croft_plan_describe, *d) for d in others]
    croft.croft_plan_destroy(croft.croft_plan_create_ex(96, 180, 64, C64, -1, croft.CROFT_MEASURE, 1))
    assert [choices(croft.croft_plan_describe, *d) for d in others] == before
    recorded = [l.split() for l in w.read_text().splitlines() if l.startswith("180 1 ")]
    assert len(recorded) == 1 and choices(croft.croft_plan_describe, 96, 180, 64)["y"] == tuple(recorded[0][3:5])
    # and this process's own memory of it, without the file
    monkeypatch.setenv("CROFT_WISDOM", str(tmp_path / "none.txt"))
    assert [choices(croft.croft_plan_describe, *d)["y"] for d in others] == [b["y"] for b in before]

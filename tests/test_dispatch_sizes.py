"""The planner's choices by size where one configuration does not fit all (dry
runs, no GPU): which side of each line a pass falls on."""
import pytest

import paper_2002_04896_amd as croft
from test_abi_cpu import parse_describe

C64, C128, F16, BF16 = croft.CROFT_C64, croft.CROFT_C128, croft.CROFT_C16F, croft.CROFT_C16B


@pytest.fixture(autouse=True)
def no_wisdom(tmp_path, monkeypatch):
    monkeypatch.setenv("CROFT_WISDOM", str(tmp_path / "none.txt"))


def one(axis, *args):
    return [p for p in parse_describe(croft.croft_plan_describe(*args))[1] if p["axis"] == axis][0]


@pytest.mark.parametrize("axis,dims,dt,waves", [
    ("x", (2048, 32, 300), C64, "1"), ("x", (4096, 8, 2), F16, "1"), ("y", (64, 2048, 300), BF16, "1"),
    ("z", (64, 64, 4096), C128, "1"), ("x", (720, 32, 64), C128, "1"), ("x", (300, 32, 64), C128, "0"),
    # strided, up to 64 MiB and beyond
    ("y", (64, 120, 1024), C64, "1"), ("y", (64, 120, 1200), C64, "0"), ("z", (64, 480, 120), C128, "1"),
    ("y", (64, 16, 512), F16, "1"), ("y", (45, 60, 64), C64, "0"), ("y", (45, 64, 64), C128, "0")])
def test_grid_size_where_nothing_was_measured(axis, dims, dt, waves):
    assert one(axis, *dims, dt)["waves"] == waves


@pytest.mark.parametrize("m,dt,forward,backward", [(200, C128, "0", "0"), (480, C64, "1", "1"),
                                                   (720, C64, "0", "1"), (576, C128, "1", "0"), (2048, C64, "1", "1")])
def test_real_x_grid_size(m, dt, forward, backward):
    got = [[p for p in parse_describe(croft.croft_plan_describe_real(2 * m, 8, 8, dt, d))[1] if p["kind"] == "real"][0]
           for d in (-1, 1)]
    assert (got[0]["waves"], got[1]["waves"]) == (forward, backward)


@pytest.mark.parametrize("dims,cand", [((512, 200, 160), "3"), ((512, 128, 100), "1"), ((512, 160, 128), "1"),
                                       ((512, 256, 128), "1"), ((640, 160, 144), "3"), ((512, 200, 120), "1")])
def test_complex128_streaming_first_pass(dims, cand):
    # beyond 192 MiB on uneven grids, beyond 256 MiB on powers of two
    assert one("x", *dims, C128)["candidate"] == cand


@pytest.mark.parametrize("axis,dims,dt,choice", [
    ("y", (64, 256, 32), C64, ("1", "0")), ("y", (64, 256, 33), C64, ("2", "0")),
    ("z", (64, 32, 256), C64, ("1", "0")), ("z", (64, 33, 256), C64, ("5", "0")),
    ("y", (64, 256, 64), C128, ("0", "1")), ("y", (64, 256, 65), C128, ("4", "0")),
    ("y", (384, 384, 384), C64, ("2", "1")), ("z", (384, 384, 384), C64, ("2", "1")),
    ("y", (384, 384, 96), C64, ("8", "0")), ("y", (383, 384, 384), C64, ("8", "0")),
    ("y", (512, 512, 64), C128, ("4", "2")), ("y", (512, 512, 512), C128, ("4", "0")),
    ("y", (512, 512, 32), C128, ("4", "0"))])
def test_choices_by_size(axis, dims, dt, choice):
    p = one(axis, *dims, dt)
    assert (p["candidate"], p["waves"]) == choice

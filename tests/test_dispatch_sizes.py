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
    ("z", (128, 64, 256), C64, ("5", "0")), ("z", (128, 72, 256), C64, ("1", "0")), ("z", (256, 62, 256), C64, ("1", "0")),
    ("z", (128, 128, 256), C64, ("5", "0")), ("z", (128, 80, 128), C128, ("5", "0")), ("z", (128, 88, 128), C128, ("2", "0")),
    ("z", (256, 58, 128), C128, ("2", "0")), ("z", (256, 60, 128), C128, ("5", "0")), ("z", (128, 44, 256), C128, ("6", "0")),
    ("z", (128, 128, 128), C128, ("5", "0")), ("y", (512, 256, 300), C128, ("5", "0")), ("y", (512, 256, 100), C128, ("4", "0")),
    ("y", (512, 256, 256), C128, ("4", "0")), ("y", (384, 384, 384), C64, ("2", "1")), ("z", (384, 384, 384), C64, ("2", "1")),
    ("y", (384, 384, 96), C64, ("8", "0")), ("y", (383, 384, 384), C64, ("8", "0")),
    ("y", (512, 512, 64), C128, ("4", "2")), ("y", (512, 512, 512), C128, ("4", "0")),
    ("y", (512, 512, 32), C128, ("4", "0"))])
def test_choices_by_size(axis, dims, dt, choice):
    p = one(axis, *dims, dt)
    assert (p["candidate"], p["waves"]) == choice


@pytest.mark.parametrize("dims,cand", [((512, 400, 128), "1"), ((512, 300, 128), "2"), ((128, 128, 128), "2")])
def test_fused_complex128_128_by_alignment(dims, cand):
    p = [q for q in parse_describe(croft.croft_plan_describe_convolution(*dims, C128))[1] if q["kind"] == "fused"]
    assert p[0]["candidate"] == cand


# the last launch that takes the stage-by-stage tile and the first that takes
# the grouped stages (candidate 0), in whole rows and in partial ones
@pytest.mark.parametrize("n,dt,few,many", [
    (288, C64, (64, 64), (64, 65)), (960, C64, (64, 32), (64, 33)), (960, C64, (45, 42), (45, 43)),
    (320, C128, (64, 32), (64, 33)), (768, C128, (64, 64), (64, 65)), (384, C128, (45, 42), (45, 43)),
    (64, F16, (64, 2048), (64, 2049)), (64, BF16, (45, 128), (45, 129)), (100, F16, (64, 128), (64, 129)),
    (320, BF16, (64, 128), (64, 129)), (972, F16, (64, 16), (64, 17))])
def test_launches_of_few_tiles_run_stage_by_stage(n, dt, few, many):
    assert one("y", few[0], n, few[1], dt)["candidate"] == "1"
    assert one("y", many[0], n, many[1], dt)["candidate"] == "0"


@pytest.mark.parametrize("axis,dims,dt,choice", [
    ("y", (64, 160, 4096), F16, ("1", "1")), ("z", (512, 512, 128), BF16, ("1", "4")), ("y", (64, 128, 2048), F16, ("1", "1")),
    ("y", (64, 128, 2049), F16, ("6", "0")), ("y", (45, 128, 8), F16, ("6", "0")), ("y", (64, 256, 256), BF16, ("0", "0")),
    ("y", (64, 256, 257), BF16, ("6", "0")), ("y", (45, 160, 200), BF16, ("0", None)), ("z", (64, 800, 384), C128, ("1", "1")),
    ("y", (64, 480, 136), C128, ("1", "0")), ("y", (64, 480, 140), C128, ("0", None)), ("y", (64, 480, 640), C128, ("1", "0")),
    ("z", (64, 640, 480), C128, ("0", None)), ("x", (288, 32, 1820), F16, ("1", "0")),
    ("x", (288, 32, 1821), F16, ("0", "0")), ("x", (640, 64, 4096), BF16, ("1", "1")), ("x", (640, 320, 400), C64, ("3", "0"))])
def test_where_the_stage_by_stage_tiles_stay(axis, dims, dt, choice):
    p = one(axis, *dims, dt)
    assert p["candidate"] == choice[0] and choice[1] in (None, p["waves"])


@pytest.mark.parametrize("axis,few,many,dt,T", [
    ("y", (64, 1021, 8), (64, 1021, 9), C64, ("256", "128")), ("x", (1021, 32, 16), (1021, 19, 27), F16, ("256", "128")),
    ("y", (64, 2039, 8), (64, 2039, 9), BF16, ("256", "128")), ("z", (64, 32, 211), (64, 33, 211), C64, ("64", "32")),
    ("y", (64, 97, 64), (64, 97, 65), C128, ("32", "16")), ("y", (64, 509, 2), (64, 509, 640), C64, ("64", "64"))])
def test_bluestein_spreads_few_lines_over_more_threads(axis, few, many, dt, T):
    got = [one(axis, *d, dt) for d in (few, many)]
    assert all(p["kernel"] == "bluestein" for p in got) and tuple(p["T"] for p in got) == T

"""The planner's built-in choices by size and alignment (dry runs, no GPU)."""
import pytest

import paper_2002_04896_amd as croft
from test_abi_cpu import parse_describe

C64, C128 = croft.CROFT_C64, croft.CROFT_C128


@pytest.fixture(autouse=True)
def no_wisdom(tmp_path, monkeypatch):
    monkeypatch.setenv("CROFT_WISDOM", str(tmp_path / "none.txt"))


def passes(*args):
    return parse_describe(croft.croft_plan_describe(*args))[1]


@pytest.mark.parametrize("dims,dt,cand", [((512, 512, 512), C64, "3"), ((512, 256, 257), C64, "3"),
                                          ((512, 256, 256), C64, "1"), ((512, 96, 100), C64, "1"),
                                          ((640, 96, 100), C64, "0"), ((512, 512, 64), C128, "1"),
                                          ((512, 512, 65), C128, "3")])
def test_streaming_first_pass_only_beyond_the_cache(dims, dt, cand):
    # above 256 MiB of grid; at or below it the padded tile, or the default
    # where there is none
    assert passes(*dims, dt)[0]["candidate"] == cand


@pytest.mark.parametrize("nx,dt,grouped", [(48, C64, False), (45, C64, True), (100, C64, True), (8, C128, False),
                                           (9, C128, True)])
def test_partial_lines_take_the_grouped_stages(nx, dt, grouped):
    # rows of nx elements: whole 128-byte lines or not
    for n in (60, 128):
        p = passes(nx, n, 4, dt)[1]
        assert (p["candidate"] == {60: "1", 128: "6"}[n]) == grouped, p


def test_a_wisdom_line_comes_before_the_rules(tmp_path, monkeypatch):
    w = tmp_path / "w.txt"
    w.write_text("512 0 0 3 0\n60 1 0 0 2\n")
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    assert passes(512, 96, 100)[0]["candidate"] == "3"
    assert passes(45, 60, 4)[1]["candidate"] == "0"


@pytest.mark.parametrize("dims,L", [((192, 180, 360), "8"), ((256, 256, 360), "16"), ((512, 250, 512), "16"),
                                    ((192, 150, 512), "8"), ((192, 180, 200), "16"), ((192, 180, 625), "8")])
def test_fused_tiles(dims, L):
    p = [q for q in parse_describe(croft.croft_plan_describe_convolution(*dims))[1] if q["kind"] == "fused"]
    assert p[0]["L"] == L


@pytest.mark.parametrize("nz,dt,forward,backward", [(256, C64, "5", "2"), (512, C64, "18", "15"),
                                                    (1024, C64, "7", "8"), (256, C128, "5", "4"),
                                                    (60, C64, None, None)])
def test_a_z_pass_that_others_follow_takes_the_y_choice(tmp_path, monkeypatch, nz, dt, forward, backward):
    # a forward real plan ends with z, a backward one starts with it; lengths
    # with no choice by axis take the same configuration in both
    def z(d):
        return [p for p in parse_describe(croft.croft_plan_describe_real(256, 256, nz, dt, d))[1] if p["axis"] == "z"][0]
    f, b = z(-1)["candidate"], z(1)["candidate"]
    assert (f, b) == (forward, backward) if forward else f == b
    # a measured choice of the y axis stays with y
    w = tmp_path / "w.txt"
    w.write_text(f"{nz} 1 {dt} 1 0 1\n")
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    assert z(1)["candidate"] == b

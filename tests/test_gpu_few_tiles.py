"""Lengths with a stage-by-stage tile beside the grouped stages, the planner
taking one or the other by size: both, named through a wisdom file, against the
runtime-radix kernel's bits, on whole rows, on partial ones and (16-bit
storage) on contiguous lines."""
import pytest
import torch

import paper_2002_04896_amd as croft

pytestmark = pytest.mark.gpu

C64, C128, F16, BF16 = croft.CROFT_C64, croft.CROFT_C128, croft.CROFT_C16F, croft.CROFT_C16B
FWD, BWD, GENERIC = croft.CROFT_FORWARD, croft.CROFT_BACKWARD, croft.CROFT_FORCE_GENERIC

STRIDED = [(n, C64) for n in (288, 320, 360, 400, 480, 576, 640, 720, 768, 960)] + \
          [(n, C128) for n in (320, 360, 384, 400, 480, 576, 640, 768, 960)] + \
          [(n, d) for d in (F16, BF16) for n in (32, 60, 64, 80, 96, 100, 120, 160, 192, 200, 288, 320, 360, 384, 400, 480,
                                                 576, 640, 720, 768, 900, 960, 972)]
LINES = [(n, d) for d in (F16, BF16) for n in (96, 100, 160, 192, 200, 288, 320, 360, 384, 480, 640, 768, 960)]


def run(nx, ny, nz, dtype, direction, flags):
    g = torch.Generator(device="cuda").manual_seed(71)
    real = {C64: torch.float32, C128: torch.float64, F16: torch.float16, BF16: torch.bfloat16}[dtype]
    x = torch.randn((nz, ny, nx, 2), generator=g, device="cuda", dtype=torch.float32).to(real).contiguous()
    out, exps = torch.full_like(x, float("nan")), None
    plan = croft.croft_plan_create_ex(nx, ny, nz, dtype, direction, flags, 1)
    try:
        if dtype in (C64, C128):
            croft.croft_execute(plan, x, out)
        else:
            ie = torch.randint(-9, 10, (nz, ny), generator=g, device="cuda", dtype=torch.int8)
            exps = torch.full((ny, nx), 99, device="cuda", dtype=torch.int8)
            croft.croft_execute_scaled(plan, x, ie, out, exps)
        torch.cuda.synchronize()
    finally:
        croft.croft_plan_destroy(plan)
    return out.view(torch.int16 if exps is not None else torch.int32 if dtype == C64 else torch.int64), exps


def check(tmp_path, monkeypatch, n, kind, dtype, dims):
    w = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(w))
    for direction in (FWD, BWD):
        w.write_text("")
        want, we = run(*dims, dtype, direction, GENERIC)
        for cand in (0, 1):
            w.write_text(f"{n} {kind} {dtype} {cand} {cand}\n")
            got, ge = run(*dims, dtype, direction, 0)
            assert torch.equal(got, want), (direction, cand)
            assert we is None or torch.equal(ge, we), (direction, cand)


@pytest.mark.parametrize("nx", [32, 45])
@pytest.mark.parametrize("n,dtype", STRIDED)
def test_strided_tiles_agree(tmp_path, monkeypatch, n, dtype, nx):
    check(tmp_path, monkeypatch, n, 1, dtype, (nx, n, 3))


@pytest.mark.parametrize("n,dtype", LINES)
def test_contiguous_tiles_agree(tmp_path, monkeypatch, n, dtype):
    check(tmp_path, monkeypatch, n, 0, dtype, (n, 7, 3))

"""The passes that run several stages per register group, at the lengths
where their shapes change: one group, two and three, with and without the
padded or split exchange, first and last length of each range, and tiles that
are not whole.  The grouped stages are the runtime-radix kernel's, butterfly
for butterfly, so the outputs must be its bits; the oracle comparison keeps
the suite's tolerances (unit roundoff times a few stages, far below them)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_04896_amd as croft
from paper_2002_04896_amd import synth
from gpu_helpers import HALF_KIND, TOL, run_fft, run_half
from test_gpu_conv import run_conv, unfused

pytestmark = pytest.mark.gpu

C64, C128, F16, BF16 = croft.CROFT_C64, croft.CROFT_C128, croft.CROFT_C16F, croft.CROFT_C16B
FWD, BWD = croft.CROFT_FORWARD, croft.CROFT_BACKWARD
GENERIC = croft.CROFT_FORCE_GENERIC

# (nz, ny, nx); strided axes beside rows that are not a multiple of a tile
SHAPES = [(18, 243, 5), (1000, 3, 17), (972, 2, 3), (960, 1, 33), (3, 900, 9), (2, 810, 4), (720, 2, 5), (25, 54, 75),
          (2, 3, 1000), (3, 2, 486), (2, 2, 720), (384, 3, 6), (5, 480, 7), (128, 4, 9), (256, 2, 11), (81, 3, 972)]


@pytest.mark.parametrize("direction", [FWD, BWD], ids=["fwd", "bwd"])
@pytest.mark.parametrize("dtype", [C64, C128], ids=["c64", "c128"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_matches_oracle_and_runtime_radix_bits(shape, dtype, direction):
    x = synth.normal_c(shape, seed=51)
    seen, y, after = run_fft(x, dtype, direction)
    assert oracle.rel_l2(y, oracle.dft3d(seen, direction)) <= TOL[dtype]
    np.testing.assert_array_equal(after, seen)
    _, g, _ = run_fft(x, dtype, direction, flags=GENERIC)
    np.testing.assert_array_equal(y, g)


@pytest.mark.parametrize("dtype", [F16, BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_half_storage_matches_oracle_and_runtime_radix_bits(shape, dtype):
    kind = HALF_KIND[dtype]
    nz, ny, nx = shape
    data, e = synth.quantize_half(synth.normal_c(shape, seed=52), kind)
    for direction in (FWD, BWD):
        out, oe = run_half(data, e, dtype, direction)
        exact = oracle.dft3d(oracle.decode_half(data, e, kind, 0), direction)
        assert oracle.rel_l2(oracle.decode_half(out, oe, kind, 2), exact) <= TOL[dtype]
        d_in = torch.from_numpy(np.ascontiguousarray(data.view(np.int16))).cuda()
        d_out, d_e = torch.empty_like(d_in), torch.empty((ny, nx), dtype=torch.int8, device="cuda")
        plan = croft.croft_plan_create_ex(nx, ny, nz, dtype, direction, GENERIC, 1)
        croft.croft_execute_scaled(plan, d_in, torch.from_numpy(e).cuda(), d_out, d_e)
        torch.cuda.synchronize()
        croft.croft_plan_destroy(plan)
        np.testing.assert_array_equal(d_out.cpu().numpy().view(np.uint16), out)
        np.testing.assert_array_equal(d_e.cpu().numpy(), oe)


def test_one_block_per_tile_whatever_the_wisdom_says(tmp_path, monkeypatch):
    """These kernels do not loop over tiles: a persistent grid named in a
    wisdom file must not leave tiles undone.  2400 tiles of 243-point lines,
    more than one wave of resident blocks."""
    wisdom = tmp_path / "w.txt"
    monkeypatch.setenv("CROFT_WISDOM", str(wisdom))
    x = torch.randn((600, 243, 64), dtype=torch.complex64, device="cuda")
    outs = []
    for line, flags in (("", GENERIC), ("243 1 0 0 1 1\n", 0)):
        wisdom.write_text(line)
        plan = croft.croft_plan_create_ex(64, 243, 600, C64, FWD, flags, 1)
        outs.append(torch.full_like(x, complex(float("nan"), 0)))
        croft.croft_execute(plan, x, outs[-1])
        torch.cuda.synchronize()
        croft.croft_plan_destroy(plan)
    assert torch.equal(*outs)


# prime lengths for the convolution lengths 32 .. 4096 in 16-bit storage, on
# the contiguous and the strided axes (n close to m / 2 and close to m / 4)
@pytest.mark.parametrize("dtype", [F16, BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", [(11, 31, 17), (37, 3, 61), (5, 127, 67), (131, 2, 251), (3, 509, 7), (2, 257, 1021),
                                   (1031, 3, 2), (2, 2, 2039), (1, 4093, 2), (1, 2, 4091)], ids=str)
def test_bluestein_half_storage(shape, dtype):
    kind = HALF_KIND[dtype]
    data, e = synth.quantize_half(synth.normal_c(shape, seed=53), kind)
    for direction in (FWD, BWD):
        out, oe = run_half(data, e, dtype, direction)
        exact = oracle.dft3d(oracle.decode_half(data, e, kind, 0), direction)
        assert oracle.rel_l2(oracle.decode_half(out, oe, kind, 2), exact) <= TOL[dtype]


@pytest.mark.parametrize("direction", [FWD, BWD], ids=["fwd", "bwd"])
def test_longest_strided_convolution(direction):
    x = synth.normal_c((2, 4093, 3), seed=54)
    seen, y, _ = run_fft(x, C64, direction)
    assert oracle.rel_l2(y, oracle.dft3d(seen, direction)) <= TOL[C64]


# (nx, ny, nz) with the fused axis nz: stage-by-stage and grouped, 16- and
# 8-line tiles, one tile and several, ragged rows; the last beyond 96 MiB of
# spectrum, where the wider tile runs
@pytest.mark.parametrize("dtype", [C64, C128], ids=["c64", "c128"])
@pytest.mark.parametrize("dims", [(16, 5, 75), (32, 3, 125), (16, 5, 135), (96, 3, 250), (8, 9, 270), (32, 1, 360),
                                  (16, 3, 500), (64, 2, 540), (16, 2, 960), (8, 3, 1000), (8, 5, 256), (16, 3, 384),
                                  (32, 2, 512), (8, 3, 1024)], ids=str)
def test_fused_multiply_matches_oracle_and_unfused_bits(dims, dtype):
    nx, ny, nz = dims
    real = np.float32 if dtype == C64 else np.float64
    x = synth.normal_c((nz, ny, nx), seed=55).real.astype(real)
    g = np.abs(synth.normal_c((nz, ny, nx // 2 + 1), seed=56).real).astype(real)
    got, energy = run_conv(x, g, dtype)
    ref, ref_e = oracle.convolve_real(x.astype(np.float64), g.astype(np.float64))
    assert oracle.rel_l2(got, ref) <= TOL[dtype]
    assert abs(energy - ref_e) <= TOL[dtype] * abs(ref_e)
    plain, _ = unfused(torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda(), dtype)
    np.testing.assert_array_equal(got, plain.cpu().numpy())


@pytest.mark.parametrize("n", [360, 512])
def test_fused_multiply_of_a_large_spectrum_equals_unfused_bitwise(n):
    x = torch.randn((n, 250, 512), dtype=torch.float32, device="cuda")
    g = torch.rand((n, 250, 257), dtype=torch.float32, device="cuda")
    out = torch.empty_like(x)
    plan = croft.croft_plan_create_convolution(512, 250, n, C64)
    croft.croft_execute_convolution(plan, x, g, out)
    torch.cuda.synchronize()
    croft.croft_plan_destroy(plan)
    assert torch.equal(out, unfused(x, g, C64)[0])

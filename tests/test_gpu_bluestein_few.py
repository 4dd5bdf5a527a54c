"""Bluestein passes of few tiles run with more threads per line than passes of
many: the same convolution, so the bits of a line do not depend on how many
lines there are.  The line stands at index 0 of the other axes, zeros
elsewhere, whose transforms then copy it exactly to every index: its transform
in a launch of few tiles and of many, every convolution length that has two
shapes, and the few-tile result against the oracle within the suite's
tolerance."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_04896_amd as croft
from gpu_helpers import TOL

pytestmark = pytest.mark.gpu

C64, C128 = croft.CROFT_C64, croft.CROFT_C128


def transform(line, shape, dtype, direction):
    """The line along the axis of its length, alone in a grid of this (nz, ny, nx)."""
    nz, ny, nx = shape
    x = torch.zeros(shape, dtype=line.dtype, device="cuda")
    if nx == len(line):
        x[0, 0, :] = line
    else:
        x[0, :, 0] = line
    plan = croft.croft_plan_create(nx, ny, nz, dtype, direction)
    try:
        out = torch.full_like(x, complex(float("nan"), 0))
        croft.croft_execute(plan, x, out)
        torch.cuda.synchronize()
        t = [p for p in croft.croft_plan_info(plan)["passes"] if p["bluestein"]][0]["threads_per_line"]
    finally:
        croft.croft_plan_destroy(plan)
    flat = out.reshape(-1, nx) if nx == len(line) else out.permute(0, 2, 1).reshape(-1, ny)
    return flat, t


# few and many as (nz, ny, nx)
@pytest.mark.parametrize("direction", [croft.CROFT_FORWARD, croft.CROFT_BACKWARD], ids=["fwd", "bwd"])
@pytest.mark.parametrize("dtype,n,few,many,threads", [
    (C64, 211, (1, 211, 16), (160, 211, 16), (64, 32)), (C64, 613, (1, 3, 613), (4, 160, 613), (256, 128)),
    (C64, 1021, (1, 1021, 16), (40, 1021, 16), (256, 128)), (C64, 2039, (1, 2039, 16), (40, 2039, 16), (256, 128)),
    (C128, 67, (1, 3, 67), (80, 64, 67), (32, 16)), (C128, 127, (1, 127, 16), (300, 127, 16), (32, 16)),
    (C128, 131, (1, 131, 16), (160, 131, 16), (64, 32)), (C128, 1009, (1, 3, 1009), (4, 160, 1009), (256, 128))])
def test_few_lines_give_the_bits_of_many(dtype, n, few, many, threads, direction):
    g = torch.Generator(device="cuda").manual_seed(72)
    real = torch.float32 if dtype == C64 else torch.float64
    line = torch.view_as_complex(torch.randn((n, 2), generator=g, device="cuda", dtype=real))
    a, ta = transform(line, few, dtype, direction)
    b, tb = transform(line, many, dtype, direction)
    assert (ta, tb) == threads
    want = oracle.dft3d(line.cpu().numpy().astype(np.complex128).reshape(1, 1, n), direction).reshape(n)
    assert oracle.rel_l2(a[0].cpu().numpy(), want) <= TOL[dtype]
    assert torch.equal(a, a[:1].expand_as(a)) and torch.equal(b, a[:1].expand_as(b))

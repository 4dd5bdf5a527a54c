"""The workloads this library is timed on, one pass through its public entry points each.

``listed()`` names them, ``draw(rng)`` gives further ones of the same ranges,
``prepare`` makes what a program holds before the call (device inputs and
outputs, the plan), ``run`` is the call, ``work`` the bytes and operations it
cannot do without, and ``exact`` the same result from torch in 64 bits.

A case is a dict: ``op`` (c2c, half, real, conv or batch), ``dtype`` (c64,
c128, f16, bf16), ``dir`` (-1 forward, +1 backward) and the grid ``nx ny nz``;
a batch has ``count`` grids whose shapes come from ``shape_seed``.  All calls
run out of place, as repeated passes must see the same input.
"""
import math

import torch

import paper_2002_04896_amd as croft
from paper_2002_04896_amd import synth

DTYPE = {"c64": croft.CROFT_C64, "c128": croft.CROFT_C128, "f16": croft.CROFT_C16F, "bf16": croft.CROFT_C16B}
REAL = {"c64": torch.float32, "c128": torch.float64, "f16": torch.float16, "bf16": torch.bfloat16}
CPLX = {"c64": torch.complex64, "c128": torch.complex128}
BYTES = {"c64": 8, "c128": 16, "f16": 4, "bf16": 4}
# half lengths the real x pass is compiled for (nx / 2), from the library's list
REAL_HALF = (16, 32, 48, 60, 64, 72, 80, 96, 100, 120, 128, 160, 192, 200, 240, 256, 288, 320, 360, 384, 400, 480, 512)


def _grid(name, op, dtype, direction, nx, ny, nz):
    return {"name": name, "op": op, "dtype": dtype, "dir": direction, "nx": nx, "ny": ny, "nz": nz}


def listed():
    return [
        # the smallest grid in use: a small periodic box, called once per time step; launches and host time count
        _grid("c64_fwd_32cube", "c2c", "c64", -1, 32, 32, 32),
        # the paper's small grid in its own precision
        _grid("c128_fwd_128cube", "c2c", "c128", -1, 128, 128, 128),
        # the inverse of a middling grid that stays in the last-level cache
        _grid("c64_bwd_256cube", "c2c", "c64", 1, 256, 256, 256),
        # the headline: a 1 GiB complex64 grid
        _grid("c64_fwd_512cube", "c2c", "c64", -1, 512, 512, 512),
        # the paper's large grid size, the largest call a user makes (8 GiB in, 8 GiB out)
        _grid("c64_fwd_1024cube", "c2c", "c64", -1, 1024, 1024, 1024),
        # double precision on an uneven grid of lengths picked to fit a box rather than a power of two
        _grid("c128_bwd_360x300x250", "c2c", "c128", 1, 360, 300, 250),
        # 16-bit storage, chosen to halve the memory of a large grid
        _grid("bf16_fwd_512cube", "half", "bf16", -1, 512, 512, 512),
        # lengths with a large prime factor, as given by data that cannot be padded
        _grid("c64_fwd_509cube", "c2c", "c64", -1, 509, 509, 509),
        # a real field forward to its half spectrum (charge or density grids)
        _grid("real_c64_fwd_512cube", "real", "c64", -1, 512, 512, 512),
        # and a double precision spectrum back to an uneven real grid of particle-mesh size
        _grid("real_c128_bwd_160x144x150", "real", "c128", 1, 160, 144, 150),
        # the reciprocal-space step of particle-mesh Ewald, with its energy
        _grid("conv_c64_192x180x200", "conv", "c64", -1, 192, 180, 200),
        # many small uneven particle-mesh grids in one call
        {"name": "batch_c64_64grids", "op": "batch", "dtype": "c64", "dir": -1, "count": 64, "shape_seed": 4},
    ]


def _smooth(rng, lo, hi):
    """A 2^a 3^b 5^c length, near log-uniform in [lo, hi], odd ones among them."""
    target = lo * (hi / lo) ** rng.random()
    odd = rng.random() < 0.25
    best = min((n for n in _SMOOTH if lo <= n <= hi and (n % 2 == 1) == odd), key=lambda n: abs(math.log(n / target)))
    return best


_SMOOTH = sorted(2 ** a * 3 ** b * 5 ** c for a in range(11) for b in range(7) for c in range(5) if 2 ** a * 3 ** b * 5 ** c <= 1024)
_PRIME_LENGTHS = (17, 31, 61, 97, 127, 158, 211, 254, 331, 398, 509, 614, 763, 1009)


def draw(rng):
    """One more case: sizes spread over the logarithm of their range, at most a fraction of the largest listed case's time."""
    op = rng.choices(("c2c", "half", "real", "conv", "batch"), (40, 15, 20, 15, 10))[0]
    direction = rng.choice((-1, 1))
    if op == "batch":
        return {"op": op, "dtype": rng.choice(("c64", "c64", "c128")), "dir": direction,
                "count": int(2 ** rng.uniform(0, 6.5)), "shape_seed": rng.randrange(1 << 30)}
    dtype = rng.choice(("f16", "bf16")) if op == "half" else rng.choice(("c64", "c64", "c128"))
    prime = op in ("c2c", "half") and rng.random() < 0.15
    most = 2 ** (25 if prime else 26 if dtype == "c128" else 27)
    while True:
        dims = [_smooth(rng, 16, 1024) for _ in range(3)]
        if op in ("real", "conv"):
            dims[0] = 2 * rng.choice(REAL_HALF)
        if prime:
            dims[rng.randrange(3)] = rng.choice(_PRIME_LENGTHS)
        if 2 ** 14 <= dims[0] * dims[1] * dims[2] <= most:
            break
    return {"op": op, "dtype": dtype, "dir": -1 if op == "conv" else direction, "nx": dims[0], "ny": dims[1], "nz": dims[2]}


class _Batch:
    """A batched plan's handle, freed with the state that holds it."""

    def __init__(self, dims, dtype, direction):
        self.handle = croft.croft_plan_create_batched(dims, dtype, direction)
        self.offsets = croft.croft_plan_batched_offsets(self.handle, len(dims))

    def __del__(self):
        if getattr(self, "handle", None):
            croft.croft_plan_destroy(self.handle)


def _normal(shape, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _charges(nx, ny, nz, seed, dtype):
    """A particle-mesh charge grid: one +-1 charge a cell at a random place in it, spread with the order-4 cardinal B-spline."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (nz, ny, nx)
    charge = torch.randint(0, 2, shape, generator=g, device="cuda", dtype=torch.int8).to(dtype) * 2 - 1
    weights = []
    for _ in range(3):
        u = torch.rand(shape, generator=g, device="cuda", dtype=dtype)
        weights.append([(1 - u) ** 3 / 6, (3 * u ** 3 - 6 * u ** 2 + 4) / 6, (-3 * u ** 3 + 3 * u ** 2 + 3 * u + 1) / 6, u ** 3 / 6])
    grid = torch.zeros(shape, device="cuda", dtype=dtype)
    for k in range(4):
        plane = torch.zeros_like(grid)
        for j in range(4):
            row = torch.zeros_like(grid)
            for i in range(4):
                row += torch.roll(charge * weights[0][i] * weights[1][j] * weights[2][k], i, 2)
            plane += torch.roll(row, j, 1)
        grid += torch.roll(plane, k, 0)
    return grid


def _influence(nx, ny, nz, dtype):
    """The particle-mesh multiplier on the half spectrum: the Gaussian-screened Coulomb kernel times the B-spline moduli."""
    def freq(n, count):
        k = torch.arange(count, device="cuda", dtype=torch.float64)
        return torch.where(k <= n // 2, k, k - n) / n

    def moduli(f):
        return 1 / (2 / 3 + torch.cos(2 * math.pi * f) / 3) ** 2

    fx, fy, fz = freq(nx, nx // 2 + 1), freq(ny, ny), freq(nz, nz)
    m2 = fz[:, None, None] ** 2 + fy[:, None] ** 2 + fx ** 2
    g = torch.exp(-(math.pi / 0.3) ** 2 * m2) / (math.pi * nx * ny * nz * m2) * (moduli(fz)[:, None, None] * moduli(fy)[:, None] * moduli(fx))
    g[0, 0, 0] = 0
    return g.to(dtype).contiguous()


def _quantised(shape, kind, seed):
    """N(0, 1) values as 16-bit pairs with one power-of-two exponent a line along x, the line's peak just under 2^12."""
    v = _normal(shape + (2,), torch.float32, seed)
    e = torch.ceil(torch.log2(v.abs().amax(dim=(2, 3)))).to(torch.int32) - 12
    return torch.ldexp(v, -e[:, :, None, None]).to(REAL[kind]), e.to(torch.int8)


def _batch_dims(case):
    return [tuple(int(v) for v in row) for row in synth.batch_dims(case["shape_seed"], case["count"])]


def _input(case, seed):
    op, dtype = case["op"], case["dtype"]
    if op == "batch":
        parts = [_charges(*d, seed + 1000 * i, REAL[dtype]).reshape(-1) for i, d in enumerate(_batch_dims(case))]
        return torch.cat(parts).to(CPLX[dtype])
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if op == "half":
        return _quantised((nz, ny, nx), dtype, seed)
    if op == "c2c":
        return _normal((nz, ny, nx), CPLX[dtype], seed)
    if op == "real" and case["dir"] == 1:
        return _normal((nz, ny, nx // 2 + 1), CPLX[dtype], seed)
    return _charges(nx, ny, nz, seed, REAL[dtype])


def prepare(case, seed):
    op, dt, direction = case["op"], case["dtype"], case["dir"]
    x = _input(case, seed)
    s = {"op": op, "in": x}
    if op == "batch":
        s["plan"] = _Batch(_batch_dims(case), DTYPE[dt], direction)
        s["out"] = torch.empty_like(x)
        return s
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if op == "c2c":
        s["plan"] = croft.Plan(nx, ny, nz, DTYPE[dt], direction)
        s["out"] = torch.empty_like(x)
    elif op == "half":
        s["plan"] = croft.Plan(nx, ny, nz, DTYPE[dt], direction)
        s["in"], s["in_exp"] = x
        s["out"] = torch.empty_like(s["in"])
        s["out_exp"] = torch.empty((ny, nx), dtype=torch.int8, device="cuda")
    elif op == "real":
        s["plan"] = croft.RealPlan(nx, ny, nz, DTYPE[dt], direction)
        shape, kind = ((nz, ny, nx // 2 + 1), CPLX[dt]) if direction == -1 else ((nz, ny, nx), REAL[dt])
        s["out"] = torch.empty(shape, dtype=kind, device="cuda")
    else:
        s["plan"] = croft.ConvolutionPlan(nx, ny, nz, DTYPE[dt])
        s["mul"] = _influence(nx, ny, nz, REAL[dt])
        s["out"] = torch.empty_like(x)
        s["energy"] = torch.empty(1, dtype=torch.float64, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "half":
        return s["plan"].scaled(s["in"], s["in_exp"], s["out"], s["out_exp"])
    if op == "conv":
        return s["plan"](s["in"], s["mul"], s["out"], s["energy"]), s["energy"]
    if op == "batch":
        croft.croft_execute_batched(s["plan"].handle, s["in"], s["out"])
        return s["out"]
    return s["plan"](s["in"], s["out"])


def work(case):
    """One read of the input and one write of the output; 5 N log2 N operations (2.5 for real data)."""
    b = BYTES[case["dtype"]]
    if case["op"] == "batch":
        sizes = [x * y * z for x, y, z in _batch_dims(case)]
        return {"bytes": 2 * b * sum(sizes), "flops": sum(5 * n * math.log2(n) for n in sizes)}
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n, half = nx * ny * nz, (nx // 2 + 1) * ny * nz
    if case["op"] == "c2c":
        return {"bytes": 2 * b * n, "flops": 5 * n * math.log2(n)}
    if case["op"] == "half":
        return {"bytes": 2 * b * n + ny * nz + nx * ny, "flops": 5 * n * math.log2(n)}
    if case["op"] == "real":
        return {"bytes": b // 2 * n + b * half, "flops": 2.5 * n * math.log2(n)}
    return {"bytes": b * n + b // 2 * half, "flops": 5 * n * math.log2(n) + 2 * half}


def exact(case, seed):
    """The same call from torch.fft in 64 bits.

    None for 16-bit storage: a stored value means something only with the
    exponent its line was given, and the exponents are the call's own choice.
    """
    op = case["op"]
    if op == "half":
        return None
    x = _input(case, seed)
    x = x.to(torch.complex128 if x.is_complex() else torch.float64)
    backward = case["dir"] == 1

    def c2c(v):
        return torch.fft.ifftn(v, norm="forward") if backward else torch.fft.fftn(v)

    if op == "batch":
        out, at = [], 0
        for nx, ny, nz in _batch_dims(case):
            n = nx * ny * nz
            out.append(c2c(x[at:at + n].reshape(nz, ny, nx)).reshape(-1))
            at += n
        return torch.cat(out)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if op == "c2c":
        return c2c(x)
    if op == "real" and not backward:
        return torch.fft.rfftn(x)
    if op == "real":
        h = torch.fft.ifftn(x, dim=(0, 1), norm="forward")
        # only the real parts of the kx = 0 and kx = nx/2 terms enter
        h[..., 0].imag.zero_()
        h[..., nx // 2].imag.zero_()
        return torch.fft.irfft(h, n=nx, dim=2, norm="forward")
    g = _influence(nx, ny, nz, REAL[case["dtype"]]).double()
    q = torch.fft.rfftn(x)
    twice = torch.full((nx // 2 + 1,), 2.0, dtype=torch.float64, device="cuda")
    twice[0] = twice[nx // 2] = 1.0
    energy = (twice * g * (q.real ** 2 + q.imag ** 2)).sum().reshape(1)
    return torch.fft.irfftn(g * q, s=(nz, ny, nx), norm="forward"), energy

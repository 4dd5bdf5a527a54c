"""Which 2^a 3^b 5^c lengths have compiled passes (dry runs): all up to 1024 but
the short ones named here, and beyond it the powers of two."""
import pytest

import paper_2002_04896_amd as croft
from test_abi_cpu import parse_describe

SMOOTH = [n for n in range(2, 1025) if any(n == 2 ** a * 3 ** b * 5 ** c for a in range(11) for b in range(7) for c in range(5))]
SHORT = [3, 5, 6, 9, 10, 12, 15]
LINES = SHORT + [18, 20, 24, 25, 27, 30, 36, 40, 45, 50, 54]


def runtime_radix(describe, kind, *args):
    return [p for p in parse_describe(describe(*args))[1] if p["kind"] == kind][0]["kernel"] == "generic"


@pytest.mark.parametrize("dtype", range(4))
def test_lengths_without_a_compiled_pass(dtype):
    assert [n for n in SMOOTH if runtime_radix(croft.croft_plan_describe, "contiguous", n, 64, 2, dtype)] == LINES
    assert [n for n in SMOOTH if runtime_radix(croft.croft_plan_describe, "strided", 64, n, 1, dtype)] == SHORT
    if dtype < 2:
        assert [n for n in SMOOTH if runtime_radix(croft.croft_plan_describe_convolution, "fused", 32, 4, n, dtype)] == LINES
    assert [runtime_radix(croft.croft_plan_describe, "contiguous", n, 4, 2, dtype) for n in (1080, 2048, 3000, 4096)] \
        == [True, False, True, False]

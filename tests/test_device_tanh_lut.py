"""The FP64 tanh of the embedding kernels (tanh_lut: addition theorem around a
table of tanh at the multiples of 2^-LOG) emulated on the CPU with every FP64
operation rounded once, against a 50-digit tanh, and the table's source (long
double tanh rounded to double) against the correctly rounded values."""
import math
import random
import re
from decimal import Decimal, getcontext
from fractions import Fraction as Fr
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2410_22867_amd" / "csrc"
SRC = (CSRC / "dp_device.h").read_text()
BODY = SRC[SRC.index("double tanh_lut(double x"):]
BODY = BODY[:BODY.index("\n}")]
CLAMP = float(re.search(r"fabs\(x\), ([0-9.]+)\)", BODY).group(1))
C7, C5 = [float(v) for v in re.search(r"fma\(f2, (-[0-9.e-]+), ([0-9.]+)\)", BODY).groups()]
C5_ONLY = float(re.search(r"LOG == 7 \? ([0-9.]+)", BODY).group(1))
C3 = float(re.search(r"fma\(f2, g, (-[0-9.]+)\)", BODY).group(1))
N = int(re.search(r"kTanhLutEntries = ([0-9]+)", (CSRC / "dp_internal.h").read_text()).group(1))


def _tanh50(x):
    getcontext().prec = 50
    e = (Decimal(2) * Decimal(x)).exp()
    return (e - 1) / (e + 1)


def _fma(a, b, c):
    return float(Fr(a) * Fr(b) + Fr(c))


def _lut(log):
    return [float(_tanh50(k / 2.0 ** log)) for k in range(N if log == 7 else N // 2)]


def _emulated(x, log, tab):
    a = min(abs(x), CLAMP)
    magic = 1.5 * 2.0 ** (52 - log)
    s = a + magic
    k = int(np.float64(s).view(np.uint64)) & 0xFFFFFFFF
    T, f = tab[k], a - (s - magic)
    f2 = f * f
    g = C5_ONLY if log == 7 else _fma(f2, C7, C5)
    g = f2 * _fma(f2, g, C3)
    u = _fma(f, g, f)
    y = T * u
    y2 = y * y
    r = 1.0 - y
    if log == 7:
        r = _fma(r, _fma(y2, y2, y2), r)
    else:
        r = _fma(r, y2, r)
        r = _fma(r, y2 * y2, r)
    return math.copysign(_fma(_fma(-T, T, 1.0) * u, r, T), x)


@pytest.mark.parametrize("log", [7, 6])
def test_tanh_lut_error(log):
    assert CLAMP * 2 ** log + 0.5 < (N if log == 7 else N // 2)  # the last index read
    tab = _lut(log)
    rng = random.Random(log)
    h = 2.0 ** -log
    xs = [0.0, -0.0, h / 2, -h / 2, h, CLAMP, -CLAMP, 30.0, -1e300, 1e-300, 19.0, 19.07]
    xs += [rng.uniform(-4, 4) for _ in range(1500)] + [rng.uniform(-20, 20) for _ in range(300)]
    xs += [(rng.randrange(0, 600) + 0.5) * h * (1 + rng.choice((-1, 1)) * 2.0 ** -50) for _ in range(400)]
    # one half ulp of the table and of the last rounding each, the rest below 2^-60
    assert max(abs(Decimal(_emulated(x, log, tab)) - (_tanh50(x) if abs(x) < 40 else Decimal(math.copysign(1, x))))
               for x in xs) <= Decimal(1.3e-16)
    small = [rng.choice((-1, 1)) * 10.0 ** rng.uniform(-12, -3) for _ in range(300)]
    assert max(abs(Decimal(_emulated(x, log, tab)) / _tanh50(x) - 1) for x in small) <= Decimal(4e-16)


def test_table_source_is_correctly_rounded():
    got = np.tanh(np.arange(N, dtype=np.longdouble) / np.longdouble(128)).astype(np.float64)
    assert np.array_equal(got, np.array(_lut(7)))

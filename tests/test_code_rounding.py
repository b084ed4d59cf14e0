"""The rounding of 16-bit codes (CodeAxis, code_query and quant_scale of csrc), modelled in exact arithmetic: the
coded box contains the true one, and a query's gap to it in codes, with its excess past the frame, never
exceeds the true gap: for frames of any size, far from the origin and a few floats wide."""
import math
import random
from fractions import Fraction as F

import numpy as np
import pytest

TOP = 65535
f32 = np.float32


def step_of(lo, hi):
    extent = float(hi) - float(lo)
    s = f32(extent * ((1.0 + 2.0**-18) / TOP))
    while float(s) * TOP < extent * (1.0 + 2.0**-40):
        s = np.nextafter(s, f32(np.inf))
    return s


def down(x, lo, inv):
    return int(min(max((float(x) - float(lo)) * inv - 2.0**-10, 0.0), TOP))


def up(x, lo, inv):
    return int(min(math.ceil((float(x) - float(lo)) * inv + 2.0**-10), TOP)) if float(x) > float(lo) else 0


def query(c, lo, inv):
    u = (float(c) - float(lo)) * inv
    a, b = math.ceil(u + 2.0**-8), math.floor(u - 2.0**-8)
    e = max(0.0, max(-(u + 2.0**-8), u - 2.0**-8 - TOP) * (1.0 - 2.0**-40))
    return min(max(a, 0), TOP), min(max(b, 0), TOP), e


def frame(rng):
    kind = rng.random()
    if kind < 0.3:  # any two floats
        lo, hi = (f32(rng.choice([1, -1]) * rng.random() * 10.0 ** rng.uniform(-44, 38)) for _ in range(2))
    elif kind < 0.6:  # away from the origin
        lo = f32(rng.uniform(-1, 1) * 10.0 ** rng.uniform(-3, 7))
        hi = f32(float(lo) + 10.0 ** rng.uniform(-6, 4))
    else:  # a few floats wide
        lo = hi = f32(rng.uniform(-1, 1) * 10.0 ** rng.uniform(-3, 7))
        for _ in range(rng.randrange(1, 40)):
            hi = np.nextafter(hi, f32(np.inf))
    return (lo, hi) if lo < hi else (hi, lo)


@pytest.mark.parametrize("seed", range(4))
def test_codes_round_outward(seed):
    rng = random.Random(seed)
    checked = 0
    with np.errstate(over="ignore"):
        for _ in range(8000):
            lo, hi = frame(rng)
            if not hi > lo:
                continue
            step = f32(float(step_of(lo, hi)) * rng.choice([1, 1, 3.7, 200.0]))  # a common one may be wider
            if not np.isfinite(step):
                continue
            S, L, inv = F(float(step)), F(float(lo)), 1.0 / float(step)
            assert S * TOP >= F(float(hi)) - L

            def inside():
                return min(max(f32(float(lo) + (float(hi) - float(lo)) * rng.random()), lo), hi)

            a, b = sorted([inside(), inside()]) if rng.random() < 0.8 else (lo, hi)
            da, ub = down(a, lo, inv), up(b, lo, inv)
            assert L + da * S <= F(float(a)) and L + ub * S >= F(float(b)), (lo, hi, a, b)
            extent = float(hi) - float(lo)
            c = rng.choice([inside(), lo, hi, a, b, np.nextafter(a, f32(-np.inf)), np.nextafter(b, f32(np.inf)),
                            f32(float(lo) - 10.0 ** rng.uniform(-6, 3) * extent),
                            f32(float(hi) + 10.0 ** rng.uniform(-6, 3) * extent)])
            if not np.isfinite(c):
                continue
            qhi, qlo, e = query(c, lo, inv)
            gap = max(da - qhi, 0) + max(qlo - ub, 0)
            true = max(F(float(a)) - F(float(c)), F(float(c)) - F(float(b)), 0)
            assert (F(gap) + F(e)) * S <= true, (lo, hi, a, b, c)
            checked += 1
    assert checked > 5000

"""The reciprocal of the sigmoid, 1 / x for x in [1, 2] from an estimate and its residual
(recip_1_2 in common.hpp), in a model of its FP32 arithmetic: equal to the division for
every x and every estimate within one unit in the last place of it."""
import numpy as np

f4, f8 = np.float32, np.float64


def to_f4(s, err):
    """s + err (the exact sum, s its FP64 rounding) rounded once to FP32: s is moved to
    odd first, which leaves no halfway case to the second rounding."""
    even = (s.view(np.int64) & 1) == 0
    s = np.where((err != 0) & even, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
    return s.astype(f4)


def two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def one_step(x, r):
    """fma(fma(-x, r, 1), r, r)."""
    e = (1.0 - x.astype(f8) * r).astype(f4)  # 48-bit products, exact differences
    return to_f4(*two_sum(r.astype(f8), e.astype(f8) * r))


def test_one_residual_step_gives_the_division_except_at_the_all_ones_significand():
    x = (np.arange(1 << 23, (1 << 24) + 1).astype(f8) / (1 << 23)).astype(f4)
    want = (1.0 / x.astype(f8)).astype(f4)  # no quotient lies within 2^-48 of a tie
    last = f4(2 - 2.0 ** -23)
    wrong = set()
    for r in (want, np.nextafter(want, f4(0)), np.nextafter(want, f4(2))):
        near = np.abs(r * x.astype(f8) - 1.0) <= np.spacing(want).astype(f8) * x
        wrong |= set(x[near & (one_step(x, r) != want)].tolist())
    assert wrong <= {float(last)}
    assert one_step(np.array([last]), np.array([f4(0.5)]))[0] == f4(0.5)  # the estimate that needs the exception
    assert (1.0 / f8(last)).astype(f4) == f4(float.fromhex("0x1.000002p-1"))

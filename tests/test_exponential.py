"""The update's exponential (csrc/som_update.hip, exp_below) against the exponential to forty digits, on the CPU: its constants as the source has
them, its steps with every rounding as the hardware does it (a fused multiply-add rounds once, to the nearest)."""
import decimal
import math
import os
import random
import re
from fractions import Fraction

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_26555_amd", "csrc", "som_update.hip")


def constants():
    body = re.search(r"double exp_below\(double x\)\n\{(.*?)\n\}", open(SOURCE).read(), re.S)[1]
    found = {name: float.fromhex(value) for name, value in re.findall(r"(\w+) = (0x1\.[0-9a-f]+p[+-]\d+)", body)}
    assert set(found) == {f"c{i}" for i in range(10)} | {"log2e", "ln2_hi", "ln2_lo"}
    assert body.count("fma(") == 13 and "__builtin_rint(x * log2e)" in body
    return found


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def exp_below(x, k):
    x = max(x, -1100.0)
    n = round(x * k["log2e"])                                  # (half to even, as rint)
    r = fma(-n, k["ln2_lo"], fma(-n, k["ln2_hi"], x))
    q = k["c9"]
    for i in range(8, -1, -1):
        q = fma(q, r, k[f"c{i}"])
    return math.ldexp(fma(fma(q, r, 1.0), r, 1.0), n)


def test_less_than_one_unit_in_the_last_place():
    k, rng = constants(), random.Random(1)
    args = [-float.fromhex(h) for h in ("0x1.7328c141eba05p+8", "0x1.83cc6ebb7f98ep+8", "0x1.732aa604fe554p+8")]          # 0.949, 0.945, 0.935
    args += [-0.0, -2.0 ** -60, -0.5 * math.log(2), -708.3, -745.1]
    args += [-745.0 * rng.random() for _ in range(2500)] + [-2.0 ** (-30 * rng.random()) * 40 for _ in range(2500)]
    args += [-(i + 0.5) * math.log(2) * (1 + s * 1e-15) for i in range(0, 1070, 7) for s in (-1, 1)]                  # ends of the reduced range
    worst = 0.0
    with decimal.localcontext() as ctx:
        ctx.prec = 40
        for x in args:
            exact = Fraction(decimal.Decimal(x).exp())
            unit = Fraction(2) ** max(math.frexp(float(exact))[1] - 53, -1074)
            worst = max(worst, float(abs(Fraction(exp_below(x, k)) - exact) / unit))
    assert 0.9 < worst < 1.0, worst
    assert exp_below(-746.0, k) == 0.0 and exp_below(-1e300, k) == 0.0 and exp_below(-math.inf, k) == 0.0 and exp_below(0.0, k) == 1.0

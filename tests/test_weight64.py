"""weight64 (rwpt_pairs64.hip), emulated with correctly rounded binary64
operations, against exp(-s2 / sigma^2) in 60 digits: the products s2 esc64 and
the constant esc64 carry half an ulp each of the exponent x, so the weight's
relative error is at most 2^-53 (2 |x| + 1.2) (two halves of the exponent's,
rounding the polynomial, the table and the last product as in exp_tab)."""
import os
import random
import re
from decimal import Decimal, getcontext
from fractions import Fraction

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_05474_amd", "csrc")

getcontext().prec = 60


def _hex_of(name, text):
    return float.fromhex(re.search(name + r"\s*=\s*(0x[0-9a-fA-F.]+p[+-]?\d+)", text).group(1))


def _source():
    return open(os.path.join(CSRC, "rwpt_pairs64.hip")).read()


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def test_constants():
    text = _source()
    c, f = Decimal(2).ln() / 64, 1
    for n in range(1, 6):
        f *= n
        assert _hex_of("kC%d" % n, text) == float(Fraction(c ** n / f))
    api = open(os.path.join(CSRC, "rwpt_api.hip")).read()
    k = Decimal(re.search(r"P\.esc64_d = \(double\)\(-([0-9.]+)L", api).group(1))
    assert abs(k - 64 / Decimal(2).ln()) < Decimal("1e-18")


def test_error():
    text = _source()
    C = [_hex_of("kC%d" % n, text) for n in range(1, 6)]
    table = open(os.path.join(CSRC, "rwpt_pairstep.h")).read()
    body = re.search(r"kExp2Frac\[64\]\s*=\s*\{(.*?)\};", table, re.S).group(1)
    tbl = [float.fromhex(v) for v in re.findall(r"0x[0-9a-fA-F.]+p[+-]\d+", body)]
    rng = random.Random(3)
    worst = 0.0
    for t in range(1500):
        sigma2 = 10.0 ** rng.uniform(-9, 2)
        x = rng.uniform(0.0, 9.0 if t % 3 else 700.0)
        s2 = x * sigma2 if t else 0.0
        esc64 = float(Fraction(-64 / Decimal(2).ln()) / Fraction(sigma2))
        t64 = s2 * esc64
        z = t64 + 6755399441055744.0
        k = int(z - 6755399441055744.0)
        f = t64 - (z - 6755399441055744.0)
        assert abs(f) <= 0.5
        p = C[4]
        for c in C[3::-1]:
            p = _fma(p, f, c)
        e = tbl[k & 63]
        w = _fma(e, p * f, e) * 2.0 ** (k >> 6)
        exact = (-(Decimal(s2) / Decimal(sigma2))).exp()
        err = float(abs(Decimal(w) - exact) / exact) * 2.0 ** 53
        worst = max(worst, err / (2.0 * float(Decimal(s2) / Decimal(sigma2)) + 1.2))
        if t == 0:
            assert w == 1.0
    assert worst <= 1.0, worst

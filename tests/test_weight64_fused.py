"""weight64 (rwpt_pairs64.hip) with the kernel's own fused operations, in exact
arithmetic rounded once each: z = fma(s2, esc64, R), f = fma(s2, esc64, R - z).
Neither rounds the product, so of the exponent x only esc64's half ulp is left,
|x| 2^-53 of the weight; the table entry and the last operation round by 2^-53
each, and f, p and p f, all scaled by a q below 0.0055, by less than 0.1 2^-53
together: at most 2^-53 (|x| + 2.1)."""
import random
from decimal import Decimal, getcontext
from fractions import Fraction

import test_weight64 as w64

getcontext().prec = 60
R = 6755399441055744.0  # 1.5 * 2^52


def test_error_of_the_fused_form():
    text = w64._source()
    C = [w64._hex_of("kC%d" % n, text) for n in range(1, 6)]
    assert w64._hex_of("kRound", text) == R
    body = open(w64.CSRC + "/rwpt_pairstep.h").read().split("kExp2Frac[64] = {")[1].split("};")[0]
    tbl = [float.fromhex(v.strip()) for v in body.split(",") if v.strip()]
    rng = random.Random(8)
    worst = 0.0
    for t in range(3000):
        sigma2 = 10.0 ** rng.uniform(-12, 3)
        x = rng.uniform(0.0, 9.0 if t % 3 else 700.0)
        s2 = x * sigma2 if t else 0.0
        esc64 = float(Fraction(-64 / Decimal(2).ln()) / Fraction(sigma2))
        z = w64._fma(s2, esc64, R)
        f = w64._fma(s2, esc64, R - z)
        assert abs(f) <= 0.5
        k = int(z - R)
        p = C[4]
        for c in C[3::-1]:
            p = w64._fma(p, f, c)
        e = tbl[k & 63]
        w = w64._fma(e, p * f, e) * 2.0 ** (k >> 6)
        arg = Decimal(s2) / Decimal(sigma2)
        exact = (-arg).exp()
        worst = max(worst, float(abs(Decimal(w) - exact) / exact) * 2.0 ** 53 / (float(arg) + 2.1))
        assert t or w == 1.0
    assert worst <= 1.0, worst

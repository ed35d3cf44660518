"""The quantizers' division (quant.h Divider) in exact arithmetic: the
five-operation sequence with every product and sum rounded once to fp32 gives
the correctly rounded quotient, as Markstein's theorem says, on random and
adversarial mantissas (all ones, near one, neighbours of the divisor)."""
import random
from fractions import Fraction


def rn(v):
    """Fraction rounded to 24 bits, ties to even (no exponent limits)."""
    if v == 0:
        return v
    s, a = (-1, -v) if v < 0 else (1, v)
    e = a.numerator.bit_length() - a.denominator.bit_length() - 24
    scale = Fraction(2) ** e
    while a / scale >= 1 << 24:
        scale *= 2
    while a / scale < 1 << 23:
        scale /= 2
    q = a / scale
    f = q.numerator // q.denominator
    r = q - f
    if r > Fraction(1, 2) or (r == Fraction(1, 2) and f & 1):
        f += 1
    return s * f * scale


def divider(x, d):
    r = rn(Fraction(1) / d)
    q = rn(x * r)
    q = rn(rn(x - q * d) * r + q)
    return rn(rn(x - q * d) * r + q)


def test_correctly_rounded():
    rng = random.Random(3)

    def mantissa():
        m = rng.getrandbits(23)
        kind = rng.randrange(4)
        if kind == 0:
            m |= 0x7ffff0
        elif kind == 1:
            m &= 0xf
        return m | 1 << 23

    for _ in range(4000):
        md = mantissa()
        mx = mantissa() if rng.random() < 0.7 else max(1 << 23, min((1 << 24) - 1,
                                                                    md + rng.randrange(-3, 4)))
        x = Fraction(rng.choice((-1, 1)) * mx) * Fraction(2) ** rng.randrange(-20, 20)
        d = Fraction(md) * Fraction(2) ** rng.randrange(-40, 20)
        assert divider(x, d) == rn(x / d), (mx, md)

"""Host model of an integer's entry into RNS: the kernel's conversion of limbs
in sums of rns_chunk, its constants of a modulus by powers, and the first
products of what has entered, every word held to its range; and the ranges'
bounds themselves, step by step."""
import math
import random
from fractions import Fraction

import pytest

from paper_1407_1465_amd import rns_tables as T
from test_rns_model import Model, R, red

MASK = (1 << 29) - 1


def chunk(limbs):
    return 6 if limbs % 6 == 0 else 7


class Entry(Model):
    def residues(self, x, base, most):
        """x's residues as k_rns_pow converts its limbs: unreduced words."""
        c, out = self.c, []
        for i, m in enumerate(base):
            v = 0
            for l0 in range(0, c.limbs, chunk(c.limbs)):
                t = v * (R - 2 * m)
                for l in range(l0, l0 + chunk(c.limbs)):
                    t += ((x >> (29 * l)) & MASK) * T.centered(R << (29 * l), m)
                v = red(t, m)
                assert abs(v) < most * 2 ** 31
            out.append(v)
        return out

    def setup(self, n):
        """c by n^(a - 2), v and v16, in the kernel's unreduced words."""
        c, self.ci = self.c, []
        for i, (r, a) in enumerate(zip(self.residues(n, c.a, 0.9376), c.a)):
            k = inv = red(r * self.t["R2A"][i], a)
            for bit in range(29, -1, -1):
                inv = red(inv * inv, a)
                m = red(inv * k, a)
                inv = m if (a - 2) >> bit & 1 else inv
            self.ci.append(red(inv * self.t["CINV"][i], a))
            assert abs(self.ci[-1]) <= 0.7501 * 2 ** 31
            assert (self.ci[-1] - red(T.centered(pow(n, -1, a) * R, a) * self.t["CINV"][i], a)) % a == 0
        self.v = [red(r * (R - 2 * b), b) for r, b in zip(self.residues(n, c.b, 0.9376), c.b)]
        assert all((v - n) % b == 0 and abs(v) < b // 2 + 2 ** 12 for v, b in zip(self.v, c.b))
        self.v16 = [red(v * self.t["V16"][j], b) for j, (v, b) in enumerate(zip(self.v, c.b))]

    def enter(self, x):
        c = self.c
        xa = self.residues(x, c.a, 0.9376)
        xb = [red(v * self.t["WR"][j], b) for j, (v, b) in enumerate(zip(self.residues(x, c.b, 0.9376), c.b))]
        assert all((v - x) % a == 0 for v, a in zip(xa, c.a))
        assert all((v - x * w) % b == 0 for v, w, b in zip(xb, c.w, c.b))
        return xa, xb


@pytest.mark.parametrize("cfg", T.CONFIGS)
def test_products_of_what_entered(cfg):
    m = Entry(cfg)
    c = m.c
    rng = random.Random(c.k + 1)
    for n in ((1 << c.bits) - 1, rng.getrandbits(c.bits) | 1 << (c.bits - 1) | 1, 3):
        while any(n % a == 0 for a in c.a):
            n -= 2
        m.setup(n)
        for x in (n - 1, rng.randrange(n), 0):
            xt = m.enter(x * c.A % n)
            y, e = m.mul(xt, xt), 2                     # both factors entered
            for times in (False, True, False):
                r = m.value(y)
                assert abs(r) <= 7 * c.k * n // 8 and r % n == pow(x, e, n) * c.A % n
                y, e = (m.mul(y, xt), e + 1) if times else (m.mul(y, y), 2 * e)


@pytest.mark.parametrize("cfg", T.CONFIGS)
def test_bounds_of_the_words(cfg):
    """In units of 2^31, red(x y) is below x y / 2 + 1 / 2 for words below x and
    y; a constant is below 1 / 2."""
    F, half = Fraction, Fraction(1, 2)

    def prod(x, y):
        return x * y / 2 + half
    limbs, k = cfg[1], 4 * cfg[0]
    entered = chunk(limbs) * F(1 << 59, 1 << 63) + F(1, 1 << 18) + half        # limbs below 2^29, constants 2^30
    assert entered < F(94, 100)
    n_a = prod(entered, half)
    inv = n_a
    for _ in range(30):                                # any bits of a - 2
        sq = prod(inv, inv)
        inv = F(math.ceil(max(sq, prod(sq, n_a)) * 2 ** 60), 2 ** 60)
        assert inv < 1
    c = prod(inv, half)
    xi = prod(prod(entered, entered), c) + F(0x00808080, 1 << 31)
    assert c <= F(3, 4) and xi < F(86, 100)
    # q in units of A (residues over moduli 2^31 less up to a few thousand), and
    # |x y| / A n below 2^-2, where |x|, |y| < 0.875 k n
    assert xi * (1 + F(1, 1 << 18)) * k + F(1, 4) < F(7, 8) * k and F(7, 8) * k < 64
    assert prod(prod(entered, half), prod(entered, half)) < F(9, 10)            # in B

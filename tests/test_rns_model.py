"""Host models of the RNS exponentiation.

The product: the kernel's word arithmetic (signed Montgomery reductions by
2^32, signed base-256 digits, 32-bit plane accumulators, the uncorrected
extension A -> B and the corrected one B -> A) on Python integers with the
generated tables' constants, every intermediate held to its word's range, for
the largest and random moduli of every configuration, against pow().

The way in: the quotient estimate of rgrp_sub_multiple (a lane's limbs as one
Horner chain of fused multiply-adds, modelled by exact rationals rounded
once per step) is the floor of y / n or one less."""
import math
import random
from fractions import Fraction

import pytest

from paper_1407_1465_amd import rns_tables as T

R = 1 << 32


def s32(x):
    x &= R - 1
    return x - R if x >> 31 else x


def red(t, m):
    """rns_red: t / 2^32 modulo m as a signed word."""
    assert -(1 << 63) <= t < 1 << 63
    t += s32(t * (-pow(m, -1, R) % R)) * m
    assert -(1 << 63) <= t < 1 << 63 and t % R == 0
    r = t >> 32
    assert -(1 << 31) <= r < 1 << 31
    return r


class Model:
    def __init__(self, cfg):
        c = self.c = T.Config(*cfg)
        self.words = {True: self.unpack(c.matrix(True), c.units), False: self.unpack(c.matrix(False), c.units + 1)}
        perm = [(i % 4) * c.units + i // 4 for i in range(c.k)]
        self.t = {n: [v[p] for p in perm] for n, v in c.residue_tables().items()}

    def unpack(self, words, tiles):
        """Matrix entries [tile][row][operand byte] from the packed layout."""
        ks = self.c.ksteps
        out = [[[0] * (64 * ks) for _ in range(16)] for _ in range(tiles)]
        for t in range(tiles):
            for s in range(ks):
                for lane in range(64):
                    for q in range(4):
                        w = words[((t * ks + s) * 64 + lane) * 4 + q]
                        for p in range(4):
                            v = (w >> (8 * p)) & 255
                            out[t][lane % 16][64 * s + 16 * (lane // 16) + 4 * q + p] = v - 256 if v > 127 else v
        return out

    def operand(self, digits, alpha=None):
        """Operand bytes of a column: residue 4 u + g is word u % 4 of lane
        group g in k step u / 4."""
        c = self.c
        x = [0] * (64 * c.ksteps)
        for i, d in enumerate(digits):
            u, g = divmod(i, 4)
            for p in range(4):
                x[64 * (u // 4) + 16 * g + 4 * (u % 4) + p] = d[p]
        if alpha is not None:
            x[64 * (c.units // 4) + 4 * (c.units % 4)] = alpha
            assert -128 <= alpha < 128
        return x

    def extend(self, to_b, digits, alpha=None):
        """(lo, hi) of every extended residue lo + 2^16 hi."""
        x = self.operand(digits, alpha)
        out = [0] * self.c.k
        for u in range(self.c.units):
            for g in range(4):
                acc = [sum(a * b for a, b in zip(self.words[to_b][u][4 * g + r], x)) for r in range(4)]
                lo, hi = acc[0] + (acc[1] << 8), acc[2] + (acc[3] << 8)
                assert all(abs(v) < 1 << 31 for v in acc + [lo, hi])
                out[4 * u + g] = lo, hi
        return out

    def setup(self, n):
        c = self.c
        self.ci = [red(T.centered(pow(n, -1, a) * R, a) * self.t["CINV"][i], a) for i, a in enumerate(c.a)]
        self.v = [T.centered(n, b) for b in c.b]
        self.v16 = [red(v * self.t["V16"][j], b) for j, (v, b) in enumerate(zip(self.v, c.b))]

    def enter(self, x):
        c = self.c
        return [T.centered(x, a) for a in c.a], [T.centered(x * w, b) for w, b in zip(c.w, c.b)]

    def mul(self, x, y):
        c = self.c
        bias = 0x00808080
        xi = []
        for i, a in enumerate(c.a):
            s = red(x[0][i] * y[0][i], a)
            biased = red(s * self.ci[i] + (bias << 32), a)
            xi.append(T.digits(biased - bias))
        q = self.extend(True, xi)
        xb = []
        for j, b in enumerate(c.b):
            s = red(x[1][j] * y[1][j], b)
            lo, hi = q[j]
            xb.append(red(s * self.t["KAPPA"][j] + lo * self.v[j] + hi * self.v16[j], b))
            assert abs(xb[-1]) < 0.9 * 2 ** 31 and xb[-1] + bias < 1 << 31
        dig = [T.digits(v) for v in xb]
        tops = self.operand(dig)
        self.alpha = (sum(a * b for a, b in zip(self.words[False][c.units][0], tops)) + 64) >> 7
        assert self.alpha == (sum(d[3] for d in dig) + 64) >> 7
        xa = [red((hi << 16) + lo, c.a[i]) for i, (lo, hi) in enumerate(self.extend(False, dig, self.alpha))]
        return xa, xb

    def value(self, x):
        c = self.c
        return sum(v * (c.B // b) for v, b in zip(x[1], c.b)) - self.alpha * c.B


@pytest.mark.parametrize("cfg", T.CONFIGS)
def test_products(cfg):
    m = Model(cfg)
    c = m.c
    rng = random.Random(c.k)
    for n in ((1 << c.bits) - 1, rng.getrandbits(c.bits) | 1, rng.getrandbits(40) | 1, 3):
        while any(n % a == 0 for a in c.a):
            n -= 2
        m.setup(n)
        bound = 3 * c.k * n // 4 + n
        x = rng.randrange(n)
        xt, e = m.enter(x * c.A % n), 1
        y = xt
        for step in range(3):
            y, e = m.mul(y, y), 2 * e
            if step == 1:
                y, e = m.mul(y, xt), e + 1
            r = m.value(y)
            assert abs(r) <= bound and r % n == pow(x, e, n) * c.A % n
            assert all((r - v) % a == 0 for v, a in zip(y[0], c.a))
        one = [1] * c.k, [T.centered(w, b) for w, b in zip(c.w, c.b)]
        r = m.value(m.mul(y, one))
        # the way out adds 64 n and takes the limbs of less than 128 n
        assert r % n == pow(x, e, n) and -64 * n <= r < 64 * n and 128 * n <= 1 << (29 * c.limbs)


def test_moduli_are_distinct_primes():
    for cfg in T.CONFIGS:
        c = T.Config(*cfg)
        ps = c.a + c.b
        assert len(set(ps)) == 2 * c.k and all(T._is_prime(p) and 1 << 30 < p < 1 << 31 for p in ps)


def fl(x):
    return float(x)                             # a Fraction rounds once, to nearest


def scaled(v, e, S, G):
    """Lane 0's value of rgrp_scaled for v below 2^(29 S + 29)."""
    L = S // G
    parts = []
    for r in range(G):
        part = float(v >> (29 * S)) if r == G - 1 else 0.0
        for j in range(L - 1, -1, -1):
            limb = (v >> (29 * (r * L + j))) & ((1 << 29) - 1)
            part = fl(Fraction(part) * (1 << 29) + limb)
        parts.append(math.ldexp(part, 29 * r * L - e))
    o = 1
    while o < G:
        parts = [parts[r] + parts[r ^ o] for r in range(G)]
        o <<= 1
    return parts[0]


@pytest.mark.parametrize("S,G", [(18, 2), (20, 4), (28, 4), (36, 2), (36, 4), (56, 8), (64, 16), (72, 4), (72, 8),
                                 (80, 16), (112, 8), (144, 8), (144, 16)])
def test_quotient_is_the_floor_or_one_less(S, G):
    rng = random.Random(S * 100 + G)
    width = 29 * S - 10
    for _ in range(60):
        bits = rng.choice([width, rng.randint(2, width), rng.randint(width - 64, width)])
        n = rng.getrandbits(bits) | (1 << (bits - 1)) | 1
        bl = n.bit_length()
        rn = 1.0 / scaled(n, bl, S, G)
        k = rng.randrange(1, 1 << 28)
        for y in (rng.randrange(n << 28), k * n - 1, k * n, k * n + 1, 0, n - 1, n):
            q = max(0, int(math.floor(scaled(y, bl, S, G) * rn - 2.0 ** -16)))
            assert y // n - 1 <= q <= y // n, (S, G, n, y, q)

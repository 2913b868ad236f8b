"""Constant tables of the residue-number-system (RNS) exponentiation kernels.

The kernels of csrc/rns_kernels.hpp hold an integer as its residues modulo
two sets of k primes just below 2^31 (bases A and B, products also called A
and B) and multiply by Montgomery's method with A in the place of the power
of two (RNS Montgomery multiplication: Posch and Posch 1995; Bajard, Didier
and Kornerup 1998; the correction of the second base extension from the
leading digits of the residues: Kawamura, Koike, Sano and Shimbo 2000).  The
two base extensions are products with constant matrices, which the kernels
run on the integer matrix cores.  This module generates those matrices and
the per-residue constants as C++ source.

Layout.  A configuration of `units` has k = 4 * units residues per base; a
wave holds 16 integers, lane l the residues (u, g) of integer l % 16 with
g = l / 16, residue index 4 * u + g.  A residue is a signed 32-bit word; as a matrix operand it is four signed
base-256 digits.  Row r of an extension's matrix gives one signed base-256
digit (plane) of a residue of the target base, so the four accumulators that
a lane receives per residue combine to a 47-bit value congruent to the
extended residue.
"""
from __future__ import annotations

import math
import os
from typing import Dict, List

R = 1 << 32
LIMB_BITS = 29          # limbs of the positional side (csrc/radix_bn.hpp)


def _is_prime(n: int) -> bool:
    """Miller-Rabin with bases 2, 3, 5, 7: exact below 3.2e9."""
    for p in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if n % p == 0:
            return n == p
    d, s = n - 1, 0
    while d % 2 == 0:
        d //= 2
        s += 1
    for a in (2, 3, 5, 7):
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def primes_below_2_31(count: int) -> List[int]:
    out, c = [], (1 << 31) - 1
    while len(out) < count:
        if _is_prime(c):
            out.append(c)
        c -= 2
    return out


def centered(x: int, m: int) -> int:
    x %= m
    return x - m if x > m // 2 else x


def digits(x: int) -> List[int]:
    """Four signed base-256 digits of a signed 32-bit value: the lower three
    in [-128, 128), the top one whatever remains."""
    out = []
    for _ in range(3):
        d = ((x + 128) & 255) - 128
        out.append(d)
        x = (x - d) >> 8
    assert -128 <= x < 128
    out.append(x)
    return out


class Config:
    """Tables of one configuration: `units` residues of each base per lane,
    positional integers of `limbs` 29-bit limbs, moduli of at most `bits`
    bits."""

    def __init__(self, units: int, limbs: int, bits: int):
        self.units, self.limbs, self.bits = units, limbs, bits
        k = self.k = 4 * units
        ps = primes_below_2_31(2 * k)
        a, b = self.a, self.b = ps[:k], ps[k:]
        self.A, self.B = math.prod(a), math.prod(b)
        # values stay within +-0.875 k n (see csrc/rns_arith.hpp): the square
        # of that must vanish against A n, and it must be small against B
        lim = (7 * k // 8 + 1) << bits
        assert (7 * k // 8 + 1) ** 2 << bits < self.A >> 2 and lim < self.B >> 6
        assert 128 << bits <= 1 << (LIMB_BITS * limbs) and 7 * k // 8 + 1 <= 64
        self.w = [pow(self.B // p, -1, p) for p in b]
        self.ksteps = -(-units // 4)
        self._check_accumulators()

    def _check_accumulators(self) -> None:
        """The plane accumulators of A -> B, combined in pairs (lo, hi) and
        multiplied by words of at most 0.5 and 0.63 times 2^31, leave room for
        the product they are added to (see rns_arith.hpp): with residues of at
        most 0.9 * 2^31, |s kappa + lo v + hi v16| / 2^32 + m / 2 is below
        that again."""
        most = 0
        for j in range(self.k):
            planes = [0] * 4
            for i in range(self.k):
                for p in range(4):
                    for r, d in enumerate(digits(centered(self.ext_ab(i, j) << (8 * p), self.b[j]))):
                        planes[r] += 128 * abs(d)
            most = max(most, planes[0] + 256 * planes[1] + 1.26 * (planes[2] + 256 * planes[3]))
        s = 0.9 * 0.9 / 2 + 0.5                 # |s| / 2^31 for s = x y / 2^32
        assert (s / 4 + most / 2 ** 33) + 0.5 < 0.9, (self.units, most)

    def ext_ab(self, i: int, j: int) -> int:
        """A -> B: q = sum xi_i (A / a_i), scaled by A^-1 w_j 2^32."""
        m = self.b[j]
        return (self.A // self.a[i]) * pow(self.A, -1, m) * self.w[j] * R % m

    def ext_ba(self, j: int, i: int) -> int:
        """B -> A: r = sum xi_j (B / b_j) - alpha B, scaled by 2^32."""
        return (self.B // self.b[j]) * R % self.a[i]

    def matrix(self, to_b: bool) -> List[int]:
        """Words [row tile][k step][lane][4] of the extension's matrix in the
        first operand's layout of the 16x16x64 product: row tile t holds the
        planes of unit t (row 4 g + plane).  The extension back has one more
        operand word, unit U of group 0, whose lowest byte is alpha (its
        coefficients are those of -B), and one more row tile, whose row 0
        sums the top digits."""
        U, k = self.units, self.k
        src, dst = (self.a, self.b) if to_b else (self.b, self.a)
        ext = self.ext_ab if to_b else self.ext_ba
        # rows[j][i][p][r]: plane r of the residue entry (j, i) times 256^p
        rows = [[[digits(centered(ext(i, j) << (8 * p), dst[j])) for p in range(4)] for i in range(k)]
                for j in range(k)]
        alpha = [digits(centered(-self.B * R, m)) for m in dst]
        assert U % 4 != 0                       # room for alpha's word

        def entry(t, row, u, kg, p):
            if t == U:
                return 1 if row == 0 and p == 3 and u < U else 0
            if u < U:
                return rows[4 * t + row // 4][4 * u + kg][p][row % 4]
            return alpha[4 * t + row // 4][row % 4] if not to_b and (u, kg, p) == (U, 0, 0) else 0

        out = []
        for t in range(U + (0 if to_b else 1)):
            for s in range(self.ksteps):
                for lane in range(64):
                    for q in range(4):
                        out.append(sum((entry(t, lane % 16, 4 * s + q, lane // 16, p) & 255) << (8 * p)
                                       for p in range(4)))
        return out

    def residue_tables(self) -> Dict[str, List[int]]:
        """Per-residue constants, [group][unit] each."""
        t: Dict[str, List[int]] = {n: [] for n in ("MA", "NA", "MB", "NB", "KAPPA", "CINV", "R2A", "WR",
                                                   "WONE", "V16")}
        for g in range(4):
            for u in range(self.units):
                i = 4 * u + g
                a, b, w = self.a[i], self.b[i], self.w[i]
                t["MA"].append(a)
                t["NA"].append(-pow(a, -1, R) % R)
                t["MB"].append(b)
                t["NB"].append(-pow(b, -1, R) % R)
                t["KAPPA"].append(centered(R * R * pow(w, -1, b) * pow(self.A, -1, b), b))
                t["CINV"].append(centered(-R * R * pow(self.A // a, -1, a), a))
                t["R2A"].append(centered(R * R, a))
                t["WR"].append(centered(w * R, b))
                t["WONE"].append(centered(w, b))
                t["V16"].append(centered(R << 16, b))
        return t

    def conversion(self, base: List[int]) -> List[int]:
        """2^(29 l) * 2^32 modulo each residue, [limb][group][unit]."""
        return [centered(R << (LIMB_BITS * l), base[4 * u + g])
                for l in range(self.limbs) for g in range(4) for u in range(self.units)]

    def positional(self) -> List[int]:
        """Limbs modulo 2^(29 limbs) of B / b_j, j in residue-index order,
        of -B and (the one integer that is not modulo) of A, two limbs more."""
        S, out = self.limbs, []
        for v, limbs in [(self.B // p, S) for p in self.b] + [(-self.B, S), (self.A, S + 4)]:
            out += [(v >> (LIMB_BITS * l)) & ((1 << LIMB_BITS) - 1) for l in range(limbs)]
        assert self.A >> (LIMB_BITS * (S + 4)) == 0
        return out


# (units, limbs, bits): moduli of up to 512, 768, 1024, 1536 and 2048 bits.
CONFIGS = [(5, 18, 512), (7, 28, 768), (9, 36, 1024), (13, 56, 1536), (17, 72, 2048)]


def _array(name: str, words: List[int]) -> str:
    body = []
    for i in range(0, len(words), 12):
        body.append("    " + ", ".join("0x%xu" % (w & 0xFFFFFFFF) for w in words[i:i + 12]) + ",")
    return "static __device__ const __attribute__((aligned(16))) uint32_t %s[%d] = {\n%s\n};\n" % (
        name, len(words), "\n".join(body))


def source(units: int, limbs: int, bits: int) -> str:
    """C++ source of one configuration: its arrays and the RnsTables
    specialisation that names them."""
    c = Config(units, limbs, bits)
    p = "rns_%d_" % units
    arrays = {"EAB": c.matrix(True), "EBA": c.matrix(False), "CA": c.conversion(c.a), "CB": c.conversion(c.b),
              "POS": c.positional()}
    arrays.update(c.residue_tables())
    out = ["// Generated by rns_tables.py; do not edit.\n"]
    for name, words in arrays.items():
        out.append(_array(p + name, words))
    out.append("template <> struct RnsTables<%d> {\n    static constexpr int LIMBS = %d, BITS = %d, ABITS = %d;\n"
               % (units, limbs, bits, c.A.bit_length()))
    for name in arrays:
        out.append("    static __device__ __forceinline__ const uint32_t *%s() { return %s; }\n" % (name.lower(), p + name))
    out.append("};\n")
    return "".join(out)


def primes_source() -> str:
    """C++ source of every configuration's base A, for host code."""
    out = ["// Generated by rns_tables.py; do not edit.\n"]
    for units, limbs, bits in CONFIGS:
        a = Config(units, limbs, bits).a
        out.append("static const uint32_t kRnsPrimes%d[%d] = {%s};\n" % (units, len(a), ", ".join("%du" % p for p in a)))
    return "".join(out)


def write(directory: str) -> None:
    """Writes rns_tables_<units>.inc for every configuration, and
    rns_primes.inc."""
    os.makedirs(directory, exist_ok=True)
    files = {"rns_tables_%d.inc" % cfg[0]: source(*cfg) for cfg in CONFIGS}
    files["rns_primes.inc"] = primes_source()
    for name, text in files.items():
        path = os.path.join(directory, name)
        if os.path.exists(path) and open(path).read() == text:
            continue
        tmp = path + ".tmp%d" % os.getpid()
        with open(tmp, "w") as f:
            f.write(text)
        os.replace(tmp, path)

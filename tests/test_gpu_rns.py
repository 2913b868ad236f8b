"""RNS exponentiation (default plans, 13 to 64 words per modulus) against
Python's pow, bit-exact: every width class, one and several waves per tile
and several tiles per workgroup (batch sizes on both sides of each launch
rule), tiles with one exponent and with sixteen, exponents on both sides of
the positional limit, moduli that share a factor with base A, short and
invalid moduli, results written over the input."""
import math
import random

import numpy as np
import pytest

from paper_1407_1465_amd import rns_tables as T
from paper_1407_1465_amd import workloads as W
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1407_1465_amd import rsagpu  # noqa: E402

CLASSES = {words: cfg for words, cfg in zip((16, 24, 32, 48, 64), T.CONFIGS)}


def check(out, want, limbs):
    got = host(out)
    bad = np.nonzero((got != W.ints_to_limbs(want, limbs)).any(axis=1))[0]
    assert bad.size == 0, "%d of %d differ, first %d" % (bad.size, len(want), bad[0])


def odd(rng, bits):
    return rng.getrandbits(bits) | 1 | 1 << (bits - 1)


def base_multiple(rng, words, bits):
    """An odd modulus of `bits` bits divisible by a prime of base A."""
    c = T.Config(*CLASSES[words])
    a = c.a[rng.randrange(c.k)]
    return odd(rng, bits - a.bit_length()) * a


@pytest.mark.parametrize("limbs", [13, 16, 24, 31, 32, 48, 61, 64])
@pytest.mark.parametrize("shared", [False, True])
def test_modexp_edges(limbs, shared):
    words = min(w for w in CLASSES if w >= limbs)
    rng = random.Random(limbs * 2 + shared)
    bits = 32 * limbs
    n = [odd(rng, bits) for _ in range(37)]
    n[1], n[2], n[3] = (1 << bits) - 1, odd(rng, 70), 3
    n[4], n[18] = base_multiple(rng, words, bits - 1), base_multiple(rng, words, bits // 2)
    x = [rng.getrandbits(bits) for _ in n]
    x[5], x[6], x[7] = 0, 1, n[7] - 1
    e = [rng.getrandbits(bits) for _ in n]
    if shared:
        e = [e[0]] * len(n)
    else:
        e[8:18] = [0, 1, 2, 65537, (1 << 64) - 1, 1 << 64, (1 << 64) + 1, (1 << bits) - 1, 1 << (bits - 1),
                   rng.getrandbits(65) | 1 << 64]
    want = [pow(*v) for v in zip(x, e, n)]
    # even moduli, zero and one: output zero, all but one counted
    bad = {20: 0, 21: 1, 22: n[22] - 1, 36: 2}
    for i, m in bad.items():
        n[i], want[i] = m, 0
    base, exp, mod = (dev(W.ints_to_limbs(v, limbs)) for v in (x, e, n))
    rsagpu.device_errors()
    check(rsagpu.modexp(base, exp, mod), want, limbs)
    assert rsagpu.device_errors() == 3
    check(rsagpu.modexp(base, exp, mod, out=base), want, limbs)
    assert rsagpu.device_errors() == 3


# one wave per residue, three waves, one wave (several tiles per workgroup)
@pytest.mark.parametrize("limbs,count", [(16, 1000), (24, 16 * 256), (24, 16 * 256 + 1), (32, 16 * 256), (32, 16 * 257),
                                         (32, 16 * 512 + 3), (32, 16 * 1024 + 17), (48, 16 * 256), (48, 16 * 256 + 1),
                                         (48, 16 * 512 + 3),
                                         (64, 300)])
def test_modexp_launch_shapes(limbs, count):
    rng = random.Random(limbs + count)
    bits = 32 * limbs
    n = [odd(rng, bits) for _ in range(40)]
    e = [rng.getrandbits(80) | 1 << 79 for _ in range(3)] + [65537]
    pick = [(rng.randrange(40), rng.choice((0, 0, 0, 1, 2, 3)) if (i // 16) % 3 else 0) for i in range(count)]
    x = [rng.getrandbits(bits) for _ in range(count)]
    cols = [W.ints_to_limbs(x, limbs), W.ints_to_limbs(e, limbs)[[k for _, k in pick]],
            W.ints_to_limbs(n, limbs)[[j for j, _ in pick]]]
    check(rsagpu.modexp(*[dev(a) for a in cols]), [pow(v, e[k], n[j]) for v, (j, k) in zip(x, pick)], limbs)


@pytest.mark.parametrize("limbs,count", [(32, 50), (32, 16 * 130), (48, 16 * 128), (48, 16 * 128 + 5), (64, 16 * 128),
                                         (64, 16 * 256 + 5), (64, 16 * 512 + 5), (96, 33), (96, 16 * 128 + 5),
                                         (128, 33), (128, 16 * 128 + 5)])
def test_crt_launch_shapes(limbs, count):
    """Keys with p and q of any odd numbers: the call exponentiates modulo each
    and recombines, whatever their factors, so moduli that share a factor with
    base A and short ones are among them."""
    rng = random.Random(limbs * 7 + count)
    h = limbs // 2
    words, bits = min(w for w in CLASSES if w >= h), 32 * (limbs // 2)
    keys = []
    while len(keys) < 6:
        p, q = odd(rng, bits), odd(rng, bits)
        if len(keys) == 2:
            p = base_multiple(rng, words, bits)
        elif len(keys) == 3:
            q = base_multiple(rng, words, bits - 3)
        elif len(keys) == 4:
            p, q = odd(rng, 100), odd(rng, 90)
        p, q = max(p, q), min(p, q)
        if math.gcd(p, q) == 1:
            keys.append((p, q, rng.getrandbits(90), rng.getrandbits(70), pow(q, -1, p)))
    key_of = [rng.randrange(6) if i % 5 else i // 40 % 6 for i in range(count)]
    c = [rng.randrange(keys[k][0] * keys[k][1]) for k in key_of]

    def crt(v, k):
        p, q, dp, dq, qinv = keys[k]
        mp, mq = pow(v, dp, p), pow(v, dq, q)
        return mq + q * ((mp - mq) * qinv % p)

    want = [crt(v, k) for v, k in zip(c, key_of)]
    cols = [W.ints_to_limbs([k[i] for k in keys], h)[key_of] for i in range(5)]
    for i, (p, q) in {1: (0, 1), 7: (1, 0)}.items():      # p = q, p even
        cols[0][i], cols[1][i] = (cols[1][i], cols[1][i]) if p == 0 else (cols[0][i] & ~np.uint32(1), cols[1][i])
        want[i] = 0
    ops = [dev(a) for a in cols]
    cd = dev(W.ints_to_limbs(c, limbs))
    rsagpu.device_errors()
    check(rsagpu.decrypt_crt(cd, *ops), want, limbs)
    assert rsagpu.device_errors() == 2
    check(rsagpu.decrypt_crt(cd, *ops, out=cd), want, limbs)
    assert rsagpu.device_errors() == 2


# buckets of a few tiles, of more tiles than half the CUs, and of a bulk batch
@pytest.mark.parametrize("per_class,inplace", [(20, True), (2200, False), (4000, True)])
def test_ops_buckets(per_class, inplace):
    """CRT decryptions under resident keys whose primes are any odd numbers: of
    every RNS class, some narrower than their class, some sharing a factor with
    base A, small runs that leave tiles with empty slots; in place and not."""
    rng = random.Random(per_class)
    ks, keys = rsagpu.KeySet(32), []
    for h in (13, 16, 24, 29, 32, 48, 64):
        words, bits = min(w for w in CLASSES if w >= h), 32 * h
        for j in range(3):
            while True:
                p, q = odd(rng, bits), odd(rng, bits)
                if j == 1:
                    q = base_multiple(rng, words, bits - 2)
                p, q = max(p, q), min(p, q)
                if math.gcd(p, q) == 1 and p != q:
                    break
            key = (p, q, rng.getrandbits(70), rng.getrandbits(90), pow(q, -1, p))
            keys.append((2 * h, key))
            assert ks.add(2 * h, p * q, 65537, *key) == len(keys) - 1
    kids = [k for j in range(0, len(keys), 3) for k in
            [j] * (per_class - 3) + [j + 1] * 2 + [j + 2]][:]
    rng.shuffle(kids)
    ins, want, offs, kinds = [], [], [], []
    at = 0
    for k in kids:
        limbs, (p, q, dp, dq, qinv) = keys[k]
        v = rng.randrange(p * q)
        enc = rng.random() < 0.1
        if enc:
            r = pow(v, 65537, p * q)
        else:
            mp, mq = pow(v, dp, p), pow(v, dq, q)
            r = mq + q * ((mp - mq) * qinv % p)
        ins.append(W.int_to_limbs(v, limbs))
        want.append(W.int_to_limbs(r, limbs))
        offs.append(at)
        kinds.append(0 if enc else 1)
        at += limbs
    pool = dev(np.concatenate(ins))
    out = pool if inplace else torch.zeros_like(pool)
    ops = rsagpu.pack_ops(kinds, kids, offs, offs).cuda()
    ws = torch.empty(rsagpu.ops_workspace_size(len(kids)), dtype=torch.uint8, device="cuda")
    rsagpu.device_errors()
    rsagpu.ops_batch(ks, ops, pool, out, ws)
    got = host(out)
    bad = [i for i, (o, w) in enumerate(zip(offs, want)) if not np.array_equal(got[o:o + len(w)], w)]
    assert not bad, "%d of %d differ, first %d (key %d)" % (len(bad), len(kids), bad[0], kids[bad[0]])
    assert rsagpu.device_errors() == 0

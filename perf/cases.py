"""Performance cases: the work a program has the library do, over its range.

Each case is one call of a public entry point of ``rsagpu`` on inputs that
are resident on the GPU:

* ``crt``     ``decrypt_crt``: RSA decryption (or signing) by CRT;
* ``modexp``  ``modexp``: encryption (verification) with a public exponent,
  plain full-exponent decryption, and modular exponentiations with a modulus
  and an exponent of their own per element, as Miller-Rabin rounds of key
  generation make them;
* ``ops``     ``ops_batch``: a mixed batch of encryptions and CRT decryptions
  under resident keys of several sizes.

Keys are built from a fixed pool of primes (pairs of it, drawn by the seed),
messages are drawn by the seed, and ciphertexts are encryptions of drawn
messages, so that every decryption's exact result is known.
"""
import random

import numpy as np
import torch

from paper_1407_1465_amd import rsagpu

E = 65537

# Primes: prime k of a size is 2 * offset above the odd number that
# random.Random("prime <bits>/<k>") draws with its two top bits set (every
# prime p has gcd(65537 * 131, p - 1) = 1).
PRIME_OFFSETS = {
    2048: (767, 228, 216, 552, 221, 1380, 1648, 2330, 175, 37, 1344, 368),
    1536: (983, 71, 508, 824, 270, 284, 83, 88, 217, 245, 162, 531),
    1024: (76, 40, 1256, 495, 718, 44, 982, 38, 467, 1456, 183, 593, 370, 98, 327, 202, 330, 425, 101, 102, 501, 145,
           603, 948),
    768: (426, 10, 66, 197, 759, 353, 1070, 209, 13, 68, 446, 98),
    512: (87, 120, 73, 160, 354, 257, 11, 177, 125, 479, 195, 129, 45, 119, 17, 534, 305, 21, 40, 369, 61, 76, 62,
          119),
    256: (100, 192, 51, 130, 15, 8, 123, 190, 21, 53, 22, 12),
    32: (22, 9, 15, 26, 0, 25, 13, 13, 3, 4, 14, 5),
}


def _primes(bits):
    return [(random.Random("prime %d/%d" % (bits, k)).getrandbits(bits) | 3 << (bits - 2) | 1) + 2 * off
            for k, off in enumerate(PRIME_OFFSETS[bits])]


def _keys(bits, count, rng):
    """`count` distinct keys with a bits-bit modulus, pairs of the prime pool."""
    ps = _primes(bits // 2)
    pairs = [(a, b) for i, a in enumerate(ps) for b in ps[:i]]
    out = []
    for p, q in rng.sample(pairs, count):
        p, q = max(p, q), min(p, q)
        d = pow(E, -1, (p - 1) * (q - 1))
        out.append({"n": p * q, "e": E, "d": d, "p": p, "q": q, "dp": d % (p - 1), "dq": d % (q - 1),
                    "qinv": pow(q, -1, p)})
    return out


def _pairs(key, e, count, rng):
    """`count` messages below n and their encryptions, a message of which is
    a random start times the powers of a random factor (so are the
    encryptions: two products each instead of an exponentiation)."""
    n = key["n"]
    m, g = rng.randrange(n), rng.randrange(1, n)
    c, gc = pow(m, e, n), pow(g, e, n)
    ms, cs = [], []
    for _ in range(count):
        ms.append(m)
        cs.append(c)
        m, c = m * g % n, c * gc % n
    return ms, cs


def _words(values, limbs):
    buf = b"".join(v.to_bytes(4 * limbs, "little") for v in values)
    return np.frombuffer(buf, dtype="<i4").reshape(len(values), limbs).copy()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# ---- the cases ----------------------------------------------------------------

# Sizes of a mixed batch, in the order of its fields n1024 .. n4096.
SIZES = (1024, 2048, 3072, 4096)


def listed():
    return [
        # The paper's own experiment: one-word modulus, e = 131, messages of
        # 0..800, its largest data size.  Smallest numbers, launch-bound.
        {"name": "paper_word", "path": "modexp", "exp": "paper", "bits": 15, "keys": 1, "count": 32768},
        # 64-bit modulus, full-length private exponent, one key.
        {"name": "rsa64_full", "path": "modexp", "exp": "d", "bits": 64, "keys": 1, "count": 4096},
        # A server's single handshake burst: a few 2048-bit private-key
        # operations under one key, where the latency of one chain counts.
        {"name": "crt2048_few", "path": "crt", "bits": 2048, "keys": 1, "count": 5},
        # The headline batch: 2048-bit CRT decryption under 64 keys.
        {"name": "crt2048_bulk", "path": "crt", "bits": 2048, "keys": 64, "count": 16384},
        # 4096-bit CRT decryptions, as many as a mixed batch holds: few long chains.
        {"name": "crt4096_mid", "path": "crt", "bits": 4096, "keys": 16, "count": 1092},
        # A ragged batch of 3072-bit keys, messages not a multiple of the keys.
        {"name": "crt3072_ragged", "path": "crt", "bits": 3072, "keys": 11, "count": 777},
        # 1024-bit CRT decryptions.
        {"name": "crt1024_mid", "path": "crt", "bits": 1024, "keys": 16, "count": 8000},
        # Public-key operations of the headline's size, e = 65537.
        {"name": "enc2048_bulk", "path": "modexp", "exp": "e", "bits": 2048, "keys": 64, "count": 16384},
        # Full-exponent decryption without CRT, one 1024-bit key.
        {"name": "full1024_bulk", "path": "modexp", "exp": "d", "bits": 1024, "keys": 1, "count": 65536},
        # One Miller-Rabin round over the candidates of a key generation:
        # every element its own odd modulus and its own full-length exponent.
        {"name": "mr2048_own", "path": "modexp", "exp": "own", "bits": 2048, "keys": 1, "count": 200},
        # A serving batch of resident 2048/4096-bit keys, most of it decryptions.
        {"name": "ops_serve", "path": "ops", "keys": 12, "n1024": 0, "n2048": 611, "n3072": 0, "n4096": 153,
         "decrypt": 0.7},
        # The bulk mixed batch: 32768 operations over 1024..4096-bit keys in
        # the ratio 4:8:2:1, half encryptions and half CRT decryptions.
        {"name": "ops_mixed", "path": "ops", "keys": 16, "n1024": 8738, "n2048": 17476, "n3072": 4369, "n4096": 2185,
         "decrypt": 0.5},
    ]


def _logint(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["crt", "crt", "crt", "enc", "full", "own", "ops", "small"])
    if kind == "small":
        if rng.random() < 0.5:
            return {"path": "modexp", "exp": "paper", "bits": 15, "keys": 1, "count": _logint(rng, 256, 32768)}
        return {"path": "modexp", "exp": rng.choice(["d", "e"]), "bits": 64, "keys": rng.randint(1, 8),
                "count": _logint(rng, 64, 8192)}
    if kind == "ops":
        t = _logint(rng, 64, 24000)
        w = [rng.random() for _ in SIZES]
        c = [int(t * x / sum(w)) for x in w]
        c = [min(v, m) for v, m in zip(c, (8738, 17476, 4369, 2185))]
        return {"path": "ops", "keys": rng.randint(1, 16), "n1024": c[0], "n2048": c[1] + 1, "n3072": c[2],
                "n4096": c[3], "decrypt": round(rng.uniform(0.3, 0.8), 2)}
    if kind == "crt":
        bits = rng.choice([512, 1024, 1536, 2048, 2048, 3072, 4096])
        hi = {512: 20000, 1024: 16384, 1536: 12000, 2048: 16384, 3072: 2500, 4096: 1092}[bits]
        return {"path": "crt", "bits": bits, "keys": rng.randint(1, 40), "count": _logint(rng, 1, hi)}
    if kind == "enc":
        bits = rng.choice([1024, 2048, 3072, 4096])
        return {"path": "modexp", "exp": "e", "bits": bits, "keys": rng.randint(1, 40),
                "count": _logint(rng, 16, 16384 * 2048 // max(bits, 2048))}
    bits = rng.choice([512, 1024, 1536, 2048])
    if kind == "full":
        hi = {512: 20000, 1024: 20000, 1536: 6000, 2048: 4000}[bits]
        return {"path": "modexp", "exp": "d", "bits": bits, "keys": rng.randint(1, 16), "count": _logint(rng, 1, hi)}
    return {"path": "modexp", "exp": "own", "bits": bits, "keys": 1, "count": _logint(rng, 1, 400)}


def _host(case, seed):
    """The case's inputs as Python integers, and what a pass gives for them."""
    rng = random.Random(seed)
    if case["path"] == "ops":
        ops, keys = [], []
        for bits in SIZES:
            cnt = case["n%d" % bits]
            if not cnt:
                continue
            first = len(keys)
            ks = _keys(bits, min(case["keys"], len(PRIME_OFFSETS[bits // 2])), rng)
            keys += [dict(k, limbs=bits // 32) for k in ks]
            per = [cnt // len(ks) + (j < cnt % len(ks)) for j in range(len(ks))]
            for j, k in enumerate(ks):
                for m, c in zip(*_pairs(k, E, per[j], rng)):
                    dec = rng.random() < case["decrypt"]
                    ops.append((1 if dec else 0, first + j, bits // 32, c if dec else m, m if dec else c))
        rng.shuffle(ops)
        return keys, ops
    count, bits = case["count"], case["bits"]
    if case["path"] == "modexp" and case["exp"] == "own":
        bases, exps, mods = [], [], []
        for _ in range(count):
            n = rng.getrandbits(bits) | 3 << (bits - 2) | 1
            bases.append(rng.randrange(2, n - 1))
            exps.append((n - 1) >> ((n - 1) & (1 - n)).bit_length() - 1)
            mods.append(n)
        return bases, exps, mods
    if case["path"] == "modexp" and case["exp"] == "paper":
        n, e = 131 * 137, 131
        return [rng.randint(0, 800) for _ in range(count)], [e] * count, [n] * count
    keys = _keys(bits, min(case["keys"], count), rng)
    key_of = [i % len(keys) for i in range(count)]
    per = [_pairs(k, E, key_of.count(j), rng) for j, k in enumerate(keys)]
    ms = [per[j][0][i // len(keys)] for i, j in enumerate(key_of)]
    cs = [per[j][1][i // len(keys)] for i, j in enumerate(key_of)]
    return keys, key_of, ms, cs


def prepare(case, seed):
    if case["path"] == "ops":
        keys, ops = _host(case, seed)
        ks = rsagpu.KeySet(len(keys))
        for k in keys:
            ks.add(k["limbs"], k["n"], k["e"], k["p"], k["q"], k["dp"], k["dq"], k["qinv"])
        offs = np.concatenate([[0], np.cumsum([o[2] for o in ops])])
        pool = np.concatenate([_words([o[3]], o[2])[0] for o in ops])
        return {"path": "ops", "ks": ks,
                "ops": rsagpu.pack_ops([o[0] for o in ops], [o[1] for o in ops], offs[:-1], offs[:-1]).cuda(),
                "in": _dev(pool), "out": torch.zeros(int(offs[-1]), dtype=torch.int32, device="cuda"),
                "ws": torch.empty(rsagpu.ops_workspace_size(len(ops)), dtype=torch.uint8, device="cuda")}
    limbs = (case["bits"] + 31) // 32
    if case["path"] == "modexp" and case["exp"] in ("own", "paper"):
        return {"path": "modexp", "args": [_dev(_words(v, limbs)) for v in _host(case, seed)]}
    keys, key_of, ms, cs = _host(case, seed)

    def column(attr, width):
        return _dev(_words([k[attr] for k in keys], width)[key_of])

    if case["path"] == "modexp":
        base = cs if case["exp"] == "d" else ms
        return {"path": "modexp", "args": [_dev(_words(base, limbs)), column(case["exp"], limbs), column("n", limbs)]}
    return {"path": "crt", "args": [_dev(_words(cs, limbs))] +
            [column(a, limbs // 2) for a in ("p", "q", "dp", "dq", "qinv")]}


def run(state):
    if state["path"] == "ops":
        rsagpu.ops_batch(state["ks"], state["ops"], state["in"], state["out"], state["ws"])
        return state["out"]
    if state["path"] == "crt":
        return rsagpu.decrypt_crt(*state["args"])
    return rsagpu.modexp(*state["args"])


def exact(case, seed):
    host = _host(case, seed)
    if case["path"] == "ops":
        return torch.from_numpy(np.concatenate([_words([o[4]], o[2])[0] for o in host[1]]))
    limbs = (case["bits"] + 31) // 32
    if case["path"] == "modexp" and case["exp"] in ("own", "paper"):
        return torch.from_numpy(_words([pow(*v) for v in zip(*host)], limbs))
    _, _, ms, cs = host
    want = cs if case["path"] == "modexp" and case["exp"] == "e" else ms
    return torch.from_numpy(_words(want, limbs))


def _products(limbs, ebits):
    """32x32-bit products of one exponentiation: the best fixed-window count
    of Montgomery products, 2 s^2 + s each (17 squarings and products for a
    public exponent)."""
    mont = 2 * limbs * limbs + limbs
    if ebits <= 17:
        return 19 * mont
    return mont * min((-(-ebits // w) - 1) * (w + 1) + 2 ** w for w in range(1, 9))


def _crt_products(limbs):
    h = limbs // 2
    return 2 * (h * h + h + _products(h, 32 * h)) + 3 * h * h + h


def work(case):
    if case["path"] == "ops":
        nbytes = prods = 0
        for bits in SIZES:
            n, limbs = case["n%d" % bits], bits // 32
            dec = n * case["decrypt"]
            nbytes += n * (24 + 8 * limbs) + min(case["keys"], n) * 9 * limbs * 2
            prods += dec * _crt_products(limbs) + (n - dec) * _products(limbs, 17)
        return {"bytes": nbytes, "flops": 2 * prods}
    limbs, n = (case["bits"] + 31) // 32, case["count"]
    if case["path"] == "crt":
        return {"bytes": 4 * n * (2 * limbs + 5 * (limbs // 2)), "flops": 2 * n * _crt_products(limbs)}
    ebits = {"e": 17, "paper": 8}.get(case["exp"], case["bits"])
    return {"bytes": 4 * n * 4 * limbs, "flops": 2 * n * _products(limbs, ebits)}

"""The way in of plain exponentiation (short exponents, which end there, and
full ones) for moduli of every length below their width: the moves of one up to
the width's limbs, as many as the wave's shortest modulus takes, at lengths
around each move's 28 bits; on narrow groups and on wide ones (more than 4096
elements, by the number of lanes)."""
import random

import numpy as np
import pytest

from paper_1407_1465_amd import workloads as W
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1407_1465_amd import rsagpu  # noqa: E402


@pytest.mark.parametrize("limbs", [13, 15, 16, 17, 24, 25, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("count", [150, 16600])
def test_moduli_of_any_length(limbs, count):
    if count > 4096 and limbs > 48:
        count = 4096                          # the RNS path's largest batch there
    assert rsagpu.get_path(limbs, 0, min(count, 4096)) == rsagpu.PATH_RNS
    rng = random.Random(limbs * 10 + (count > 200))
    bits = 32 * limbs
    lengths = [bits - d for d in range(12)] + [b + d for b in range(bits - 28, 2, -28) for d in (0, 1)] + [2, 3, 40]
    mods = [rng.getrandbits(b) | 1 | 1 << (b - 1) for b in lengths for _ in range(2)]
    mods[:4] = [(1 << bits) - 1, (1 << (bits - 1)) + 1, (1 << (bits - 28)) - 1, 3]
    exps = [65537, 3, 1, 0, (1 << 64) - 1, rng.getrandbits(64) | 1 << 63, rng.getrandbits(66) | 1 << 65]
    # runs of one length, and lengths mixed within a wave
    pick = [(i // 40 % len(mods) if i % 80 < 40 else rng.randrange(len(mods)), i // 16 % 7 if i % 3 else 0)
            for i in range(count)]
    x = [rng.getrandbits(bits) for _ in range(count)]
    cols = [W.ints_to_limbs(x, limbs), W.ints_to_limbs(exps, limbs)[[k for _, k in pick]],
            W.ints_to_limbs(mods, limbs)[[j for j, _ in pick]]]
    got = host(rsagpu.modexp(*[dev(a) for a in cols]))
    want = W.ints_to_limbs([pow(v, exps[k], mods[j]) for v, (j, k) in zip(x, pick)], limbs)
    bad = np.nonzero((got != want).any(axis=1))[0]
    assert bad.size == 0, "%d of %d differ, first %d (modulus of %d bits)" % (
        bad.size, count, bad[0], mods[pick[bad[0]][0]].bit_length())
    assert rsagpu.device_errors() == 0

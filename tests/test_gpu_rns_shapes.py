"""Launch rules of the RNS calls, both sides of each that the sizes of
test_gpu_rns.py leave out: three waves to a tile (2048-bit keys), the batch
sizes at which 512-bit and 2048-bit moduli go to the positional kernels, a
processing order of three rounds of tiles, and both shapes of an ops bucket by
its size."""
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
import test_gpu_rns as rns  # noqa: E402

CUS = torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("limbs,tiles,more", [(64, 200, 0), (32, 2 * CUS, 0), (32, 2 * CUS, 1), (48, CUS, 0),
                                              (128, 384, 0), (96, 3 * CUS, -7)])
def test_crt(limbs, tiles, more):
    rns.test_crt_launch_shapes(limbs, 16 * tiles + more)


@pytest.mark.parametrize("limbs,tiles,more", [(16, 4 * CUS, 0), (16, 4 * CUS, 1), (64, CUS, 0), (64, CUS, 1)])
def test_modexp(limbs, tiles, more):
    rns.test_modexp_launch_shapes(limbs, 16 * tiles + more)


@pytest.mark.parametrize("h,count", [(h, n) for h in (24, 32, 48) for n in (16 * (CUS // 2), 16 * (CUS // 2) + 1, 5000)])
def test_ops_bucket_by_its_size(h, count):
    """One key, so a bucket of whole tiles but the last; the batch is no bulk one."""
    rng = random.Random(h + count)
    p, q = sorted((rng.getrandbits(32 * h) | 1 | 1 << (32 * h - 1) for _ in range(2)), reverse=True)
    dp, dq, qinv = rng.getrandbits(80), rng.getrandbits(77), rng.randrange(p)
    ks = rsagpu.KeySet(1)
    ks.add(2 * h, p * q, 65537, p, q, dp, dq, qinv)
    c = [rng.randrange(p * q) for _ in range(count)]

    def crt(v):
        mp, mq = pow(v, dp, p), pow(v, dq, q)
        return mq + q * ((mp - mq) * qinv % p)
    offs = np.arange(count, dtype=np.int64) * 2 * h
    pool = dev(W.ints_to_limbs(c, 2 * h).reshape(-1))
    out = torch.zeros_like(pool)
    ws = torch.empty(rsagpu.ops_workspace_size(count), dtype=torch.uint8, device="cuda")
    rsagpu.ops_batch(ks, rsagpu.pack_ops([1] * count, [0] * count, offs, offs).cuda(), pool, out, ws)
    got = host(out).reshape(count, 2 * h)
    bad = np.nonzero((got != W.ints_to_limbs([crt(v) for v in c], 2 * h)).any(axis=1))[0]
    assert bad.size == 0, "%d of %d differ, first %d" % (bad.size, count, bad[0])

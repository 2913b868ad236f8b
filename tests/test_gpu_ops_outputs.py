"""Operations of one batch that name the same output range (a batch filled up
with copies of an operation, its input elsewhere): every output is the
operation's result, however many rounds of tiles the copies take.  And
the same batch in a workspace that holds the bucket lists alone."""
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

HALVES = (13, 24, 32, 48, 64)
LISTS_ALONE = 33024, 128                      # workspace bytes without the words between kernels: header, per operation


@pytest.mark.parametrize("copies", [1, 40, 800, 3500])
@pytest.mark.parametrize("lists_alone", [False, True])
def test_copies_of_an_operation(copies, lists_alone):
    rng = random.Random(copies)
    ks, ops, ins, outs, at = rsagpu.KeySet(8), [], [], [], 0
    for j, h in enumerate(HALVES):
        p, q = sorted((rng.getrandbits(32 * h) | 1 | 1 << (32 * h - 1) for _ in range(2)), reverse=True)
        dp, dq = rng.getrandbits(70), rng.getrandbits(66)
        qinv = rng.randrange(p)
        ks.add(2 * h, p * q, 65537, p, q, dp, dq, qinv)
        c = rng.randrange(p * q)
        mp, mq = pow(c, dp, p), pow(c, dq, q)
        outs.append(W.int_to_limbs(mq + q * ((mp - mq) * qinv % p), 2 * h))
        ins.append(W.int_to_limbs(c, 2 * h))
        ops += [(1, j, at, at)] * copies
        at += 2 * h
    rng.shuffle(ops)
    desc = rsagpu.pack_ops(*zip(*ops)).cuda()
    pool, want = dev(np.concatenate(ins)), dev(np.concatenate(outs))
    out = torch.zeros_like(pool)
    size = LISTS_ALONE[0] + LISTS_ALONE[1] * len(ops) if lists_alone else rsagpu.ops_workspace_size(len(ops))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        out.zero_()
        rsagpu.ops_batch(ks, desc, pool, out, ws)
        got, exp = host(out), host(want)
        bad = np.nonzero(got != exp)[0]
        assert bad.size == 0, "%d of %d words differ, first %d" % (bad.size, len(exp), bad[0])
    assert rsagpu.device_errors() == 0
    with pytest.raises(rsagpu.RSAError):
        rsagpu.ops_batch(ks, desc, pool, out, ws[:LISTS_ALONE[0] + LISTS_ALONE[1] * len(ops) - 1])

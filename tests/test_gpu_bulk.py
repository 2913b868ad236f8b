"""A bulk batch (at least 16384 operations) over keys of every RNS width, with
each number of forks: on a caller's stream, and captured there into a HIP graph
(the forked buckets' events among each other and with the caller) and replayed,
with eager work and synchronisation between the replays; with few decryptions
and with none."""
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

HALVES = (16, 24, 32, 48, 64)
COUNT = 16600


@pytest.fixture(scope="module")
def material():
    rng = random.Random(7)
    keys = []
    for h in HALVES:
        for _ in range(2):
            p, q = sorted((rng.getrandbits(32 * h) | 1 | 1 << (32 * h - 1) for _ in range(2)), reverse=True)
            keys.append((2 * h, p, q, rng.getrandbits(68), rng.getrandbits(66), rng.randrange(p)))
    # a few values under each key and kind; the operations draw from them
    values = []
    for limbs, p, q, dp, dq, qinv in keys:
        vs = [rng.randrange(p * q) for _ in range(40)]
        dec = []
        for v in vs:
            mp, mq = pow(v, dp, p), pow(v, dq, q)
            dec.append(mq + q * ((mp - mq) * qinv % p))
        values.append((W.ints_to_limbs(vs, limbs), W.ints_to_limbs([pow(v, 17, p * q) for v in vs], limbs),
                       W.ints_to_limbs(dec, limbs)))
    return keys, values


def batch(material, share, seed):
    """COUNT operations, a share of them decryptions: descriptors, inputs, outputs."""
    keys, values = material
    rng = random.Random(seed)
    kinds = [1 if rng.random() < share else 0 for _ in range(COUNT)]
    kids = [rng.randrange(len(keys)) for _ in range(COUNT)]
    pick = [rng.randrange(40) for _ in range(COUNT)]
    ins = np.concatenate([values[k][0][v] for k, v in zip(kids, pick)])
    want = np.concatenate([values[k][1 + kd][v] for kd, k, v in zip(kinds, kids, pick)])
    offs = np.concatenate([[0], np.cumsum([keys[k][0] for k in kids])])
    return rsagpu.pack_ops(kinds, kids, offs[:-1], offs[:-1]).cuda(), dev(ins), want


@pytest.mark.parametrize("share", [0.5, 0.001, 0.0])
@pytest.mark.parametrize("forks", [3, 2, 1, 0])
def test_bulk_batch(material, forks, share):
    keys, _ = material
    ks = rsagpu.KeySet(len(keys))
    for limbs, p, q, dp, dq, qinv in keys:
        ks.add(limbs, p * q, 17, p, q, dp, dq, qinv)
    ks.set_forks(forks)
    ops, ins, want = batch(material, share, 1)
    ops2, ins2, want2 = batch(material, 0.4, 2)
    ws, ws2 = (torch.empty(rsagpu.ops_workspace_size(COUNT), dtype=torch.uint8, device="cuda") for _ in range(2))
    out, out2 = torch.zeros_like(ins), torch.zeros_like(ins2)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        rsagpu.ops_batch(ks, ops, ins, out, ws)             # the stream's fork set is made
        s.synchronize()
        assert np.array_equal(host(out), want)
        with torch.cuda.graph(g, stream=s):
            rsagpu.ops_batch(ks, ops, ins, out, ws)
    torch.cuda.current_stream().wait_stream(s)
    for _ in range(3):
        out.zero_()
        out2.zero_()
        g.replay()
        rsagpu.ops_batch(ks, ops2, ins2, out2, ws2)         # eager, on the default stream, beside the replay
        torch.cuda.synchronize()
        assert np.array_equal(host(out), want) and np.array_equal(host(out2), want2)
    del g
    assert rsagpu.device_errors() == 0
    ks.close()

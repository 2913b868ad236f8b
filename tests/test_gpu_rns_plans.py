"""Plans and the RNS kernels: which of the two a call runs, and what the tuner
and plans set meanwhile leave of it."""
import ctypes
import random
import threading

import pytest

from paper_1407_1465_amd import workloads as W
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1407_1465_amd import rsagpu  # noqa: E402


@pytest.fixture
def default_plans():
    yield
    for limbs in (16, 24, 32, 48, 64):
        for kind in range(5):
            rsagpu.set_plan(limbs, kind, 0, 0, 0)


def test_a_plan_set_during_a_call(default_plans):
    """One thread sets and restores the plan that a call in another reads: the
    call takes the one or the other, never the path of one with the window of
    the other (48 words at window 6 would ask for 231 KiB of a workgroup's
    LDS)."""
    count, limbs = 8200, 48
    rng = random.Random(1)
    n = rng.getrandbits(1536) | 1 | 1 << 1535
    x = [rng.getrandbits(1536) for _ in range(count)]
    base, exp, mod = (dev(W.ints_to_limbs(v, limbs)) for v in (x, [3] * count, [n] * count))
    out = torch.empty_like(base)
    lib, stop = rsagpu.raw_lib(), threading.Event()
    rsagpu.modexp(base, exp, mod, out=out)

    def toggle():
        while not stop.is_set():
            lib.rsa_set_plan(limbs, 0, 29, 8, 6)
            lib.rsa_set_plan(limbs, 0, 0, 0, 0)
    t = threading.Thread(target=toggle)
    t.start()
    try:
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        args = [ctypes.c_void_p(a.data_ptr()) for a in (base, exp, mod, out)]
        for i in range(4000):
            assert lib.rsa_modexp_batch(*args, count, limbs, stream) == 0, "call %d" % i
    finally:
        stop.set()
        t.join()
    assert (host(out) == W.ints_to_limbs([pow(v, 3, n) for v in x], limbs)).all()


@pytest.mark.parametrize("kind,count", [(3, 16384), (3, 300), (4, 300), (4, 16384), (1, 300)])
def test_the_tuner_keeps_rns_for_crt(kind, count, default_plans):
    """Kinds 3 and 4 are timed under one another's calls by the batch's size;
    RNS is several times as fast as any plan for 4096-bit keys in all of
    them, and stays."""
    other = {3: 4, 4: 3}.get(kind)
    if other:
        rsagpu.set_plan(64, other, 29, 16, 4)
    rsagpu.autotune(128, kind, 0, count)
    assert rsagpu.get_path(64, kind) == rsagpu.PATH_AUTO
    assert rsagpu.get_path(64, kind, count) == rsagpu.PATH_RNS
    if other:                                 # the plan set before is back, with its path
        p = rsagpu.get_plan(64, other)
        assert (p.lanes_per_op, p.window_bits) == (16, 4) and rsagpu.get_path(64, other) == rsagpu.PATH_POSITIONAL


@pytest.mark.parametrize("exp_bits,count", [(17, 1000), (17, 16384), (0, 200), (0, 5000)])
def test_the_tuner_keeps_rns_for_full_exponents(exp_bits, count, default_plans):
    """A plan found for public exponents, or for a batch beyond RNS's sizes,
    serves those calls; full exponents of a batch within them keep RNS.  All
    are exact, with the window of any plan."""
    rsagpu.autotune(64, 0, exp_bits, count)
    assert rsagpu.get_path(64, 0) == rsagpu.PATH_AUTO
    assert rsagpu.get_path(64, 0, 200) == rsagpu.PATH_RNS
    rng = random.Random(count)
    n = rng.getrandbits(2048) | 1 | 1 << 2047
    x, e = [rng.getrandbits(2048) for _ in range(200)], [rng.getrandbits(70), 65537] * 100
    base, exp, mod = (dev(W.ints_to_limbs(v, 64)) for v in (x, e, [n] * 200))
    want = W.ints_to_limbs([pow(v, k, n) for v, k in zip(x, e)], 64)
    assert (host(rsagpu.modexp(base, exp, mod)) == want).all()


def test_the_tuner_may_find_a_plan_that_beats_rns():
    """Whatever it finds for 512-bit halves, the call runs it and is exact."""
    try:
        rsagpu.autotune(32, 1, 0, 8192)
        path = rsagpu.get_path(16, 1, 8192)
        assert path == (rsagpu.PATH_RNS if rsagpu.get_path(16, 1) == rsagpu.PATH_AUTO else rsagpu.PATH_POSITIONAL)
    finally:
        rsagpu.set_plan(16, 1, 0, 0, 0)


def test_paths_by_batch_size():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    P, R = rsagpu.PATH_POSITIONAL, rsagpu.PATH_RNS
    for limbs, kind, last in ((16, 0, 64 * cus), (13, 0, 64 * cus), (16, 1, 32 * cus), (64, 0, 16 * cus),
                              (49, 0, 16 * cus)):
        assert rsagpu.get_path(limbs, kind, last) == R and rsagpu.get_path(limbs, kind, last + 1) == P, (limbs, kind)
    for limbs, kind in ((24, 0), (32, 0), (48, 0), (24, 1), (32, 1), (48, 1), (64, 1), (16, 3), (64, 4)):
        assert rsagpu.get_path(limbs, kind, 1) == R and rsagpu.get_path(limbs, kind, 1 << 20) == R
    for limbs, kind in ((12, 0), (12, 1), (65, 0), (128, 0), (12, 3), (64, 2)):
        assert rsagpu.get_path(limbs, kind, 100) == P

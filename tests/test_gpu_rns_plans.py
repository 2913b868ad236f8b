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

"""The positional kernels of the widths that run in RNS by default, under
default plans with the path set to positional: the tests of those widths' plain
and CRT calls, key orders, workgroup shapes and bulk batches, run on them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1407_1465_amd import rsagpu  # noqa: E402
import test_gpu_keyset as keyset  # noqa: E402
import test_gpu_parity as parity  # noqa: E402
import test_gpu_rns as rns  # noqa: E402
import test_zz_no_alloc as static  # noqa: E402


@pytest.fixture(autouse=True)
def positional():
    slots = [(w, k) for w in (16, 24, 32, 48, 64) for k in (0, 1, 3, 4)]
    for w, k in slots:
        rsagpu.set_path(w, k, rsagpu.PATH_POSITIONAL)
    assert all(rsagpu.get_path(w, k, 100) == rsagpu.PATH_POSITIONAL for w, k in slots)
    yield
    for w, k in slots:
        rsagpu.set_path(w, k, rsagpu.PATH_AUTO)


@pytest.mark.parametrize("limbs", [13, 16, 24, 32, 48, 64])
@pytest.mark.parametrize("shared", [False, True])
def test_modexp_edges(limbs, shared):
    rns.test_modexp_edges(limbs, shared)


# more than a round of two waves per SIMD at 64 words
@pytest.mark.parametrize("limbs,count", [(16, 3000), (32, 3000), (48, 3000), (64, 16700)])
def test_modexp_batches(limbs, count):
    rns.test_modexp_launch_shapes(limbs, count)


# one pair of waves a workgroup, two by the batch's size (2 lanes) and by the
# lanes (8 and 16), several workgroups and a ragged last one
@pytest.mark.parametrize("limbs,count", [(32, 8736), (48, 2053), (64, 50), (64, 8197), (96, 33), (96, 2053), (128, 33),
                                         (128, 2053)])
def test_crt(limbs, count):
    rns.test_crt_launch_shapes(limbs, count)


@pytest.mark.parametrize("bits,count", [(1024, 90), (2048, 70), (3072, 45), (4096, 45)])
def test_crt_vs_oracle(bits, count):
    parity.test_crt_vs_oracle_plain_decrypt(bits, count)


@pytest.mark.parametrize("per_class,inplace", [(20, True), (2200, False), (4000, True)])
def test_ops(per_class, inplace):
    rns.test_ops_buckets(per_class, inplace)


def test_mixed_workload():
    keyset.test_workload_mixed_sizes_full()


def test_crt_orders():
    """Key runs of any length, keys that share a hash bucket, data errors."""
    for bits, runs in next(m.args[1] for m in parity.test_crt_key_runs_of_any_length.pytestmark
                           if m.name == "parametrize"):
        if bits >= 1024:
            parity.test_crt_key_runs_of_any_length(bits, runs)
    parity.test_crt_keys_whose_buckets_meet()
    parity.test_crt_grouped_by_key_with_data_errors(2048)
    parity.test_crt_two_pair_workgroups_for_two_lane_halves()


def test_headline_workload():
    parity.test_workload_rsa2048_crt_full_size()


@pytest.mark.parametrize("args", [(2048, 5, 1093, 301, 6148), (1024, 3, 517, 40, 5124),
                                  (4096, 16, 203, 37, static.W.SEED_BASE + 4)])
def test_static_call(args):
    static.test_static_entry_point_equals_allocating_one(*args)

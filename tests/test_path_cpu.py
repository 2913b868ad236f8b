"""Which kernels a class's calls take (rsa_set_path, rsa_get_path) on a host
without a GPU: plans set by the caller, the default, cached plans and the batch
tuner's starting state."""
import json

import pytest

from paper_1407_1465_amd import rsagpu, tune

AUTO, POSITIONAL, RNS = rsagpu.PATH_AUTO, rsagpu.PATH_POSITIONAL, rsagpu.PATH_RNS


def plan_of(width, kind):
    p = rsagpu.get_plan(width, kind)
    return (p.radix_bits, p.lanes_per_op, p.window_bits)


@pytest.fixture(autouse=True)
def default_plans():
    yield
    for kind in (0, 1, 3, 4):
        for width in (32, 64):
            rsagpu.set_plan(width, kind, 0, 0, 0)


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("kind", [0, 1, 3, 4])
def test_a_plan_set_by_the_caller_is_obeyed(width, kind):
    """The default plan too: it names a positional kernel."""
    default = plan_of(width, kind)
    assert rsagpu.get_path(width, kind) == AUTO
    rsagpu.set_plan(width, kind, *default)
    assert plan_of(width, kind) == default and rsagpu.get_path(width, kind) == POSITIONAL
    if kind > 1:
        assert rsagpu.get_path(width, kind, 100) == POSITIONAL
    rsagpu.set_path(width, kind, AUTO)
    assert plan_of(width, kind) == default and rsagpu.get_path(width, kind) == AUTO
    if kind > 1:
        assert rsagpu.get_path(width, kind, 100) == RNS
    rsagpu.set_path(width, kind, POSITIONAL)
    assert rsagpu.get_path(width, kind) == POSITIONAL
    rsagpu.set_plan(width, kind, 0, 0, 0)
    assert plan_of(width, kind) == default and rsagpu.get_path(width, kind) == AUTO


def test_widths_without_rns_and_bad_arguments():
    assert rsagpu.get_path(8, 3, 100) == POSITIONAL and rsagpu.get_path(32, 2, 100) == POSITIONAL
    for bad in ((32, 5, AUTO), (32, 0, RNS), (32, 0, -1), (0, 0, AUTO), (96, 1, AUTO)):
        with pytest.raises(rsagpu.RSAError):
            rsagpu.set_path(*bad)
    for bad in ((32, -1), (129, 0), (96, 3)):
        with pytest.raises(rsagpu.RSAError):
            rsagpu.get_path(*bad)


def test_cached_plans_leave_rns_what_it_serves(tmp_path, monkeypatch):
    """Entries without a path come from a search among positional kernels."""
    monkeypatch.setenv("RSAGPU_TUNE_FILE", str(tmp_path / "plans.json"))
    plan = {"radix_bits": 29, "lanes_per_op": 4, "window_bits": 5, "padded_limbs": 36}
    for entry, want in ((plan, AUTO), (dict(plan, path=AUTO), AUTO), (dict(plan, path=POSITIONAL), POSITIONAL)):
        json.dump({"gfx950/w64/k3/e0/n1024": entry}, open(tune.cache_path(), "w"))
        assert tune.apply_cached("gfx950") == 1
        assert plan_of(32, 3) == (29, 4, 5) and rsagpu.get_path(32, 3) == want


def test_candidate_plans_leave_the_path():
    for path in (AUTO, POSITIONAL):
        rsagpu.set_path(32, 3, path)
        tune.candidate_plans(32, 3)
        assert rsagpu.get_path(32, 3) == path


@pytest.mark.parametrize("kind", [3, 4])
def test_the_batch_tuner_goes_back_to_its_start(kind):
    """With no candidate faster, and with one that loses the final check."""
    slot = (64, kind)
    start = plan_of(*slot)
    chosen, _ = tune.tune_batch(None, [slot], timer=lambda: 10.0)
    assert chosen[slot] == start and plan_of(*slot) == start and rsagpu.get_path(*slot) == AUTO
    calls = {}

    def fickle():
        calls[plan_of(*slot)] = n = calls.get(plan_of(*slot), 0) + 1
        return 9.0 if plan_of(*slot) != start and n < 3 else 10.0
    chosen, _ = tune.tune_batch(None, [slot], timer=fickle)
    assert chosen[slot] == start and plan_of(*slot) == start and rsagpu.get_path(*slot) == AUTO


def test_the_batch_tuner_can_choose_the_start_plan_positionally():
    slot = (64, 3)
    start = plan_of(*slot)

    def timer():
        return 9.0 if plan_of(*slot) == start and rsagpu.get_path(*slot) == POSITIONAL else 10.0
    chosen, ms = tune.tune_batch(None, [slot], timer=timer)
    assert chosen[slot] == start + ("positional",) and ms == 9.0
    assert plan_of(*slot) == start and rsagpu.get_path(*slot) == POSITIONAL

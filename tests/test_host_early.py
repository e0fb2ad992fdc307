"""Kernels of a call that run while the host waits for what validation found, on a runtime that runs none (fake_hip.cpp)."""
import os
import shutil

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(str(tmp_path_factory.mktemp("fake_hip")))


def _hops(kernels):
    return [k for k in kernels if k.startswith("k_hop")]


@pytest.mark.parametrize("P,radix,longest", [(100, 4, 300), (100, 100, 300), (100, 4, 60), (200, 14, 200), (100, 100, 60), (300, 2, 60), (600, 25, 60)])
def test_a_call_finds_its_places_early_once_there_is_memory(runtime, P, radix, longest):
    """And, of up to 512 ranks, the totals of its phases: no partial sums to add up at its end.  (300 ranks, radix 2: more classes than
    the host adds up itself.)"""
    (first, _), (second, _) = fake_hip.run(runtime, "early", [[P, radix, longest, 0, 0]] * 2)
    assert first[-1] == "k_phase_sums" and (second[-1] == "k_phase_sums") == (P > 512)
    assert _hops(first) == _hops(second) and "k_self_copy" not in second
    early = [k for k in second if k.startswith("k_t_places") or k == "k_row_totals"]
    assert len(early) == 1 and (early[0] == "k_row_totals") == (radix == P) == ("k_t_bases" not in second)
    assert second.index(early[0]) == (2 if "k_validate_finish" in second else 1)


def test_places_found_in_memory_that_is_replaced_are_found_again(runtime):
    """The own blocks' layout makes the metadata of long blocks larger than what was there when validation began."""
    (_, _), (kernels, _), (again, _) = fake_hip.run(runtime, "early", [[48, 2, 300, 0, 0], [48, 2, 900000, 0, 0], [48, 2, 900000, 0, 0]])
    assert kernels.count("k_t_places") == 2 and again.count("k_t_places") == 1
    assert _hops(kernels) == _hops(again) == ["k_hop_long"] * 6


@pytest.mark.parametrize("P,radix", [(100, 4), (100, 100), (600, 25)])
def test_a_refused_call_has_ended(runtime, P, radix):
    (_, _), (kernels, done) = fake_hip.run(runtime, "early", [[P, radix, 60, 0, 0], [P, radix, 60, 0, 1]])
    assert any(k.startswith("k_t_places") or k == "k_row_totals" for k in kernels) and not _hops(kernels) and done


@pytest.mark.parametrize("P,radix,before", [(513, 512, [513, 2]), (600, 599, [700, 26]), (100, 99, [100, 4]), (513, 512, None), (400, 399, None)])
def test_a_schedule_of_two_phases_without_t_has_no_places(runtime, P, radix, before):
    """Radix P - 1: every block moves once, so there is nothing to find early."""
    rc, kernels = fake_hip.run(runtime, "no_places", P, radix, before)
    assert rc == 0 and len(_hops(kernels)) == 2 and not [k for k in kernels if k.startswith("k_t_")]


@pytest.mark.parametrize("kind,P,radix", [("one pass", 200, 4), ("pipelined", 100, 4), ("two passes", 100, 4)])
def test_a_call_whose_workspace_is_too_small_has_ended(runtime, kind, P, radix):
    kernels, done = fake_hip.run(runtime, "small_workspace", kind, P, radix)
    assert any(k.startswith("k_t_places") for k in kernels) and not _hops(kernels) and done


@pytest.mark.parametrize("P,radix,noalloc", [(100, 4, False), (100, 100, False), (100, 10, False), (100, 10, True)])
def test_early_kernels_that_were_for_nothing_are_left_out(runtime, P, radix, noalloc):
    """After two calls in a row whose phases had no use for them, until one comes that has."""
    calls = ["direct"] + ["engine"] * 4 + ["direct"] * 2 + ["engine", "direct"] * 2 + ["engine"] * 3 + ["direct"] * 2
    want = [True] + [True] * 2 + [False] * 2 + [False, True] + [True] * 4 + [True] * 2 + [False] + [False, True]
    assert fake_hip.run(runtime, "early_use", P, radix, calls, noalloc) == want


def test_calls_that_launch_none_do_not_count(runtime):
    calls = ["engine", "staged", "staged", "slots", "slots", "direct", "engine", "staged", "engine", "staged", "engine"]
    want = [True] + [False] * 4 + [True] * 2 + [False] + [True] + [False] * 2
    assert fake_hip.run(runtime, "early_use", 100, 4, calls, False) == want


@pytest.mark.parametrize("P,radix,early", [(100, 10, True), (512, 23, True), (512, 500, True), (513, 23, False), (100, 9, False), (100, 2, False), (100, 100, False)])
def test_the_call_that_allocates_nothing_has_them_in_two_phases(runtime, P, radix, early):
    """Up to 512 ranks: it waits for a copy behind them."""
    assert fake_hip.run(runtime, "early_use", P, radix, ["direct"] * 2, True) == [early] * 2


@pytest.mark.parametrize("P,radix", [(600, 25), (600, 2), (300, 2), (100, 4), (512, 512)])
def test_what_early_kernels_look_up_is_the_calls_own(runtime, P, radix):
    """Plans and sizing queries do not wait for a call in flight, and their validation writes the head of the context's status block and the sums
    of the classes behind it: 64 bytes, and 8 for each of 2016.  A kernel ahead of the host may not have run by then."""
    by_kernel, at = fake_hip.run(runtime, "verdict", P, radix)
    assert (at is not None) == by_kernel
    assert at is None or at >= 64 + 8 * 2016

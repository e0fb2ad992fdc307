"""What the host code enqueues, on a runtime that runs it as late as it may (fake_hip.cpp)."""
import os
import shutil

import pytest

import fake_hip

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(str(tmp_path_factory.mktemp("fake_hip")))


@pytest.mark.parametrize("then", ["call", "call elsewhere", "query", "plan"])
@pytest.mark.parametrize("P,radix", [(16, 2), (100, 4), (300, 2)])
def test_places_of_t_are_not_overwritten_on_their_way(runtime, P, radix, then):
    """The places of T's classes go to the device from pinned memory after a call has returned: nothing may write there
    until the copy is done.  (300 ranks: more classes than the host adds up itself.)"""
    assert fake_hip.run(runtime, "upload", P, radix, then) == {"violations": 0}


@pytest.mark.parametrize("plan", [("long", 70, 3), ("long", 20, 20), ("engine", 90, 4)])
@pytest.mark.parametrize("call", [("long", 60, 60), ("long", 64, 2), ("engine", 100, 4)])
def test_a_plan_counts_in_a_status_block_of_its_own(runtime, call, plan):
    """Making a plan does not wait for a call in flight on another stream of the context, whose kernels count in the context's
    status block: k_hop_long moves as many units as stand there."""
    r = fake_hip.run(runtime, "plan_status", *call, *plan)
    assert r["seen"] > 0 and r["shared"] == []


@pytest.mark.parametrize("P,radix", [(16, 16), (100, 4)])
@pytest.mark.parametrize("between", ["nothing", "ranks per node", "no counts", "refused", "empty", "empty start", "profiled start",
                                     "profiled start there", "noalloc", "query"])
def test_a_call_on_another_stream_is_behind_the_one_in_flight(runtime, between, P, radix):
    """They share the context's workspace, whatever was called between them."""
    assert fake_hip.run(runtime, "order", between, P, radix) == {"behind": True}


@pytest.mark.parametrize("t_layout", [0, 1])
@pytest.mark.parametrize("P,size,radix", [(16, 4 << 20, 16), (16, 4 << 20, 2), (64, 300001, 8), (200, 40000, 200)])
def test_a_plan_of_long_blocks_holds_one_list_of_units_per_phase(runtime, P, size, radix, t_layout):
    """16 bytes per 4 KiB of payload and two per block, and with several phases the places in T: 20 bytes per block and phase."""
    r = fake_hip.run(runtime, "plan_bytes", P, size, radix, t_layout)
    phases = r["phases"]
    assert r["meta"] <= phases * (16 * (P * P * size // 4096 + 2 * P * P) + 20 * P * P) + 65536
    assert 0 <= r["said"] + 4096 <= 8192


@pytest.mark.parametrize("plan", [False, True])
@pytest.mark.parametrize("P,radix", [(16, 4), (100, 3)])
def test_no_schedule_is_kept_whose_tables_were_only_recorded(runtime, P, radix, plan):
    """In a capture that allows allocations the kernels that fill a new schedule's tables would not have run."""
    assert fake_hip.run(runtime, "recording", P, radix, plan) == {"refused": True, "tables": 1}


@pytest.mark.parametrize("seed", range(12))
def test_sequences_of_operations(runtime, seed):
    """Every kernel of an immediate call, on whatever stream, is behind all earlier calls of its context."""
    r = fake_hip.run(runtime, "sequence", seed, 120)
    assert r["calls"] > 20 and r["late"] == [] and r["violations"] == 0


@pytest.mark.parametrize("kind", ["large", "far in S", "far in R"])
def test_the_single_launch_is_not_asked_in_vain_for_long(runtime, kind):
    """Problems that it declines, other inputs each time: four times, then not again, until one comes that it would have taken.  Neither a
    call that would not ask it nor one of another schedule is such a one."""
    asked = fake_hip.run(runtime, "single_launch", [[kind, 3]] * 12)
    assert asked == [True] * 4 + [False] * 8
    asked = fake_hip.run(runtime, "single_launch", [[kind, 3]] * 5 + [["own options", 3], ["own options", 2]] + [[kind, 3]] * 2 + [["small", 3]] + [[kind, 3]] * 5)
    assert asked == [True] * 4 + [False] * 6 + [True] * 4 + [False]
    asked = fake_hip.run(runtime, "single_launch", [[kind, 3]] * 5 + [["small", 2]] + [[kind, 3]] * 5)
    assert asked == [True] * 4 + [False] + [True] + [True] * 4 + [False]


@pytest.mark.parametrize("units", [256, 64, 32, 16, 8])
@pytest.mark.parametrize("P,radix", [(512, 23), (300, 2), (65, 8)])
def test_rows_of_validation_lie_in_front_of_the_tables(runtime, units, P, radix):
    """Also where a device shows as few compute units as one of its parts has: what one workgroup writes does not get less."""
    end, tables = fake_hip.run(runtime, "rows_of_validation", units, P, radix)
    assert 0 < end <= tables


@pytest.mark.parametrize("first", ["destroyed", "recorded"])
@pytest.mark.parametrize("plan", [False, True])
@pytest.mark.parametrize("kind", ["direct", "engine", "slots", "staged"])
def test_a_schedule_outlives_the_stream_it_was_made_on(runtime, kind, plan, first):
    """Its tables are in memory of the library's: who uses it next on another stream does not ask for the first one."""
    assert fake_hip.run(runtime, "stream_gone", kind, 100, 4, plan, first) == 0

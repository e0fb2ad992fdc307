"""Which kernels a call or a start launches, on a runtime that runs none (fake_hip.cpp): the statistics name k_hop_direct,
k_hop_senders and k_hop_pairs alike, and not the kernel that finds the places in T.  The problems of the GPU tests of these kernels reach
the kernels that they are there for."""
import os
import shutil

import pytest

import fake_hip
import paper_2411_02581_amd as tuna
import test_gpu_pairs
import test_gpu_t_places

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")
EXACT, SLOTS = 1, 0


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fake_hip.build(str(tmp_path_factory.mktemp("fake_hip")))


def _parameters(test, names):
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names)


def _phases(P, rpn, rl, rg):
    """Rounds, and blocks that a rank sends, of every phase."""
    dims = [(P, rl)] if rpn in (0, 1, P) else [(rpn, rl), (P // rpn, rg)]
    out = []
    for size, r in dims:
        r, x = min(r, size), 1
        while x < size:
            out.append((min(r - 1, (size - 1) // x), sum(v // x % r > 0 for v in range(size)) * (P // size)))
            x *= r
    return out


def _by_senders(rounds, blocks):
    """Many rounds, up to about 256."""
    return 12 <= rounds <= 1024 and (blocks + 255) // 256 * rounds <= blocks


def _lanes(longest):
    return 1 if longest <= 16 else 4 if longest <= 64 else 16


def test_problems_of_the_linear_schedule_reach_their_kernel(runtime):
    """k_hop_pairs with each number of lanes per block and kind of access, alone: it moves the ranks' own blocks too."""
    names = _parameters(test_gpu_pairs.test_tiles, "longest,quantum,lay_args")
    problems = [(P, 0, P, P, n, q, EXACT, lay) for P in _parameters(test_gpu_pairs.test_tiles, "P") for n, q, lay in names]
    problems += [(P, 0, P, P, n, q, EXACT, {}) for P, n, q in _parameters(test_gpu_pairs.test_several_steps, "P,longest,quantum") if P < 4000]
    seen = set()
    for prob, kernels in zip(problems, fake_hip.run(runtime, "routes", problems, False)):
        assert [k for k, _ in kernels] == ["k_hop_pairs"], prob
        assert kernels[0][1][0] == _lanes(prob[4]), prob
        seen.add(tuple(kernels[0][1]))
    assert seen == {(1, 0), (4, 0), (4, 1), (16, 0), (16, 1), (16, 2)}


def test_problems_of_several_phases_reach_their_kernels(runtime):
    """k_hop_senders from 12 rounds on, k_hop_direct below and where a message has hardly a block (1023 rounds), with the places from k_t_places_slots from radix 8 on, k_t_places
    below."""
    for t_layout in (EXACT, SLOTS):
        problems = [(c[0], c[1], c[2], c[3], c[4], c[5], t_layout, c[7]) for c in test_gpu_t_places.CASES]
        seen, places = set(), set()
        for prob, kernels in zip(problems, fake_hip.run(runtime, "routes", problems, False)):
            P, rpn, rl, rg, longest = prob[:5]
            phases = _phases(P, rpn, rl, rg)
            hops = [(k, a) for k, a in kernels if k.startswith("k_hop")]
            if longest > 256 or (longest > 64 and P * P * longest // 2 > 112 << 20):      # k_hop_rows takes large payloads
                want = ["k_hop_rows"] * len(phases)
            else:
                want = ["k_hop_senders" if _by_senders(*ph) else "k_hop_direct" for ph in phases]
            assert [k for k, _ in hops] == want, prob
            for k, a in hops:
                if k == "k_hop_senders":
                    assert a[0] == _lanes(longest) and a[2] == t_layout, prob
                    seen.add((a[0], a[1]))
            for k, _ in kernels:
                if k in ("k_t_places", "k_t_places_slots"):
                    assert t_layout == EXACT and (k == "k_t_places_slots") == (min(rl, rpn or P) >= 8), prob
                    places.add(k)
        assert seen == {(1, 0), (4, 0), (4, 1), (16, 0), (16, 1), (16, 2)}
        assert places == ({"k_t_places", "k_t_places_slots"} if t_layout == EXACT else set())


@pytest.mark.parametrize("P,kernel", [(8192, "k_t_places_slots"), (8193, "k_t_places")])
def test_places_of_many_ranks(runtime, P, kernel):
    """The slot indices of up to 8192 ranks fit the LDS that k_t_places_slots has."""
    kernels = fake_hip.run(runtime, "routes", [(P, 0, 91, 91, 4, 4, EXACT, {})], False)[0]
    assert [k for k, _ in kernels if k.startswith("k_t_places")] == [kernel]


def test_starts_of_plans_run_the_kernel_that_reads_resolved_blocks(runtime):
    problems = [(130, 0, 130, 130, 60, 4, EXACT, {}), (170, 0, 13, 13, 64, 4, EXACT, {}), (300, 0, 20, 20, 256, 16, SLOTS, {"align": 16})]
    for prob, kernels in zip(problems, fake_hip.run(runtime, "routes", problems, True)):
        assert [k for k, _ in kernels] == ["k_hop_direct"] * len(_phases(prob[0], 0, prob[2], 0)), prob
        assert all(a[-1] == 1 for _, a in kernels), prob


@pytest.mark.parametrize("own_first", [True, False])
def test_own_blocks_go_with_the_first_launch(runtime, own_first):
    """A launch for the ranks' own blocks only where the first phase is by senders and there are no places in T to find, or where
    blocks are longer than 64 KiB."""
    if own_first:
        problems = [(100, 0, 100, 100, 60, 4, EXACT, {}), (100, 0, 4, 4, 60, 4, EXACT, {}), (100, 0, 4, 4, 60, 4, SLOTS, {}),
                    (100, 0, 100, 100, 3000, 4, EXACT, {}), (100, 0, 4, 4, 3000, 4, SLOTS, {}), (170, 0, 13, 13, 60, 4, EXACT, {}),
                    (20, 0, 20, 20, 200000, 4, EXACT, {}), (20, 0, 3, 3, 200000, 4, EXACT, {})]
    else:
        problems = [(170, 0, 13, 13, 60, 4, SLOTS, {})]
    for prob, kernels in zip(problems, fake_hip.run(runtime, "routes", problems, False)):
        assert ("k_self_copy" in [k for k, _ in kernels]) == (not own_first), prob


@pytest.mark.parametrize("longest", [8, 60])
@pytest.mark.parametrize("P,radix", [(1024, 32), (1024, 1023), (1024, 12), (1024, 13), (2048, 46), (2048, 600), (3000, 1500), (1024, 4)])
def test_the_cost_model_prices_blocks_by_the_kernel_that_finds_them(P, radix, longest):
    """Short blocks of several phases cost four times the constant, three times where k_hop_senders finds them."""
    rc, c = tuna.tuna_model_constants(tuna.TUNA_MODE_FUSED)
    assert rc == 0
    phases, payload = _phases(P, 0, radix, 0), P * P * longest // 2
    blocks = sum(n * P for _, n in phases)
    priced = sum(n * P * (3 if _by_senders(z, n) else 4) for z, n in phases)
    want = c[0] + c[1] * len(phases) + c[2] * (len(phases) + 1) * P * P / 1e6 + c[5] * priced / 1e6 + c[6] * payload * blocks / (P * P) / 1e9
    rc, ms = tuna.tuna_predict_ms(P, 0, radix, radix, tuna.TUNA_MODE_FUSED, tuna.TUNA_T_EXACT, payload, longest, 4)
    assert rc == 0 and ms == pytest.approx(want, rel=1e-9)


@pytest.mark.parametrize("plan", [False, True])
def test_tall_tiles_where_neighbouring_segments_have_one_sender_each(runtime, plan):
    """In the order of the slot indices, with T in exact size and in slots, the first phase runs tall tiles from seven rounds on; in message
    order, which batches of rounds need, it does not."""
    problems = [(600, 0, r, r, n, 4, t, {}, o) for r in (7, 8, 9, 12, 13, 25) for n in (16, 60, 200) for t in (EXACT, SLOTS) for o in ({}, {"block_count": 30})]
    for prob, kernels in zip(problems, fake_hip.run(runtime, "routes", problems, plan)):
        hops = [(k, a) for k, a in kernels if k.startswith("k_hop")]
        assert len(hops) > 1, prob
        name, args = hops[0]
        rounds, batches = prob[2] - 1, bool(prob[8])
        assert name == ("k_hop_direct" if plan or batches or rounds < 12 else "k_hop_senders"), prob
        assert (args[3] if name == "k_hop_senders" else args[1]) == (rounds >= 7 and not batches), prob


@pytest.mark.parametrize("plan", [False, True])
def test_short_blocks_keep_the_order_of_the_slot_indices(runtime, plan):
    """Whatever T's layout is: no second schedule is made when validation has told.  Longer blocks with T in slots have one."""
    problems = [(300, 0, r, r, n, 4, t, {"gap": 4}) for r in (4, 20) for n in (16, 200, 1000) for t in (EXACT, SLOTS)]
    for prob, tables in zip(problems, fake_hip.run(runtime, "schedules", problems, plan)):
        assert tables == (2 if prob[6] == SLOTS and prob[4] == 1000 else 1), prob

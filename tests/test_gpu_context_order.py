"""Operations of one context that follow each other without a host synchronisation, on one stream and on several: each
result is that of the same call made alone, with three-stage phases."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0x5A


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


class Prob:
    def __init__(self, tuna, counts, seed, gap=0):
        dev = "cuda:0"
        self.tuna, self.lay = tuna, wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32), gap=gap)
        lay, gen = self.lay, torch.Generator(device=dev)
        gen.manual_seed(seed)
        self.send = torch.empty(lay.send_bytes // 8 + 1, dtype=torch.int64, device=dev).random_(generator=gen)
        self.meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
        self.recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
        assert self.call(4, mode=tuna.TUNA_MODE_STAGED) == 0
        torch.cuda.synchronize()
        self.want = self.recv.clone()

    def args(self):
        sc, sd, rc_, rd = self.meta
        return (self.send, sc, sd, self.recv, rc_, rd, self.lay.P, 0)

    def options(self, **fields):
        o = self.tuna.tuna_opts_init()
        o.mode = self.tuna.TUNA_MODE_FUSED                   # small problems too take the general path
        for k, v in fields.items():
            setattr(o, k, v)
        return o

    def call(self, radix, stream=None, **fields):
        return self.tuna.tuna_alltoallv_ex(None, *self.args(), radix, radix, self.options(**fields), stream)

    def clear(self):
        self.recv.fill_(CANARY)
        torch.cuda.synchronize()

    def ok(self):
        return torch.equal(self.recv, self.want)


def _uniform(P, longest, seed):
    return np.random.default_rng(seed).integers(0, longest // 4 + 1, (P, P)) * 4


@pytest.mark.parametrize("radix", [2, 48])
def test_a_plan_is_made_while_a_call_of_long_blocks_is_in_flight(tuna, radix):
    """Both count the units of their blocks on the device."""
    big, other = Prob(tuna, _uniform(48, 900000, 1), 1), Prob(tuna, _uniform(24, 120000, 2), 2)
    side = torch.cuda.Stream()
    for it in range(6):
        big.clear()
        other.clear()
        print("plan beside a call", radix, it, flush=True)
        assert big.call(radix, side) == 0
        rc, plan = tuna.tuna_alltoallv_init_ex(None, *other.args(), 3, 3, other.options(), None)
        assert rc == 0, tuna.tuna_strerror(rc)
        try:
            st = tuna.tuna_get_stats()                       # the call's
            assert st.hop_kernels == tuna.TUNA_HOP_LONG and st.P == 48
            own = int(np.trace(big.lay.sendcounts))
            assert radix == 2 or st.phase[0].payload_bytes == big.lay.payload_bytes - own
            assert tuna.tuna_start(plan) == 0
            torch.cuda.synchronize()
            assert big.ok() and other.ok(), it
            assert tuna.tuna_get_stats().hop_kernels == tuna.TUNA_HOP_LONG
        finally:
            assert tuna.tuna_plan_free(plan) == 0
    tuna.tuna_release()


@pytest.mark.parametrize("P,radix", [(16, 2), (100, 4), (300, 2)])
def test_calls_that_send_the_places_of_t_to_the_device(tuna, P, radix):
    """Back to back on one stream and with a plan and a sizing query between them, whose validation reads other sums of classes."""
    def counts(k):
        c = _uniform(P, 300, k)
        c[1, P - 2] = c[P - 1, 3] = 70004                    # too long for the kernels that find their blocks themselves
        return c
    a, b = Prob(tuna, counts(1), 1, gap=1), Prob(tuna, 2 * counts(2), 2, gap=1)
    exact = {"t_layout": tuna.TUNA_T_EXACT}
    side = torch.cuda.Stream()
    for it in range(8):
        a.clear()
        b.clear()
        print("places on their way", P, radix, it, flush=True)
        assert a.call(radix, side, **exact) == 0
        if it % 4 == 1:
            assert tuna.tuna_workspace_bytes(b.meta[0], P, 0, radix, radix)[0] == 0
        if it % 4 == 2:
            rc, plan = tuna.tuna_alltoallv_init_ex(None, *b.args(), radix, radix, b.options(**exact), None)
            assert rc == 0 and tuna.tuna_plan_free(plan) == 0
        assert b.call(radix, None if it % 4 == 3 else side, **exact) == 0
        assert tuna.tuna_get_stats().hop_kernels & tuna.TUNA_HOP_ENGINE
        torch.cuda.synchronize()
        assert a.ok() and b.ok(), it
    tuna.tuna_release()


@pytest.mark.parametrize("P,radix", [(48, 2), (48, 48), (300, 2), (300, 300)])
def test_a_call_behind_a_refused_one_on_another_stream(tuna, P, radix):
    """A refused call returns as soon as the host knows that it is: what its validation clears is cleared by then.  The call
    behind it counts its units and bytes there."""
    prob = Prob(tuna, _uniform(P, 900000 if P < 100 else 60000, 3), 3)
    bad = prob.meta[0].clone()
    bad[1, 2] += 4                                           # not the transpose of the receive counts
    sides = [torch.cuda.Stream(), torch.cuda.Stream()]
    totals = None
    for it in range(12):
        prob.clear()
        print("behind a refused call", P, radix, it, flush=True)
        a = list(prob.args())
        a[1] = bad
        assert tuna.tuna_alltoallv_ex(None, *a, radix, radix, prob.options(), sides[it % 2]) == tuna.TUNA_ERR_COUNT_MISMATCH
        assert prob.call(radix, sides[1 - it % 2]) == 0
        st = tuna.tuna_get_stats()
        assert (st.hop_kernels == tuna.TUNA_HOP_LONG) == (P < 100 or radix == 300)
        now = [(st.phase[x].payload_bytes, st.phase[x].staged_bytes) for x in range(st.n_phases)]
        totals = totals or now
        assert now == totals and all(b > 0 for b, _ in now)
        torch.cuda.synchronize()
        assert prob.ok(), it
    tuna.tuna_release()


@pytest.mark.parametrize("P,radix,longest", [(12, 12, 200000), (12, 2, 100000), (9, 3, 300001), (40, 40, 36000), (2, 2, 3000000)])
def test_long_blocks_without_allocations(tuna, P, radix, longest):
    """Two calls in a row: the units of the second are counted from zero again, in memory that still holds the first one's."""
    counts = np.random.default_rng(P).integers(longest // 4, longest + 1, (P, P))
    counts[P - 1, 0], counts[0, 1] = 0, 5
    a, b = Prob(tuna, counts, 1, gap=3), Prob(tuna, counts[::-1].copy(), 2)
    for it in range(3):
        a.clear()
        b.clear()
        print("long blocks, noalloc", P, radix, it, flush=True)
        for p in (a, b):
            rc = tuna.tuna_alltoallv_noalloc(*p.args(), radix, radix)
            assert rc == 0, tuna.tuna_strerror(rc)
            assert tuna.tuna_get_stats().hop_kernels == tuna.TUNA_HOP_LONG
        torch.cuda.synchronize()
        assert a.ok() and b.ok(), it
    tuna.tuna_release()


@pytest.mark.parametrize("radix", [3, 64])
def test_calls_of_long_blocks_back_to_back(tuna, radix):
    """One behind the other on one stream and on two, no host synchronisation between them, behind a call of another hop."""
    a, b, c = Prob(tuna, _uniform(64, 200000, 4), 4), Prob(tuna, _uniform(50, 300000, 5), 5, gap=2), Prob(tuna, _uniform(80, 30, 6), 6)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for it in range(4):
        for p in (a, b, c):
            p.clear()
        print("long blocks back to back", radix, it, flush=True)
        assert c.call(radix, s1) == 0
        assert a.call(radix, s1) == 0
        assert tuna.tuna_get_stats().hop_kernels == tuna.TUNA_HOP_LONG if it % 2 else True
        assert b.call(radix, s2 if it % 2 else s1) == 0
        torch.cuda.synchronize()
        assert a.ok() and b.ok() and c.ok(), it
    tuna.tuna_release()


def test_statistics_of_a_plan_outlive_it(tuna):
    prob, other = Prob(tuna, _uniform(30, 3000, 7), 7), Prob(tuna, _uniform(30, 900, 8), 8)
    assert other.call(3) == 0
    rc, plan = tuna.tuna_alltoallv_init_ex(None, *prob.args(), 3, 3, prob.options(profile=1), None)
    assert rc == 0
    assert tuna.tuna_start(plan) == 0
    before = [(ph.payload_bytes, ph.staged_bytes) for ph in tuna.tuna_get_stats().phase]
    assert tuna.tuna_plan_free(plan) == 0
    assert [(ph.payload_bytes, ph.staged_bytes) for ph in tuna.tuna_get_stats().phase] == before and before[0][0] > 0
    tuna.tuna_release()

"""Phases whose blocks are all short (k_hop_direct) or of up to 64 KiB (k_hop_rows): byte parity with the CPU oracle
at the edges of the lanes (16, 64 and 256 bytes, one byte and one word on either side), of the tiles (15 to 17, 63 to
65, 257 ranks) and of the two tile shapes (few and many blocks per round), with rare blocks of many steps of a wave
among tiny ones and at the longest block that the kernels take (65536 bytes), for byte-, word-, chunk- and line-granular sizes, dense and
gapped receive regions, immediate calls, plans and the call that allocates nothing; the totals per phase equal those
of a plan, which scans them."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0xB7


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


def _counts(P, longest, quantum, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(0, longest // quantum + 1, (P, P)) * quantum
    c[rng.random((P, P)) < 0.2] = 0
    if longest > 8192:                                      # most blocks tiny, a few long ones
        c[rng.random((P, P)) < 0.9] %= 40 // quantum * quantum or quantum
    c[rng.integers(P), rng.integers(P)] = longest          # the longest block there is
    return np.ascontiguousarray(c, dtype=np.int32)


CASES = [(15, 15, 1, 3), (17, 16, 4, 2), (64, 16, 8, 64), (65, 17, 1, 4), (130, 63, 1, 130), (257, 64, 8, 16), (128, 64, 64, 12),
         (129, 65, 1, 2), (63, 255, 1, 8), (200, 256, 4, 200), (144, 240, 16, 12), (96, 256, 128, 4), (66, 257, 1, 66),
         (65, 260, 4, 65), (33, 1000, 1, 3), (144, 1024, 16, 12), (48, 2048, 128, 48), (70, 8191, 1, 8), (31, 9000, 4, 2),
         (72, 65536, 4, 9), (34, 65535, 1, 34), (24, 65540, 4, 5), (20, 65536, 128, 20)]


@pytest.mark.parametrize("t_layout", ["exact", "slots"])
@pytest.mark.parametrize("P,longest,quantum,radix", CASES)
def test_short_and_row_blocks(tuna, P, longest, quantum, radix, t_layout):
    counts = _counts(P, longest, quantum, P * 1000 + longest)
    if quantum >= 64:
        counts[counts > 0] = longest                        # whole blocks: displacements keep the granularity
    for Q in (0, 12 if P == 144 else 0):
        lay = wl.make_layout(counts, gap=8 * (quantum == 4), permute_seed=5 if quantum == 1 else None)
        host = wl.payload_position_hash(longest, lay.send_bytes)
        want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
        assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
        dev = "cuda:0"
        send = torch.from_numpy(host).to(dev)
        recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
        sc, sd, rc_, rd = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
        o = tuna.tuna_opts_init()
        o.mode = tuna.TUNA_MODE_FUSED                       # small problems too take the general path
        o.t_layout = tuna.TUNA_T_EXACT if t_layout == "exact" else tuna.TUNA_T_SLOTS
        totals = []

        def check(what):
            torch.cuda.synchronize()
            bad = np.flatnonzero(recv.cpu().numpy() != want)
            assert bad.size == 0, "%s: %d bytes differ, first at %d" % (what, bad.size, bad[0])
            recv.fill_(CANARY)
            st = tuna.tuna_get_stats()
            totals.append([(st.phase[x].payload_bytes, st.phase[x].staged_bytes) for x in range(st.n_phases)])

        print("short blocks", P, longest, quantum, radix, Q, t_layout, flush=True)
        for _ in range(2):
            rc = tuna.tuna_alltoallv_ex(None, send, sc, sd, recv, rc_, rd, P, Q, radix, radix, o)
            assert rc == 0, tuna.tuna_strerror(rc)
            check("call")
        rc, plan = tuna.tuna_alltoallv_init_ex(None, send, sc, sd, recv, rc_, rd, P, Q, radix, radix, o)
        assert rc == 0, tuna.tuna_strerror(rc)
        try:
            assert tuna.tuna_start(plan) == 0
            check("plan")
        finally:
            tuna.tuna_plan_free(plan)
        assert totals[0] == totals[1] == totals[2]
        if radix == P and Q == 0:
            assert totals[0][0][0] == int(counts.sum()) - int(np.trace(counts))
        rc = tuna.tuna_alltoallv_noalloc(send, sc, sd, recv, rc_, rd, P, Q, radix, radix)
        if rc == tuna.TUNA_ERR_NOALLOC_LIMIT:
            assert lay.payload_bytes > 8 << 20
            continue
        assert rc == 0, tuna.tuna_strerror(rc)
        torch.cuda.synchronize()
        assert np.array_equal(recv.cpu().numpy(), want), "noalloc"


def _staged(lay):
    """Staged bytes of the linear schedule's only phase: every received block's chunks between the 16-byte boundaries
    of R, every rank's share rounded up to a line."""
    n, d = lay.recvcounts.astype(np.int64), lay.rdispls
    chunks = np.where(n > 0, (d % 16 + n + 15) // 16, 0)
    np.fill_diagonal(chunks, 0)
    return int(((chunks.sum(axis=1) + 7) // 8 * 8).sum()) * 16


@pytest.mark.parametrize("radix", [4, 96])
@pytest.mark.parametrize("name", ["normal 1 KiB", "normal 1 KiB chunks", "normal 6 KiB", "Zipf"])
def test_totals_of_call_and_plan_agree(tuna, name, radix):
    """Dense receive regions, where a plan keeps the destination-tiled hop and counts pieces of runs for its units: the
    staged bytes that it reports are the call's all the same."""
    P, dev = 96, "cuda:0"
    counts = {"normal 1 KiB": lambda: wl.counts_normal(P, 3, 1024.0, 256.0, 4),
              "normal 1 KiB chunks": lambda: wl.counts_normal(P, 3, 1024.0, 256.0, 16),
              "normal 6 KiB": lambda: wl.counts_normal(P, 4, 6144.0, 1536.0, 4),
              "Zipf": lambda: wl.counts_zipf(P, 12, 1.2, 16384, 4)}[name]()
    lay = wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32))
    sc, sd, rc_, rd = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    send = torch.zeros(lay.send_bytes, dtype=torch.uint8, device=dev)
    recv = torch.zeros(lay.recv_bytes, dtype=torch.uint8, device=dev)
    o = tuna.tuna_opts_init()
    o.t_layout = tuna.TUNA_T_EXACT

    def totals():
        st = tuna.tuna_get_stats()
        return [(st.phase[x].payload_bytes, st.phase[x].staged_bytes) for x in range(st.n_phases)]

    print("totals of call and plan", name, radix, flush=True)
    assert tuna.tuna_alltoallv_ex(None, send, sc, sd, recv, rc_, rd, P, 0, radix, radix, o) == 0
    call = totals()
    rc, plan = tuna.tuna_alltoallv_init_ex(None, send, sc, sd, recv, rc_, rd, P, 0, radix, radix, o)
    assert rc == 0
    try:
        assert tuna.tuna_start(plan) == 0
        torch.cuda.synchronize()
        assert totals() == call
    finally:
        tuna.tuna_plan_free(plan)
    if radix == P:
        assert call[0][1] == _staged(lay)

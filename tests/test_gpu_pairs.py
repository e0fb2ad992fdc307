"""The linear schedule of short blocks (k_hop_pairs): byte parity with the CPU oracle on both sides of its tiles (8, 16, 32 and
64 ranks), for each number of lanes per block and kind of access, dense, gapped and permuted regions, empty blocks and
ranks; own blocks included; a workgroup's several steps at sizes where it has them.  The totals of the phase are those of
the counts, without the own blocks."""
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


def _staged(lay):
    n, d = lay.recvcounts.astype(np.int64), lay.rdispls
    chunks = np.where(n > 0, (d % 16 + n + 15) // 16, 0)
    np.fill_diagonal(chunks, 0)
    return int(((chunks.sum(axis=1) + 7) // 8 * 8).sum()) * 16


def _run(tuna, counts, radix, lay_args):
    dev, P = "cuda:0", counts.shape[0]
    lay = wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32), **lay_args)
    host = wl.payload_position_hash(P, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    send = torch.from_numpy(host).to(dev)
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    o = tuna.tuna_opts_init()
    o.mode = tuna.TUNA_MODE_FUSED                            # small problems too take the general path
    print("pairs", P, int(counts.max()), radix, lay_args, flush=True)
    for n in range(2):
        rc = tuna.tuna_alltoallv_ex(None, send, meta[0], meta[1], recv, meta[2], meta[3], P, 0, radix, radix, o)
        assert rc == 0, tuna.tuna_strerror(rc)
        torch.cuda.synchronize()
        bad = np.flatnonzero(recv.cpu().numpy() != want)
        assert bad.size == 0, "%d bytes differ, first at %d" % (bad.size, bad[0])
        recv.fill_(CANARY)
        st = tuna.tuna_get_stats()
        if counts.max() > 0:
            assert st.hop_kernels == tuna.TUNA_HOP_DIRECT and st.n_phases == 1
            assert st.phase[0].payload_bytes == int(counts.sum()) - int(np.trace(counts))
            assert st.phase[0].staged_bytes == _staged(lay)
    tuna.tuna_release()


@pytest.mark.parametrize("longest,quantum,lay_args", [
    (15, 1, {"permute_seed": 3}), (16, 4, {}), (16, 8, {"gap": 3}), (16, 16, {}), (17, 1, {}), (64, 4, {"gap": 1, "permute_seed": 5}),
    (64, 16, {"align": 16}), (64, 64, {}), (65, 1, {"permute_seed": 7}), (256, 4, {}), (256, 16, {"align": 16}), (256, 128, {"align": 128})])
@pytest.mark.parametrize("P", [2, 3, 8, 9, 16, 17, 31, 33, 64, 65, 130, 257])
def test_tiles(tuna, P, longest, quantum, lay_args):
    rng = np.random.default_rng(P * 1000 + longest)
    counts = rng.integers(0, longest // quantum + 1, (P, P)) * quantum
    counts[rng.random((P, P)) < 0.2] = 0
    if P > 8:
        counts[P // 2] = 0                                   # a rank that sends nothing, one that receives nothing
        counts[:, P - 2] = 0
    counts[0, P - 1] = counts[P - 1, P - 1] = longest
    _run(tuna, counts, P, lay_args)


@pytest.mark.parametrize("P,longest,quantum", [(4200, 8, 4), (2100, 48, 4), (2060, 64, 16), (2100, 96, 4)])
def test_several_steps(tuna, P, longest, quantum):
    rng = np.random.default_rng(P)
    counts = rng.integers(0, longest // quantum + 1, (P, P), dtype=np.int32) * quantum
    _run(tuna, counts, 0, {})


@pytest.mark.parametrize("size", [3, 15, 16, 200, 256, 257, 3001, 65536])
@pytest.mark.parametrize("P,radix", [(2, 2), (19, 19), (40, 3), (170, 13), (300, 300)])
def test_own_blocks_only(tuna, P, radix, size):
    """Nothing but the blocks that ranks keep for themselves, which the launch of the first phase moves: calls and plans, T in
    either layout."""
    dev = "cuda:0"
    counts = np.zeros((P, P), dtype=np.int32)
    np.fill_diagonal(counts, size)
    counts[P // 2, P // 2] = 0
    lay = wl.make_layout(counts, gap=1)
    host = wl.payload_position_hash(size, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    send = torch.from_numpy(host).to(dev)
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    args = [send] + [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls)] + [recv] + \
           [torch.from_numpy(a).to(dev) for a in (lay.recvcounts, lay.rdispls)]
    o = tuna.tuna_opts_init()
    o.mode = tuna.TUNA_MODE_FUSED
    for o.t_layout in (tuna.TUNA_T_EXACT, tuna.TUNA_T_SLOTS):
        print("own blocks", P, radix, size, o.t_layout, flush=True)
        assert tuna.tuna_alltoallv_ex(None, *args, P, 0, radix, radix, o) == 0
        torch.cuda.synchronize()
        assert np.array_equal(recv.cpu().numpy(), want)
        recv.fill_(CANARY)
        rc, plan = tuna.tuna_alltoallv_init_ex(None, *args, P, 0, radix, radix, o)
        assert rc == 0, tuna.tuna_strerror(rc)
        try:
            assert tuna.tuna_start(plan) == 0
            torch.cuda.synchronize()
            assert np.array_equal(recv.cpu().numpy(), want), "plan"
        finally:
            tuna.tuna_plan_free(plan)
        recv.fill_(CANARY)
    tuna.tuna_release()

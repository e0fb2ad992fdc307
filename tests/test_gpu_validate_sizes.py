"""The validation pass at the sizes where its shape changes: one and several 64 x 64 tiles, workgroups that take one and
two of them (22 x 22 and 23 x 23 tiles), rows added up by the host (at most 64 workgroups and 24 classes of waiting blocks)
and by a kernel.  A valid problem arrives byte for byte, and a wrong entry anywhere -- also in the last row and column
-- is reported with its code before anything moves."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0x3C


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


@pytest.mark.parametrize("P,radix", [(3, 2), (64, 2), (65, 8), (256, 2), (511, 8), (512, 512), (513, 8), (1408, 38), (1409, 3)])
def test_validation(tuna, P, radix):
    rng = np.random.default_rng(P)
    counts = np.ascontiguousarray(4 * rng.integers(0, 11, (P, P)), dtype=np.int32)
    counts[P - 1, P - 1] = 40
    lay = wl.make_layout(counts)
    host = wl.payload_position_hash(9, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    dev = "cuda:0"
    send = torch.from_numpy(host).to(dev)
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    o = tuna.tuna_opts_init()
    o.mode = tuna.TUNA_MODE_FUSED

    def call(sc=lay.sendcounts, sd=lay.sdispls, rc_=lay.recvcounts, rd=lay.rdispls):
        d = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (sc, sd, rc_, rd)]
        rc = tuna.tuna_alltoallv_ex(None, send, d[0], d[1], recv, d[2], d[3], P, 0, radix, radix, o)
        torch.cuda.synchronize()
        return rc

    print("validation", P, radix, flush=True)
    for r, c in ((0, P - 1), (P - 1, P - 1), (P - 1, 0), (P // 2, P // 3)):
        bad = lay.recvcounts.copy()
        bad[r, c] += 4
        assert call(rc_=bad) == tuna.TUNA_ERR_COUNT_MISMATCH
        bad = lay.sendcounts.copy()
        bad[r, c] = -4
        assert call(sc=bad) == tuna.TUNA_ERR_NEGATIVE_COUNT
        bad, some = lay.sdispls.copy(), lay.sendcounts.copy()
        bad[r, c] = -8
        if some[r, c] > 0:
            assert call(sd=bad) == tuna.TUNA_ERR_ARG
    assert bool((recv == CANARY).all())                     # nothing moved
    assert call() == 0
    assert np.array_equal(recv.cpu().numpy(), want)
    st = tuna.tuna_get_stats()
    assert st.total_payload_bytes == lay.payload_bytes and st.max_block_bytes == counts.max() and st.granularity == 4


def test_windows_count_from_the_first_long_block_on(tuna):
    """1536 ranks are 24 x 24 tiles, of which some workgroups take two, one behind the other: blocks of 64 bytes in the first, one of 65 in
    the second.  What a tile holds before its workgroup has seen a block of more than 64 bytes is in no window, whichever of its waves are
    ahead, so the blocks do not cluster and a plan's phase runs the direct hop; every time."""
    P = 1536
    counts = np.zeros((P, P), dtype=np.int32)
    counts[:64, :384] = 64                                   # tiles 0 to 5
    counts[64 * 21 + 5, 64 * 8 + 3:64 * 14:64] = 65          # one block in each of the tiles 512 to 517
    mean = counts.sum() / P**2
    assert 65 < 8 * 64 * mean < 64 * 64 / 4                  # clustered with a part of a first tile's window, not without
    lay = wl.make_layout(counts)
    host = wl.payload_position_hash(9, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    dev = "cuda:0"
    send = torch.from_numpy(host).to(dev)
    d = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    for _ in range(8):
        recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
        rc, plan = tuna.tuna_alltoallv_init(send, d[0], d[1], recv, d[2], d[3], P, 0, P, P)
        assert rc == 0 and tuna.tuna_start(plan) == 0
        torch.cuda.synchronize()
        assert tuna.tuna_get_stats().hop_kernels == tuna.TUNA_HOP_DIRECT
        assert np.array_equal(recv.cpu().numpy(), want)
        assert tuna.tuna_plan_free(plan) == 0

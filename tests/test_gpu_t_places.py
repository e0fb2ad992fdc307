"""The places of waiting blocks in exact-size T and the phases that find their blocks by them: on both sides of the radix
and of the rank count where the kernel that lays them out changes, classes of one block and of several batches of a
workgroup, ranks that no tile divides, hierarchies, gapped and permuted regions, empty blocks; on both sides of the number
of rounds from which a workgroup takes the blocks of one sender, with each of its block sizes and kinds of access, and with
several steps per workgroup.  Reference: the same call with three-stage phases and T in slots, which asks for no places."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


CASES = [
    # P, ranks per node, local radix, global radix, longest block, quantum, share of empty blocks, layout arguments
    (9, 0, 8, 8, 40, 1, 0.0, {}), (9, 0, 7, 7, 40, 1, 0.0, {}), (64, 0, 8, 8, 16, 4, 0.3, {"gap": 3, "permute_seed": 1}),
    (65, 0, 8, 8, 64, 8, 0.0, {}), (257, 0, 16, 16, 16, 4, 0.0, {}), (1025, 0, 32, 32, 300, 4, 0.2, {"gap": 1, "permute_seed": 2}),
    (1024, 0, 1023, 1023, 16, 8, 0.0, {}), (1100, 0, 17, 17, 15, 1, 0.5, {}), (1300, 0, 36, 36, 64, 4, 0.0, {"gap": 4}),
    (1500, 0, 40, 40, 256, 16, 0.0, {"align": 16}), (96, 12, 8, 8, 60, 4, 0.0, {}), (1024, 32, 32, 32, 16, 4, 0.1, {"gap": 2, "permute_seed": 3}),
    (1200, 60, 16, 20, 64, 1, 0.0, {}), (2100, 70, 8, 30, 12, 4, 0.0, {}), (2049, 0, 46, 46, 16, 8, 0.0, {}),
    # 11, 12 and 13 rounds; the first and the last phase with their own; one block per lane, four and sixteen lanes per block
    (144, 0, 12, 12, 16, 4, 0.0, {}), (169, 0, 13, 13, 16, 1, 0.1, {"gap": 5, "permute_seed": 4}), (170, 0, 13, 13, 64, 4, 0.0, {}),
    (183, 0, 14, 14, 64, 16, 0.1, {"align": 16}), (300, 0, 20, 20, 256, 16, 0.1, {"align": 16}), (259, 0, 16, 16, 256, 1, 0.0, {}),
    (270, 0, 15, 15, 128, 128, 0.3, {"align": 128}), (600, 30, 13, 20, 200, 4, 0.2, {"gap": 1, "permute_seed": 6}), (390, 15, 15, 13, 64, 1, 0.0, {}),
]


def _run(tuna, P, rpn, rl, rg, counts, lay_args):
    dev = "cuda:0"
    lay = wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32), **lay_args)
    meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    send = torch.empty(lay.send_bytes // 8 + 1, dtype=torch.int64, device=dev).random_(generator=gen)
    recv = torch.zeros(lay.recv_bytes // 8 + 1, dtype=torch.int64, device=dev)
    args = (send, meta[0], meta[1], recv, meta[2], meta[3], P, rpn, rl, rg)
    print("places", P, rpn, rl, rg, lay_args, lay.payload_bytes, flush=True)
    o = tuna.tuna_opts_init()
    o.mode, o.t_layout = tuna.TUNA_MODE_STAGED, tuna.TUNA_T_SLOTS
    assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
    torch.cuda.synchronize()
    want, staged = recv.clone(), tuna.tuna_get_stats()
    o.mode, o.t_layout = tuna.TUNA_MODE_FUSED, tuna.TUNA_T_EXACT
    for n in range(2):
        recv.zero_()
        assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
        torch.cuda.synchronize()
        assert torch.equal(recv, want), n
        st = tuna.tuna_get_stats()
        assert st.hop_kernels in (tuna.TUNA_HOP_DIRECT, tuna.TUNA_HOP_ROWS)
        for x in range(st.n_phases):
            assert st.phase[x].payload_bytes == staged.phase[x].payload_bytes, x
    # whatever T's layout and whichever way its blocks are found, the phases move the same 16-byte chunks
    exact = [st.phase[x].staged_bytes for x in range(st.n_phases)]
    o.t_layout = tuna.TUNA_T_SLOTS
    recv.zero_()
    assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
    torch.cuda.synchronize()
    assert torch.equal(recv, want)
    st = tuna.tuna_get_stats()
    assert [st.phase[x].staged_bytes for x in range(st.n_phases)] == exact
    tuna.tuna_release()


@pytest.mark.parametrize("i", range(len(CASES)))
def test_places(tuna, i):
    P, rpn, rl, rg, longest, q, empty, lay_args = CASES[i]
    rng = np.random.default_rng(100 + i)
    counts = rng.integers(0, longest // q + 1, (P, P)) * q
    counts[rng.random((P, P)) < empty] = 0
    _run(tuna, P, rpn, rl, rg, counts, lay_args)


@pytest.mark.parametrize("P,radix,size", [(8192, 91, 4), (8193, 91, 4), (8193, 91, 20)])
def test_places_of_many_ranks(tuna, P, radix, size):
    """One pair in eight exchanges a word or five: most classes' blocks are empty.  (20 bytes are moved by four lanes each,
    several steps of one sender's blocks per workgroup.)"""
    rng = np.random.default_rng(P)
    _run(tuna, P, 0, radix, radix, (rng.integers(0, 8, (P, P), dtype=np.int32) == 3).astype(np.int32) * size, {})

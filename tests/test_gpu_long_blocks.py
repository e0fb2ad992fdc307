"""Phases of long blocks (Algorithm "TuNA", lines 15-20 as one hop, from a list of 4 KiB units): the edges of the units
and of their 16-byte pieces, odd addresses, gaps and permuted regions, empty and tiny blocks among long ones, hierarchies,
T in both layouts, own blocks, more segments than a workgroup lays out at a time; calls and plans.  Reference: the same
call with three-stage phases, another set of kernels."""
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


def _uniform(P, mean, q):
    return np.random.default_rng(P + mean).integers(0, 2 * mean // q + 1, (P, P)) * q


def _edges(P):
    """Blocks that end just before, at and behind a unit, a piece and a line, tiny and empty ones; the others 64 KiB and a bit."""
    c = np.random.default_rng(P).integers(65536, 66000, (P, P))
    some = [0, 1, 3, 4, 7, 15, 16, 17, 127, 128, 129, 4080, 4095, 4096, 4097, 4111, 4112, 8191, 8192, 8193, 8207, 8208]
    c[np.random.default_rng(P + 1).random((P, P)) < 0.4] = 0
    for k, n in enumerate(some):
        c[k % P, (3 * k + 1) % P] = n
    return c


def _sparse(P):
    c = np.where(np.random.default_rng(P).random((P, P)) < 0.3, 90000, 0)
    c[3, 7] = 5000011
    return c


CASES = [
    # P, counts, ranks per node, radix, layout arguments, T in slots, offset of the send buffer, long by the rule
    (2, lambda P: _uniform(P, 150000, 1), 0, 2, {}, 0, 0, True),
    (5, lambda P: _uniform(P, 300001, 1), 0, 2, {}, 0, 3, True),
    (16, lambda P: _uniform(P, 150000, 16), 0, 16, {"align": 16}, 0, 0, True),
    (16, lambda P: _uniform(P, 150000, 16), 0, 4, {"gap": 5, "permute_seed": 3}, 0, 1, True),
    (31, _edges, 0, 31, {}, 0, 0, True),
    (31, _edges, 0, 2, {}, 0, 0, True),
    (31, _edges, 0, 3, {"gap": 3, "permute_seed": 9}, 1, 2, True),
    (40, lambda P: np.full((P, P), 131072), 0, 6, {"align": 128}, 0, 0, True),
    (24, _edges, 4, 2, {"gap": 1}, 0, 0, True),
    (24, _edges, 6, 24, {}, 1, 0, True),
    (300, _sparse, 0, 17, {}, 0, 0, True),
    (300, _sparse, 0, 300, {"gap": 3}, 0, 5, True),
    (64, lambda P: np.full((P, P), 16892), 0, 64, {}, 0, 0, False),
    (64, lambda P: np.full((P, P), 16900), 0, 8, {}, 0, 0, True),
    (200, lambda P: np.full((P, P), 22524), 0, 200, {}, 0, 0, False),
    (200, lambda P: np.full((P, P), 22532), 0, 200, {}, 0, 0, True),
    (160, lambda P: np.full((P, P), 32764), 0, 13, {}, 0, 0, False),
    (160, lambda P: np.full((P, P), 32772), 0, 13, {}, 0, 0, True),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_long_blocks(tuna, i):
    P, make, rpn, radix, lay_args, slots, off, is_long = CASES[i]
    dev = "cuda:0"
    lay = wl.make_layout(np.ascontiguousarray(make(P), dtype=np.int32), **lay_args)
    print("long blocks", i, P, rpn, radix, lay_args, slots, off, lay.payload_bytes, flush=True)
    meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    gen = torch.Generator(device=dev)
    gen.manual_seed(i)
    room = torch.empty(lay.send_bytes // 8 + 2, dtype=torch.int64, device=dev).random_(generator=gen).view(torch.uint8)
    send, before = room[off:off + lay.send_bytes], room.clone()
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    args = (send, meta[0], meta[1], recv, meta[2], meta[3], P, rpn, radix, radix)
    o = tuna.tuna_opts_init()
    o.mode = tuna.TUNA_MODE_STAGED
    assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
    torch.cuda.synchronize()
    want, staged = recv.clone(), tuna.tuna_get_stats()
    o.mode, o.t_layout = tuna.TUNA_MODE_FUSED, tuna.TUNA_T_SLOTS if slots else tuna.TUNA_T_EXACT

    def check(what):
        torch.cuda.synchronize()
        assert torch.equal(recv, want), what
        assert torch.equal(room, before), what
        st = tuna.tuna_get_stats()
        assert (st.hop_kernels == tuna.TUNA_HOP_LONG) == is_long, (what, st.hop_kernels)
        for x in range(st.n_phases):
            assert st.phase[x].payload_bytes == staged.phase[x].payload_bytes, (what, x)

    for n in range(2):                                      # the second call finds the counters of the first
        recv.fill_(CANARY)
        assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
        check("call %d" % n)
    rc, plan = tuna.tuna_alltoallv_init_ex(None, *args, o)
    assert rc == 0, tuna.tuna_strerror(rc)
    try:
        for n in range(2):
            recv.fill_(CANARY)
            assert tuna.tuna_start(plan) == 0
            check("start %d" % n)
    finally:
        assert tuna.tuna_plan_free(plan) == 0
    tuna.tuna_release()

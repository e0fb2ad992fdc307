"""Kernels of a call that run ahead of the host: calls of one schedule that have a use for them and calls that have none in turn, until they
are left out and come back, and sizing queries and plans behind a call that is still in flight.  Byte for byte against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0x4B
DEV = "cuda:0"


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


class Prob:
    def __init__(self, counts, seed):
        self.lay = lay = wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32))
        host = wl.payload_position_hash(seed, lay.send_bytes)
        self.want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
        assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, self.want, lay.recvcounts, lay.rdispls) == 0
        self.send = torch.from_numpy(host).to(DEV)
        self.recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=DEV)
        self.sc, self.sd, self.rc, self.rd = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]

    def args(self):
        return self.send, self.sc, self.sd, self.recv, self.rc, self.rd

    def arrived(self):
        return np.array_equal(self.recv.cpu().numpy(), self.want)


def _short(P, seed=0):
    return np.random.default_rng(P + seed).integers(0, 61, (P, P))


def _engine(P):
    """Short blocks and two that are too long for the kernels that find their blocks themselves."""
    c = _short(P, 1)
    c[1, P - 2] = c[P - 1, 3] = 70001
    return c


@pytest.mark.parametrize("P,radix", [(100, 10), (100, 100), (300, 2), (513, 23), (513, 512), (700, 5)])
@pytest.mark.parametrize("how", ["call", "noalloc"])
def test_calls_that_use_them_and_calls_that_do_not(tuna, P, radix, how):
    if how == "noalloc" and P == 700:
        P = 400                                              # what fits into the static array
    probs = {"direct": Prob(_short(P), 3), "engine": Prob(_engine(P), 5)}
    wrong = probs["direct"].rc.clone()
    wrong[0, P - 1] += 1
    o = tuna.tuna_opts_init()
    o.mode, o.t_layout = tuna.TUNA_MODE_FUSED, tuna.TUNA_T_EXACT

    def call(p, rc=None):
        a = list(p.args())
        a[4] = a[4] if rc is None else rc
        return tuna.tuna_alltoallv_noalloc(*a, P, 0, radix, radix) if how == "noalloc" else tuna.tuna_alltoallv_ex(None, *a, P, 0, radix, radix, o)

    for n, kind in enumerate(["direct", "direct"] + ["engine"] * 4 + ["direct"] * 3 + ["engine", "direct"] * 2 + ["engine"] * 3 + ["direct"] * 2):
        p = probs[kind]
        p.recv.fill_(CANARY)
        print("early", how, P, radix, n, kind, flush=True)
        assert call(probs["direct"], wrong) == tuna.TUNA_ERR_COUNT_MISMATCH
        assert call(p) == 0
        torch.cuda.synchronize()
        assert p.arrived(), (n, kind)


@pytest.mark.parametrize("P,radix", [(600, 25), (700, 2), (300, 2)])
def test_queries_and_plans_behind_a_call_in_flight(tuna, P, radix):
    """They do not wait for it, and what their validation finds is another problem's: nothing to move, and blocks too long for any such hop."""
    p, other = Prob(_short(P), 7), Prob(_engine(96), 9)
    nothing = torch.zeros((P, P), dtype=torch.int32, device=DEV)
    o = tuna.tuna_opts_init()
    o.mode, o.t_layout = tuna.TUNA_MODE_FUSED, tuna.TUNA_T_EXACT
    stream, plan_stream = torch.cuda.Stream(), torch.cuda.Stream()
    for n in range(6):
        p.recv.fill_(CANARY)
        torch.cuda.synchronize()
        print("in flight", P, radix, n, flush=True)
        assert tuna.tuna_alltoallv_ex(None, *p.args(), P, 0, radix, radix, o, stream) == 0
        rc, _ = tuna.tuna_workspace_bytes(nothing, P, 0, radix, radix)
        assert rc == 0
        rc, plan = tuna.tuna_alltoallv_init_ex(None, *other.args(), 96, 0, 4, 4, o, plan_stream)
        assert rc == 0
        torch.cuda.synchronize()
        assert p.arrived(), n
        assert tuna.tuna_plan_free(plan) == 0

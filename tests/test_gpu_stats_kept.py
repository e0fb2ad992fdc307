"""The statistics of the last call stay what they were while nothing but queries follow it: a sizing query
(tuna_workspace_bytes) validates counts on the default context's status block, and so does a plan that has nothing
to move, but the per-phase totals there belong to the call -- also while the call is still in flight on a stream
that the query's stream does not wait for.  Rank counts on both sides of the size up to which the host adds up the
validation pass's partial results (64 tiles of 64 x 64)."""
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


def _phases(tuna):
    st = tuna.tuna_get_stats()
    return [(st.phase[x].payload_bytes, st.phase[x].staged_bytes) for x in range(st.n_phases)]


@pytest.mark.parametrize("P,longest", [(96, 200), (96, 3000), (512, 100), (520, 100), (520, 1500)])
def test_totals_survive_queries(tuna, P, longest):
    dev = "cuda:0"
    lay = wl.make_layout(wl.counts_uniform_bytes(P, P + longest, longest), gap=1)
    sc, sd, rc_, rd = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    send = torch.zeros(lay.send_bytes, dtype=torch.uint8, device=dev)
    recv = torch.zeros(lay.recv_bytes, dtype=torch.uint8, device=dev)
    zero = torch.zeros((P, P), dtype=torch.int32, device=dev)
    stream = torch.cuda.Stream()

    def call(s=None):
        assert tuna.tuna_alltoallv(send, sc, sd, recv, rc_, rd, P, 4, 0, s) == 0

    print("totals survive queries", P, longest, flush=True)
    call()
    want = _phases(tuna)
    # every block moves once per non-zero digit of its distance
    hops = sum(int(lay.sendcounts[(np.arange(P) + k) % P, np.arange(P)].astype(np.int64).sum()) *
               sum(1 for x in range(8) if (k // 4 ** x) % 4) for k in range(1, P))
    assert sum(b for b, _ in want) == hops and all(b > 0 and c >= b for b, c in want)
    rc, nbytes = tuna.tuna_workspace_bytes(sc, P, 0, 4, 4)
    assert rc == 0 and nbytes > 0
    assert _phases(tuna) == want
    for _ in range(8):                                      # the query runs beside the call
        torch.cuda.synchronize()
        call(stream)
        assert tuna.tuna_workspace_bytes(sc, P, 0, 4, 4)[0] == 0
        assert _phases(tuna) == want
    rc, plan = tuna.tuna_alltoallv_init(send, zero, sd, recv, zero, rd, P, 0, 4, 4)
    assert rc == 0
    try:
        assert _phases(tuna) == want
    finally:
        assert tuna.tuna_plan_free(plan) == 0
    torch.cuda.synchronize()

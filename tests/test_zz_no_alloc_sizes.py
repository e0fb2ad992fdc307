"""The call that allocates nothing where its validation pass changes hands: the results of up to 64 workgroups and 24 classes of waiting
blocks are copied to the host and added up there (512 ranks have 64 tiles, 513 more; radix 2 has 28 classes from 129 ranks on), others by a
kernel.  Twice each, byte for byte against the oracle, with a refused and an empty call between."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0xA5


@pytest.mark.parametrize("P,rpn,rl,rg", [(2, 0, 2, 2), (65, 0, 8, 8), (128, 0, 2, 2), (129, 0, 2, 2), (512, 0, 23, 23), (513, 0, 23, 23), (512, 0, 512, 512), (513, 0, 512, 512),
                                         (192, 12, 4, 4)])
def test_sizes(P, rpn, rl, rg):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as tuna
    counts = np.random.default_rng(P + rl).integers(0, 41, (P, P)).astype(np.int32)
    counts[P - 1, 0] = 40
    lay = wl.make_layout(counts)
    host = wl.payload_position_hash(3, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    dev = "cuda:0"
    send = torch.from_numpy(host).to(dev)
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    sc, sd, rc_, rd = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    wrong, none = rc_.clone(), torch.zeros_like(sc)
    wrong[0, P - 1] += 1
    for n in range(2):
        recv.fill_(CANARY)
        print("no-alloc sizes", P, rpn, rl, n, flush=True)
        assert tuna.tuna_alltoallv_noalloc(send, sc, sd, recv, wrong, rd, P, rpn, rl, rg) == tuna.TUNA_ERR_COUNT_MISMATCH
        assert tuna.tuna_alltoallv_noalloc(send, none, sd, recv, none, rd, P, rpn, rl, rg) == 0
        torch.cuda.synchronize()
        assert bool((recv == CANARY).all())
        assert tuna.tuna_alltoallv_noalloc(send, sc, sd, recv, rc_, rd, P, rpn, rl, rg) == 0
        torch.cuda.synchronize()
        assert np.array_equal(recv.cpu().numpy(), want)

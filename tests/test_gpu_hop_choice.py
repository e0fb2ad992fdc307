"""Which kernel a one-kernel phase runs (Algorithm "TuNA", lines 15-20 as one hop).  Blocks of up to 256 bytes: the
direct hop, which finds them itself, unless the payload is large and they are longer than 64 bytes.  Those and blocks of
up to 64 KiB, all rounds of a phase at once: the row hop, which finds them too -- except where the destination-tiled hop can run and is the faster one.  That one needs dense receive
regions and data at least word-granular; for a schedule's last phase, whose blocks all go into R, blocks that are
mostly interior (mean of 700 bytes or more, at most a quarter of them under 256 bytes); for the phases before it,
which store whole chunks into T, a mean block of 512 bytes or more.  A plan, which has paid for its metadata, keeps
it there; a call does for mean blocks above 4 KiB, 3.5 KiB or 1.5 KiB, by its payload (256 MiB, 1 GiB), where it can
run in every phase.  On whole lines the copy engine's hop is the better one from a mean block of 16 KiB (a plan: from
a longest block of 12 KiB), unless T is in slots.  The copy engine's hop does everything else, also where long blocks
lie side by side, so that a few waves of the row hop would move most of the payload.  The statistics say which of the
four ran, and under profiling a phase's tiled hop is timed as its unpack time and every other one as its pack time;
every case is also compared with the CPU oracle byte for byte."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
CANARY = 0x5A
P = 96


@pytest.fixture(scope="module")
def tuna():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02581_amd as t
    t.load()
    return t


def _normal(seed=11, mean=1024.0):
    return wl.counts_normal(P, seed, mean, mean / 4, 4)


def _mostly_short():
    c = wl.counts_normal(P, 13, 1400.0, 256.0, 4).copy()
    rng = np.random.default_rng(5)
    c[rng.random((P, P)) < 0.4] = 64              # two blocks in five under 256 bytes; the mean stays above 700
    assert c.mean() > 800
    return c


def _zipf(longest):
    c = wl.counts_zipf(P, 12, 1.2, min(longest, 65536), 4).copy()
    c[5, 17] = longest
    return c


def _equal(n):
    return np.full((P, P), n, dtype=np.int32)


def _except(n, rest):
    """Blocks of `rest` bytes, and of n where the sender and the receiver say so."""
    def make(where):
        i = np.arange(P)
        return np.where(np.broadcast_to(where(i[:, None], i[None, :]), (P, P)), n, rest).astype(np.int32)
    return make


E, T, D, R = "engine", "tiled", "direct", "rows"
CASES = {
    # name: (counts, layout arguments, options, call: (kernel of the phases before the last, of the last[, of the only
    # phase of a linear schedule, where it is another one]), plan: likewise); None: three stages
    "normal 1 KiB, dense": (_normal, {}, {}, (R, R), (T, T)),
    "normal 1 KiB, chunk-granular": (lambda: _normal() // 16 * 16, {"align": 16}, {}, (R, R), (T, T)),
    "normal 3.9 KiB, dense": (lambda: _normal(14, 3900.0), {}, {}, (R, R), (T, T)),
    "normal 4.3 KiB, dense": (lambda: _normal(14, 4300.0), {}, {}, (T, T), (T, T)),
    "every other block empty, the others 4 KiB": (lambda: _except(4092, 0)(lambda s, r: (s + r) % 2 == 0), {}, {}, (R, R), (T, R)),
    "whole lines, 12 KiB": (lambda: _equal(12288), {"align": 128}, {}, (R, R), (R, R)),
    "whole lines, 12.1 KiB": (lambda: _equal(12288 + 128), {"align": 128}, {}, (R, R), (E, E)),
    "whole lines, 16 KiB": (lambda: _equal(16384), {"align": 128}, {}, (R, R), (E, E)),
    "whole lines, 16.1 KiB": (lambda: _equal(16384 + 128), {"align": 128}, {}, (E, E), (E, E)),
    "whole lines, 16.1 KiB, T in slots": (lambda: _equal(16384 + 128), {"align": 128}, {"t_layout": 0}, (R, R, E), (R, R, E)),
    "gaps between the blocks of R": (_normal, {"gap": 8}, {}, (R, R), (R, R)),
    "gaps, normal 4.3 KiB": (lambda: _normal(14, 4300.0), {"gap": 8}, {}, (R, R), (R, R)),
    "byte-granular sizes": (lambda: _normal() + 1, {}, {}, (R, R), (R, R)),
    "Zipf sizes (most blocks tiny, mean 800 bytes)": (lambda: _zipf(16384), {}, {}, (R, R), (T, E)),
    "Zipf sizes, longest block 65536 bytes, gaps": (lambda: _zipf(65536), {"gap": 8}, {}, (R, R), (E, E)),
    "Zipf sizes, longest block 65540 bytes, gaps": (lambda: _zipf(65540), {"gap": 8}, {}, (E, E), (E, E)),
    "Zipf sizes, longest block 65540 bytes": (lambda: _zipf(65540), {}, {}, (T, E), (T, E)),
    "mean block of 700 bytes": (lambda: _equal(700), {}, {}, (R, R), (T, T)),
    "mean block of 696 bytes": (lambda: _equal(696), {}, {}, (R, R), (T, R)),
    "mean block of 516 bytes": (lambda: _equal(516), {}, {}, (R, R), (T, R)),
    "mean block of 508 bytes": (lambda: _equal(508), {}, {}, (R, R), (R, R)),
    "mean block of 260 bytes": (lambda: _equal(260), {}, {}, (R, R), (R, R)),
    "longest block 257 bytes": (lambda: _equal(257), {}, {}, (R, R), (R, R)),
    "longest block 256 bytes": (lambda: _equal(256), {}, {}, (D, D), (D, D)),
    "longest block 256 bytes, gaps": (lambda: _equal(256), {"gap": 3}, {}, (D, D), (D, D)),
    "two blocks in five short": (_mostly_short, {}, {}, (R, R), (T, R)),
    "64 KiB to one rank, gaps": (lambda: _except(65536, 40)(lambda s, r: r == 7), {"gap": 8}, {}, (E, E), (E, E)),
    "64 KiB to one rank": (lambda: _except(65536, 40)(lambda s, r: r == 7), {}, {}, (T, E), (T, E)),
    "1 KiB to one rank": (lambda: _except(1024, 40)(lambda s, r: r == 7), {}, {}, (R, R), (E, E)),
    "300 bytes to one rank": (lambda: _except(300, 40)(lambda s, r: r == 7), {}, {}, (R, R), (R, R)),
    "64 KiB from one rank": (lambda: _except(65536, 40)(lambda s, r: s == 7), {"gap": 8}, {}, (E, E, R), (E, E)),
    "16 KiB among eight ranks": (lambda: _except(16384, 40)(lambda s, r: (s < 8) & (r < 8)), {}, {}, (E, E), (E, E)),
    "one block of 64 KiB among tiny ones": (lambda: _except(65536, 40)(lambda s, r: (s == 7) & (r == 9)), {}, {}, (R, R), (E, E)),
    "rounds in batches": (_normal, {}, {"block_count": 3}, (E, E), (E, E)),
    "rounds in batches, short blocks": (lambda: _equal(64), {}, {"block_count": 3}, (D, D), (D, D)),
    "three-stage phases": (_normal, {}, {"mode": "staged"}, None, None),
}


def _check(tuna, name, want, n_phases):
    st = tuna.tuna_get_stats()
    assert st.n_phases == n_phases
    bit = {E: tuna.TUNA_HOP_ENGINE, T: tuna.TUNA_HOP_TILED, D: tuna.TUNA_HOP_DIRECT, R: tuna.TUNA_HOP_ROWS}
    kernels = [] if want is None else [want[-1]] if n_phases == 1 else [want[0]] * (n_phases - 1) + [want[1]]
    assert st.hop_kernels == sum(bit[k] for k in set(kernels)), (name, st.hop_kernels)
    for x in range(n_phases):
        ph = st.phase[x]
        if want is None:                                    # pack, exchange and unpack all ran
            assert ph.ms_pack > 0 and ph.ms_exchange > 0 and ph.ms_unpack > 0, (name, x)
        elif kernels[x] == T:
            assert ph.ms_unpack > 0 and ph.ms_pack == 0 and ph.ms_exchange == 0, (name, x)
        else:
            assert ph.ms_pack > 0 and ph.ms_unpack == 0 and ph.ms_exchange == 0, (name, x)


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("radix", [4, P])
def test_which_hop_runs(tuna, name, radix):
    make, lay_args, opts, call, plan_kernels = CASES[name]
    counts = np.ascontiguousarray(make(), dtype=np.int32)
    lay = wl.make_layout(counts, **lay_args)
    host = wl.payload_position_hash(21, lay.send_bytes)
    want = np.full(lay.recv_bytes, CANARY, dtype=np.uint8)
    assert oracle.alltoallv(host, lay.sendcounts, lay.sdispls, want, lay.recvcounts, lay.rdispls) == 0
    dev = "cuda:0"
    send = torch.from_numpy(host).to(dev)
    recv = torch.full((lay.recv_bytes,), CANARY, dtype=torch.uint8, device=dev)
    meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    o = tuna.tuna_opts_init()
    o.profile = 1
    o.t_layout = opts.get("t_layout", tuna.TUNA_T_EXACT)
    o.mode = tuna.TUNA_MODE_STAGED if opts.get("mode") == "staged" else tuna.TUNA_MODE_FUSED
    o.block_count = opts.get("block_count", 0)
    n_phases = 1 if radix == P else 4
    print("case %s, radix %d" % (name, radix), flush=True)
    rc = tuna.tuna_alltoallv_ex(None, send, meta[0], meta[1], recv, meta[2], meta[3], P, 0, radix, radix, o)
    assert rc == 0, tuna.tuna_strerror(rc)
    torch.cuda.synchronize()
    assert np.array_equal(recv.cpu().numpy(), want), name
    _check(tuna, name, call, n_phases)
    rc, plan = tuna.tuna_alltoallv_init_ex(None, send, meta[0], meta[1], recv, meta[2], meta[3], P, 0, radix, radix, o)
    assert rc == 0, tuna.tuna_strerror(rc)
    try:
        recv.fill_(CANARY)
        assert tuna.tuna_start(plan) == 0
        torch.cuda.synchronize()
        assert np.array_equal(recv.cpu().numpy(), want), name + " (plan)"
        _check(tuna, name + " (plan)", plan_kernels, n_phases)
    finally:
        assert tuna.tuna_plan_free(plan) == 0


def _device_problem(P, counts, gap=0, permute_seed=None):
    """A problem too large for the oracle's test time: its payload is made on the device, its reference is the call with
    three-stage phases (another set of kernels)."""
    dev = "cuda:0"
    lay = wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32), gap=gap, permute_seed=permute_seed)
    meta = [torch.from_numpy(a).to(dev) for a in (lay.sendcounts, lay.sdispls, lay.recvcounts, lay.rdispls)]
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    send = torch.empty((lay.send_bytes + 7) // 8, dtype=torch.int64, device=dev).random_(generator=gen)
    recv = torch.zeros((lay.recv_bytes + 7) // 8, dtype=torch.int64, device=dev)
    return lay, send, meta, recv


def _half(P, n):
    i = np.arange(P)
    return np.where((i[:, None] + i[None, :]) % 2 == 0, n, 0).astype(np.int32)


# (a negative radix: every other block is empty, so that the last phase cannot be tiled)
@pytest.mark.parametrize("P,mean,radix,want", [(320, 3300, 8, R), (320, 3700, 8, T), (640, 2400, 8, R), (640, 2800, 640, T),
                                               (1024, 1400, 16, R), (1024, 1650, 16, T), (1024, 1700, -16, R)])
def test_hop_of_a_call_by_payload(tuna, P, mean, radix, want):
    counts = wl.counts_normal(P, P + mean, float(mean), mean / 4.0, 4) if radix > 0 else _half(P, 2 * mean)
    radix = abs(radix)
    lay, send, meta, recv = _device_problem(P, counts)
    print("hop by payload", P, mean, radix, lay.payload_bytes, flush=True)
    results = []
    for mode in (tuna.TUNA_MODE_STAGED, tuna.TUNA_MODE_FUSED):
        o = tuna.tuna_opts_init()
        o.mode, o.t_layout = mode, tuna.TUNA_T_EXACT
        recv.zero_()
        rc = tuna.tuna_alltoallv_ex(None, send, meta[0], meta[1], recv, meta[2], meta[3], P, 0, radix, radix, o)
        assert rc == 0, tuna.tuna_strerror(rc)
        torch.cuda.synchronize()
        results.append(recv.clone())
        st = tuna.tuna_get_stats()
    assert torch.equal(*results)
    assert st.hop_kernels == {R: tuna.TUNA_HOP_ROWS, T: tuna.TUNA_HOP_TILED}[want], st.hop_kernels
    del results
    tuna.tuna_release()


@pytest.mark.parametrize("P,radix,want,plan_want", [(1024, 32, E, E), (1024, 1024, R, R), (512, 32, R, E)])
def test_hop_of_long_blocks_a_radix_apart(tuna, P, radix, want, plan_want):
    """16 KiB at every 32nd distance: evenly spread over a rank's blocks, but one run of the first phase's at radix 32."""
    i = np.arange(P)
    lay, send, meta, recv = _device_problem(P, np.where((i[None, :] - i[:, None]) % 32 == 5, 16384, 4), gap=4)
    print("long blocks a radix apart", P, radix, flush=True)
    args = (send, meta[0], meta[1], recv, meta[2], meta[3], P, 0, radix, radix)
    o = tuna.tuna_opts_init()
    o.mode, o.t_layout = tuna.TUNA_MODE_STAGED, tuna.TUNA_T_EXACT
    assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
    torch.cuda.synchronize()
    reference = recv.clone()
    recv.zero_()
    o.mode = tuna.TUNA_MODE_FUSED
    assert tuna.tuna_alltoallv_ex(None, *args, o) == 0
    torch.cuda.synchronize()
    bit = {E: tuna.TUNA_HOP_ENGINE, R: tuna.TUNA_HOP_ROWS}
    assert torch.equal(recv, reference) and tuna.tuna_get_stats().hop_kernels == bit[want]
    rc, plan = tuna.tuna_alltoallv_init_ex(None, *args, o)
    assert rc == 0
    try:
        recv.zero_()
        assert tuna.tuna_start(plan) == 0
        torch.cuda.synchronize()
        assert torch.equal(recv, reference) and tuna.tuna_get_stats().hop_kernels == bit[plan_want]
    finally:
        assert tuna.tuna_plan_free(plan) == 0
    tuna.tuna_release()


@pytest.mark.parametrize("P,longest,quantum,radix,opts,call,plan_kernel", [
    (1024, 200, 1, 16, {}, D, D), (1536, 200, 1, 16, {}, R, R),            # 100 and 225 MiB in three phases
    (2048, 60, 4, 16, {}, D, D),                                          # blocks of up to 64 bytes, whatever the payload
    (1536, 128, 16, 1536, {}, D, D), (2048, 144, 16, 2048, {}, R, R),     # one phase: 144 and 288 MiB, chunk-granular
    (2048, 200, 1, 2048, {}, D, D),                                       # and 400 MiB, byte-granular
    (1536, 200, 1, 4, {"Q": 32, "gap": 3, "permute": 7}, R, R), (1536, 256, 4, 8, {"slots": 1, "gap": 8, "permute": 8}, R, R),
    (1536, 128, 128, 12, {"Q": 128}, R, R),                               # whole lines
    (2048, 256, 4, 4, {"staggered": 1}, E, E), (2048, 200, 1, 4, {"staggered": 1}, D, D),
    (1024, 256, 4, 32, {"block_count": 9}, D, D), (1536, 256, 4, 32, {"block_count": 9}, E, E),
    (512, 256, 4, 512, {"to": 3}, D, E), (512, 256, 4, 16, {"from": 3}, D, E), (512, 256, 4, 512, {"from": 3}, D, D),
    (512, 256, 4, 16, {"share": 64}, D, D), (512, 64, 4, 512, {"to": 3}, D, D)])
def test_hop_of_short_blocks(tuna, P, longest, quantum, radix, opts, call, plan_kernel):
    counts = wl.counts_uniform_elements(P, P + longest, longest // quantum, quantum)
    i = np.arange(P)
    if "to" in opts:                                        # one receiver, one sender, one pair in so many
        counts = np.where(np.broadcast_to(i[None, :] == opts["to"], (P, P)), longest, 0)
    if "from" in opts:
        counts = np.where(np.broadcast_to(i[:, None] == opts["from"], (P, P)), longest, 0)
    if "share" in opts:
        counts = np.where((i[:, None] * 37 + i[None, :] * 11) % opts["share"] == 0, longest, 0)
    Q = 16 if "staggered" in opts else opts.get("Q", 0)
    lay, send, meta, recv = _device_problem(P, counts, opts.get("gap", 0), opts.get("permute"))
    args = (send, meta[0], meta[1], recv, meta[2], meta[3], P, Q, radix, radix)
    print("hop of short blocks", P, longest, quantum, radix, opts, lay.payload_bytes >> 20, "MiB", flush=True)
    bit = {E: tuna.TUNA_HOP_ENGINE, D: tuna.TUNA_HOP_DIRECT, R: tuna.TUNA_HOP_ROWS}

    def options(mode):
        o = tuna.tuna_opts_init()
        o.mode, o.t_layout = mode, tuna.TUNA_T_SLOTS if "slots" in opts else tuna.TUNA_T_EXACT
        if mode == tuna.TUNA_MODE_FUSED:
            o.staggered, o.block_count = opts.get("staggered", 0), opts.get("block_count", 0)
        return o

    assert tuna.tuna_alltoallv_ex(None, *args, options(tuna.TUNA_MODE_STAGED)) == 0
    torch.cuda.synchronize()
    want = recv.clone()
    recv.zero_()
    assert tuna.tuna_alltoallv_ex(None, *args, options(tuna.TUNA_MODE_FUSED)) == 0
    torch.cuda.synchronize()
    assert torch.equal(recv, want) and tuna.tuna_get_stats().hop_kernels == bit[call]
    rc, plan = tuna.tuna_alltoallv_init_ex(None, *args, options(tuna.TUNA_MODE_FUSED))
    assert rc == 0, tuna.tuna_strerror(rc)
    try:
        recv.zero_()
        assert tuna.tuna_start(plan) == 0
        torch.cuda.synchronize()
        assert torch.equal(recv, want) and tuna.tuna_get_stats().hop_kernels == bit[plan_kernel]
    finally:
        assert tuna.tuna_plan_free(plan) == 0
    tuna.tuna_release()

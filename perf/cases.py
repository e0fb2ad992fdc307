"""The calls a program makes of this library, from the smallest to the largest, and how each is timed.

Every case is one non-uniform all-to-all of P virtual ranks whose buffers lie in one GPU's memory: `prepare`
makes the counts, displacements and payload on the GPU, `run` is one pass through a public entry point, and the
result is the whole receive buffer.  Sizes and distributions are those of this repository's configurations
(`workloads/`), its benchmark and its tests.

Fields of a case
  entry           call: the immediate flat call; hier: the immediate call with both radices and ranks per node;
                  staged: the immediate call with the three steps of the paper kept apart (an option of the call);
                  noalloc: the call for programs that may not allocate; plan: a start of a persistent plan
  P, ranks_per_node, radix, global_radix   (radix 0: left to the library)
  sizes, bytes    distribution of the block sizes and its parameter:
                  uniform  elements U{0 .. bytes / quantum};  normal  mean `bytes`, deviation a quarter of it;
                  zipf  power law s = 1.2 up to `bytes`;  constant  `bytes` everywhere;
                  fft_n1 / fft_n2  the sparse and the nearly uniform pattern of a distributed FFT's transposes
  quantum         element size: all counts are multiples of it
  align           1: blocks lie back to back (the usual MPI layout); 16: every block starts on 16 bytes
"""
from __future__ import annotations

import math
import weakref

import torch

import paper_2411_02581_amd as tuna

DEVICE = "cuda:0"


def _case(name, entry, P, sizes, size_bytes, quantum, radix=0, ranks_per_node=0, global_radix=0, align=1):
    case = {"entry": entry, "P": P, "ranks_per_node": ranks_per_node, "radix": radix, "global_radix": global_radix,
            "sizes": sizes, "bytes": size_bytes, "quantum": quantum, "align": align}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a handful of ranks that exchange a few integers each: what a call costs before any byte moves
        _case("call_16_int32_r2", "call", 16, "uniform", 256, 4, radix=2),
        # the same regime for a serving loop that may not allocate; an odd number of ranks
        _case("noalloc_200_words_r16", "noalloc", 200, "uniform", 240, 4, radix=16),
        # byte strings of any length and alignment between a few hundred ranks: fits into the caches
        _case("call_256_bytes_r4", "call", 256, "uniform", 1024, 1, radix=4),
        # byte strings again, large enough for HBM, exchanged again and again with one set of counts
        _case("plan_1000_bytes", "plan", 1000, "uniform", 1024, 1),
        # few ranks with large float blocks (a repartitioning of arrays)
        _case("call_60_large", "call", 60, "uniform", 1 << 20, 4),
        # skewed graph-like traffic on a hierarchy of 64 nodes of 16 ranks: a fifth of the blocks empty, rare large ones
        _case("hier_1024_zipf_r4_r8", "hier", 1024, "zipf", 16384, 4, radix=4, ranks_per_node=16, global_radix=8),
        # the degenerate uniform exchange on a hierarchy
        _case("hier_2048_const_r16", "hier", 2048, "constant", 256, 256, radix=16, ranks_per_node=32, global_radix=16),
        # many ranks, one or two doubles per pair: the small-message regime the tunable radix is for
        _case("call_2048_tiny_r46", "call", 2048, "uniform", 16, 8, radix=46),
        # the paper's three steps kept apart
        _case("staged_1024_normal_r32", "staged", 1024, "normal", 1024, 4, radix=32),
        # the sparse transpose of an FFT over very many ranks
        _case("call_8192_fft", "call", 8192, "fft_n1", 64, 64),
        # the headline problem, 16 GiB, in four digit phases and in one
        _case("call_4096_normal_r8", "call", 4096, "normal", 1024, 4, radix=8),
        _case("call_4096_normal_linear", "call", 4096, "normal", 1024, 4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any entry point, rank counts and sizes spread over their logarithms, at most 4 GiB of payload."""
    entry = rng.choice(("call", "call", "call", "hier", "hier", "plan", "plan", "staged", "noalloc"))
    rpn = grx = 0
    if entry == "hier":
        rpn, nodes = _log_int(rng, 2, 64), _log_int(rng, 2, 64)
        P = rpn * nodes
        grx = rng.choice((2, 4, 8, nodes, 0))
    else:
        P = _log_int(rng, 8, 256) if entry == "noalloc" else _log_int(rng, 8, 4096)
    radix = rng.choice((2, 3, 4, 8, 16, max(2, int(round(math.sqrt(P)))), 0, 0))
    if entry == "call" and P >= 256 and rng.random() < 0.15:
        name = rng.choice(("fft_n1", "fft_n2"))
        return _case(None, entry, P, name, 64 if name == "fft_n1" else 512, 64, radix=radix)
    most = {"noalloc": 4 << 20, "staged": 1 << 30}.get(entry, 4 << 30)          # payload of the largest such case
    mean = math.exp(rng.uniform(math.log(8), math.log(max(9.0, min(1 << 20, most / P / P)))))
    sizes = rng.choice(("uniform", "uniform", "normal", "zipf", "constant"))
    quantum = rng.choice((1, 4, 4, 8, 16)) if mean >= 64 else rng.choice((1, 4, 8))
    size = {"uniform": 2 * mean, "zipf": 16 * mean}.get(sizes, mean)
    size = max(quantum, min(int(size) // quantum * quantum, 1 << 22))
    if sizes == "constant":
        quantum = size
    return _case(None, entry, P, sizes, size, quantum, radix=radix, ranks_per_node=rpn, global_radix=grx,
                 align=rng.choice((1, 1, 1, 16)))


def _zipf_weights(case):
    k = torch.arange(1, case["bytes"] // case["quantum"] + 2, dtype=torch.float64)
    w = k ** -1.2
    return w / w.sum()


def _counts(case, gen):
    P, size, q = case["P"], case["bytes"], case["quantum"]
    kind = case["sizes"]
    if kind == "uniform":
        return torch.randint(0, size // q + 1, (P, P), generator=gen, device=DEVICE, dtype=torch.int32) * q
    if kind == "normal":
        v = torch.randn((P, P), generator=gen, device=DEVICE).mul_(size / 4.0).add_(size).clamp_(min=0.0)
        return v.div_(q).round_().to(torch.int32) * q
    if kind == "zipf":
        cdf = torch.cumsum(_zipf_weights(case), 0).to(DEVICE)
        u = torch.rand((P, P), generator=gen, device=DEVICE, dtype=torch.float64)
        return torch.searchsorted(cdf, u).clamp_(max=cdf.numel() - 1).to(torch.int32) * q
    c = torch.full((P, P), size, dtype=torch.int32, device=DEVICE)
    if kind == "fft_n1":
        c[math.ceil(0.625 * P):] = 0
        c[:, math.ceil(0.78125 * P):] = 0
    elif kind == "fft_n2":
        c[P - 1] = size // 4
    return c


def _moments(case):
    """Mean and standard deviation of one block's bytes, and the most it can have."""
    size, q, kind = case["bytes"], case["quantum"], case["sizes"]
    if kind == "uniform":
        n = size // q
        return n * q / 2.0, q * math.sqrt(n * (n + 2) / 12.0), n * q
    if kind == "normal":
        return float(size), size / 4.0 + q, 3 * size
    if kind == "zipf":
        w = _zipf_weights(case)
        k = torch.arange(w.numel(), dtype=torch.float64) * q
        mean = float((w * k).sum())
        return mean, math.sqrt(float((w * k * k).sum()) - mean * mean), int(k[-1])
    return float(size), 0.0, size


def _capacity(case):
    """Bytes of the program's buffers: what P x P blocks of the distribution take, with room for their spread."""
    n, (mean, sd, most) = case["P"] ** 2, _moments(case)
    if case["align"] > 1:
        mean, most = mean + case["align"], most + case["align"]
    room = min(n * most, n * mean + 10 * math.sqrt(n) * sd + 4 * most)
    return (int(room) // 4096 + 1) * 4096


def _displs(counts, align):
    """Offsets of the blocks, row after row, every start rounded up to `align` bytes; and where each ends."""
    step = counts.reshape(-1).to(torch.int64)
    if align > 1:
        step = (step + align - 1) // align * align
    end = torch.cumsum(step, 0)
    return (end - step).reshape(counts.shape), end.reshape(counts.shape)


class Problem:
    """One problem resident on the GPU, and for a persistent case its plan."""

    def __init__(self, case, seed):
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(seed)
        self.P, self.entry = case["P"], case["entry"]
        self.ranks_per_node, self.radix, self.global_radix = case["ranks_per_node"], case["radix"], case["global_radix"]
        room = _capacity(case)
        self.sendcounts = _counts(case, gen)
        self.sdispls, end = _displs(self.sendcounts, case["align"])
        self.sendcounts.masked_fill_(end > room, 0)        # (next to never: what does not fit is not sent)
        self.recvcounts = self.sendcounts.t().contiguous()
        self.rdispls, _ = _displs(self.recvcounts, case["align"])
        self.send = torch.empty(room // 8, dtype=torch.int64, device=DEVICE).random_(generator=gen)
        self.recv = torch.zeros(room // 8, dtype=torch.int64, device=DEVICE)
        self.opts = self.plan = None
        if self.entry == "staged":
            self.opts = tuna.tuna_opts_init()
            self.opts.mode = tuna.TUNA_MODE_STAGED
        if self.entry == "plan":
            rc, self.plan = tuna.tuna_alltoallv_init(*self.arrays(), self.P, self.ranks_per_node, self.radix, self.radix)
            _check(rc)
            weakref.finalize(self, tuna.tuna_plan_free, self.plan)

    def arrays(self):
        return self.send, self.sendcounts, self.sdispls, self.recv, self.recvcounts, self.rdispls


def _check(rc):
    if rc != tuna.TUNA_OK:
        raise RuntimeError(tuna.tuna_strerror(rc))


def prepare(case, seed):
    return Problem(case, seed)


def run(state):
    s = state
    if s.entry == "plan":
        _check(tuna.tuna_start(s.plan))
    elif s.entry == "call":
        _check(tuna.tuna_alltoallv(*s.arrays(), s.P, s.radix))
    elif s.entry == "hier":
        _check(tuna.tuna_alltoallv_hier(*s.arrays(), s.P, s.ranks_per_node, s.radix, s.global_radix))
    elif s.entry == "staged":
        _check(tuna.tuna_alltoallv_ex(None, *s.arrays(), s.P, 0, s.radix, s.radix, s.opts))
    else:
        _check(tuna.tuna_alltoallv_noalloc(*s.arrays(), s.P, 0, s.radix, s.radix))
    return s.recv


def work(case):
    """The payload read once and written once; an immediate call also reads the four matrices (24 bytes per pair)."""
    P = case["P"]
    payload = P * P * _moments(case)[0]
    if case["sizes"] == "fft_n1":
        payload = math.ceil(0.625 * P) * math.ceil(0.78125 * P) * case["bytes"]
    return {"bytes": 2.0 * payload + (0.0 if case["entry"] == "plan" else 24.0 * P * P), "flops": 0.0}


def tolerance(case):
    return "exact"                       # bytes are moved: every one of them has to arrive

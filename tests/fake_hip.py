"""The library's host code on the runtime of fake_hip.cpp.  `python fake_hip.py <runtime> <case> [arguments]` runs one
case of CASES in a process of its own (the real runtime must not be loaded) and prints its result as JSON; `run` does so."""
import ctypes
import json
import os
import re
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def build(folder):
    """The runtime, under the name that the library asks for."""
    out = os.path.join(folder, "libamdhip64.so.7")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-Wl,-soname,libamdhip64.so.7", "-o", out, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return out


def run(runtime, case, *args):
    p = subprocess.run([sys.executable, os.path.abspath(__file__), runtime, case, json.dumps(args)], stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads(p.stdout.splitlines()[-1])


class Lib:
    """The library on that runtime; problems whose payload is never read."""

    def __init__(self, runtime):
        self.fake = ctypes.CDLL(runtime, mode=ctypes.RTLD_GLOBAL)
        for name, res, args in (("fake_notes", ctypes.c_int, []), ("fake_name", ctypes.c_char_p, [ctypes.c_int]),
                                ("fake_stream", ctypes.c_long, [ctypes.c_int]), ("fake_ptr", ctypes.c_size_t, [ctypes.c_int]),
                                ("fake_end", ctypes.c_size_t, [ctypes.c_int]),
                                ("fake_before", ctypes.c_long, [ctypes.c_int, ctypes.c_long]),
                                ("fake_waited", ctypes.c_long, [ctypes.c_long]), ("fake_length", ctypes.c_long, [ctypes.c_long]), ("fake_violations", ctypes.c_int, []),
                                ("fake_allocated", ctypes.c_ulonglong, [])):
            f = getattr(self.fake, name)
            f.restype, f.argtypes = res, args
        sys.path.insert(0, ROOT)
        import paper_2411_02581_amd.binding as b
        import workloads
        self.b, self.wl, self.lib = b, workloads, b.load()

    def problem(self, counts, **layout):
        lay = self.wl.make_layout(np.ascontiguousarray(counts, dtype=np.int32), **layout)
        return lay, [0x7000000000] + [a.ctypes.data for a in (lay.sendcounts, lay.sdispls)] + [0x7800000000] + \
            [a.ctypes.data for a in (lay.recvcounts, lay.rdispls)]

    def options(self, **fields):
        o = self.b.tuna_opts_t()
        assert self.lib.tuna_opts_init(ctypes.byref(o)) == 0
        o.mode = self.b.TUNA_MODE_FUSED                        # not the single launch
        for k, v in fields.items():
            setattr(o, k, v)
        return o

    def call(self, prob, radix, stream, rpn=0, rg=None, ctx=None, **fields):
        return self.lib.tuna_alltoallv_ex(ctx, *prob[1], prob[0].P, rpn, radix, rg or radix, ctypes.byref(self.options(**fields)), stream)

    def plan(self, prob, radix, stream, rpn=0, rg=None, ctx=None, **fields):
        plan = ctypes.c_void_p(None)
        rc = self.lib.tuna_alltoallv_init_ex(ctx, *prob[1], prob[0].P, rpn, radix, rg or radix, ctypes.byref(self.options(**fields)), stream,
                                             ctypes.byref(plan))
        assert rc == 0, rc
        return plan

    def kernels(self, first=0):
        """[name, stream, template arguments] of the kernels launched from note `first` on."""
        out = []
        for i in range(first, self.fake.fake_notes()):
            name = self.fake.fake_name(i).decode()
            n, at = re.search(r"(\d+)k_", name).group(1), name.index("k_")
            n = next(int(n[j:]) for j in range(len(n)) if n[j] != "0" and at + int(n[j:]) <= len(name))
            args = re.match(r"I((?:L[a-z]+\d+E)+)E", name[at + n:])
            out.append([name[at:at + n], self.fake.fake_stream(i), [int(v) for v in re.findall(r"L[a-z]+(\d+)E", args.group(1))] if args else []])
        return out


def _engine_counts(P):
    """Short blocks and a few that are too long for the kernels that find their blocks themselves: the copy engine's hop."""
    c = np.random.default_rng(P).integers(0, 300, (P, P)).astype(np.int32)
    c[1, P - 2] = c[P - 1, 3] = 70001
    return c


S1, S2, S3 = 0x1000, 0x2000, 0x3000


def case_upload(t, P, radix, then):
    """A call that sends the places of T's classes to the device, and behind it, before the copy is done, another operation
    on the context."""
    prob = t.problem(_engine_counts(P), gap=1)
    assert t.call(prob, radix, S1, t_layout=t.b.TUNA_T_EXACT) == 0
    if then == "call":
        other = t.problem(_engine_counts(P) * 2, gap=1)
        assert t.call(other, radix, S1, t_layout=t.b.TUNA_T_EXACT) == 0
    elif then == "call elsewhere":
        assert t.call(prob, radix, S2, t_layout=t.b.TUNA_T_EXACT) == 0
    elif then == "query":
        n = ctypes.c_size_t(0)
        assert t.lib.tuna_workspace_bytes(prob[1][1], P, 0, radix, radix, ctypes.byref(n)) == 0
    elif then == "plan":
        t.plan(t.problem(_engine_counts(P) * 2, gap=1), radix, S2, t_layout=t.b.TUNA_T_EXACT)
    return {"violations": t.fake.fake_violations()}


def case_plan_status(t, counts, P, radix, plan_counts, plan_P, plan_radix):
    """A plan is made on one stream while a call of the same context is in flight on another: do its kernels write into the
    status block that the call uses?"""
    sizes = {"long": lambda P: np.full((P, P), 40000), "engine": _engine_counts}
    assert t.call(t.problem(sizes[counts](P)), radix, S1) == 0
    status = [t.fake.fake_ptr(i) for i, k in enumerate(t.kernels()) if k[0] == "k_validate"][0]
    first = t.fake.fake_notes()
    t.plan(t.problem(sizes[plan_counts](plan_P)), plan_radix, S2)
    words = [(k[0], t.fake.fake_ptr(first + i)) for i, k in enumerate(t.kernels(first)) if k[0] in ("k_zero64", "k_layout_base")]
    # (sums of classes, which the plan's validation leaves as it finds them, are the first 16 KiB and 64 bytes)
    return {"seen": len(words), "shared": [n for n, p in words if status <= p < status + 32768]}


def case_order(t, between, P, radix):
    """A call, something else that leaves it in flight, and a call on another stream: is that one's first kernel behind the
    first call?"""
    prob = t.problem(np.full((P, P), 300), gap=1)
    nothing = t.problem(np.zeros((P, P)), gap=1)
    plans = [t.plan(nothing, 2, S3), t.plan(prob, radix, S3, profile=1)]
    assert t.call(prob, radix, S1) == 0
    length = t.fake.fake_length(S1)
    if between == "ranks per node":
        assert t.call(prob, radix, S2, rpn=7) == t.b.TUNA_ERR_ARG
    elif between == "no counts":
        assert t.call((prob[0], [None] * 6), radix, S3) == t.b.TUNA_ERR_ARG
    elif between == "refused":
        wrong = t.problem(np.full((P, P), 300), gap=1)
        wrong[0].sendcounts[1, 2] += 4
        assert t.call(wrong, radix, S3) == t.b.TUNA_ERR_COUNT_MISMATCH
    elif between == "empty":
        assert t.call(nothing, radix, S3) == 0
    elif between == "empty start":
        assert t.lib.tuna_start(plans[0], S3) == 0
    elif between == "profiled start":
        assert t.lib.tuna_start(plans[1], S3) == 0
    elif between == "profiled start there":
        assert t.lib.tuna_start(plans[1], S2) == 0
    elif between == "noalloc":
        assert t.lib.tuna_alltoallv_noalloc(*prob[1], P, 0, radix, radix, S3) == 0
    elif between == "query":
        n = ctypes.c_size_t(0)
        assert t.lib.tuna_workspace_bytes(prob[1][1], P, 0, radix, radix, ctypes.byref(n)) == 0
    first = t.fake.fake_notes()
    assert t.call(prob, radix, S2) == 0
    assert t.fake.fake_stream(first) == S2
    return {"behind": t.fake.fake_before(first, S1) >= length > 0}


def case_plan_bytes(t, P, size, radix, t_layout):
    prob = t.problem(np.full((P, P), size), gap=1)
    plan = t.plan(t.problem(np.full((P, P), 0)), radix, S1)     # (the context, and the schedule's tables)
    assert t.lib.tuna_plan_free(plan) == 0
    before = t.fake.fake_allocated()
    plan = t.plan(prob, radix, S1, t_layout=t_layout)
    took = t.fake.fake_allocated() - before
    st = t.b.tuna_stats_t()
    assert t.lib.tuna_start(plan, S1) == 0 and t.lib.tuna_get_stats(ctypes.byref(st)) == 0
    assert st.hop_kernels == t.b.TUNA_HOP_LONG
    return {"phases": st.n_phases, "meta": took - st.temp_bytes, "said": st.workspace_bytes - took}


def case_recording(t, P, radix, plan):
    """A call or the making of a plan on a stream that is being recorded into a graph, and again when it is not: the kernels
    that fill the schedule's tables the second time."""
    prob = t.problem(np.full((P, P), 300), gap=1)
    assert t.call(prob, P, S1) == 0                            # (the context is made)
    t.fake.fake_record(S1, 1)
    rc = t.lib.tuna_alltoallv_init(*prob[1], P, 0, radix, radix, S1, ctypes.byref(ctypes.c_void_p(None))) if plan else t.call(prob, radix, S1)
    t.fake.fake_record(S1, 0)
    first = t.fake.fake_notes()
    assert t.call(prob, radix, S1) == 0
    return {"refused": rc == t.b.TUNA_ERR_HIP, "tables": [k[0] for k in t.kernels(first)].count("k_build_tables")}


def case_routes(t, problems, plan):
    """The payload kernels of each of `problems` and the kernels of their places in T."""
    out = []
    for P, rpn, rl, rg, longest, q, t_layout, layout, *more in problems:
        options = dict(more[0] if more else {}, t_layout=t_layout)
        counts = np.random.default_rng(P).integers(0, longest // q + 1, (P, P)) * q
        counts[0, P - 1] = longest
        prob = t.problem(counts, **layout)
        first = t.fake.fake_notes()
        if plan:
            p = t.plan(prob, rl, S1, rpn=rpn, rg=rg, **options)
            first = t.fake.fake_notes()
            assert t.lib.tuna_start(p, S1) == 0
        else:
            assert t.call(prob, rl, S1, rpn=rpn, rg=rg, **options) == 0
        out.append([[k[0], k[2]] for k in t.kernels(first) if k[0].startswith(("k_hop", "k_copy", "k_t_", "k_self_copy"))])
        assert t.lib.tuna_release() == 0 or plan
    return out


def case_sequence(t, seed, steps):
    """Random operations on two contexts and three streams; kernels of immediate calls that are not behind every earlier call of
    their context, and copies whose source was overwritten."""
    rng = np.random.default_rng(seed)
    big = _engine_counts(100)
    big[big > 0] += 8000                                       # 64 MiB and more: metadata on a second stream, or two passes
    kinds = {"short": (np.full((90, 90), 40), {}), "rows": (np.full((50, 50), 900), {"gap": 1}), "engine": (_engine_counts(64), {"gap": 1}),
             "many phases": (_engine_counts(300), {}), "long": (np.full((24, 24), 50000), {}), "pipelined": (big, {"gap": 1})}
    probs = {k: t.problem(c, **lay) for k, (c, lay) in kinds.items()}
    nothing = t.problem(np.zeros((50, 50)))
    wrong = t.problem(np.full((50, 50), 900))
    wrong[0].sendcounts[1, 2] += 4
    rc, other = t.b.tuna_ctx_create()
    assert rc == 0
    ends, plans, late, calls = {None: [], other: []}, [], [], 0
    names = list(probs)
    for step in range(steps):
        ctx, s = (None, other)[rng.integers(2)], int(rng.choice([S1, S2, S3]))
        what = rng.choice(["call"] * 4 + ["refused", "empty", "bad", "plan", "start", "start", "free", "query", "noalloc", "stats"])
        kind, radix = names[rng.integers(len(names))], int(rng.choice([2, 3, 8, 14, 400]))
        first = t.fake.fake_notes()
        if what == "call":
            calls += 1
            mode = t.b.TUNA_MODE_STAGED if rng.random() < 0.2 else t.b.TUNA_MODE_FUSED
            assert t.call(probs[kind], radix, s, ctx=ctx, mode=mode, t_layout=int(rng.integers(3)), profile=int(rng.random() < 0.2)) == 0
            for i, k in enumerate(t.kernels(first)):
                if not k[0].startswith("k_build"):             # (a new schedule's tables)
                    late += [[step, kind, k[0]] for stream, upto in ends[ctx] if stream != k[1] and t.fake.fake_before(first + i, stream) < upto]
            ends[ctx].append((s, t.fake.fake_length(s)))
        elif what == "refused":
            assert t.call(wrong, radix, s, ctx=ctx) == t.b.TUNA_ERR_COUNT_MISMATCH
        elif what == "empty":
            assert t.call(nothing, radix, s, ctx=ctx) == 0
        elif what == "bad":
            assert t.call((nothing[0], [None] * 6), radix, s, ctx=ctx) == t.b.TUNA_ERR_ARG
        elif what == "plan":
            prob = nothing if rng.random() < 0.2 else probs[kind]
            plans.append(t.plan(prob, radix, s, ctx=ctx, t_layout=int(rng.integers(3)), profile=int(rng.random() < 0.5)))
        elif what == "start" and plans:
            assert t.lib.tuna_start(plans[rng.integers(len(plans))], s) == 0
        elif what == "free" and plans and rng.random() < 0.3:  # (waits for the device)
            assert t.lib.tuna_plan_free(plans.pop()) == 0
        elif what == "query":
            assert t.lib.tuna_workspace_bytes(probs[kind][1][1], probs[kind][0].P, 0, radix, radix, ctypes.byref(ctypes.c_size_t(0))) == 0
        elif what == "noalloc":
            assert t.lib.tuna_alltoallv_noalloc(*probs["short"][1], probs["short"][0].P, 0, radix, radix, s) == 0
        elif what == "stats" and rng.random() < 0.2:           # (waits for the call)
            assert t.lib.tuna_ctx_get_stats(ctx, ctypes.byref(t.b.tuna_stats_t())) == 0
    return {"calls": calls, "late": late[:5], "violations": t.fake.fake_violations()}


def case_early(t, calls):
    """The kernels of each of `calls` in turn, [P, radix, longest block, mode], without those of new schedules; and whether the host has
    waited for them all when the call returns."""
    out = []
    for P, radix, longest, staged, wrong in calls:
        counts = np.random.default_rng(P).integers(0, longest + 1, (P, P))
        counts[0, P - 1] = longest
        prob = t.problem(counts, gap=1)
        if wrong:
            prob[0].sendcounts[1, 2] += 4
        first = t.fake.fake_notes()
        rc = t.call(prob, radix, S1, mode=t.b.TUNA_MODE_STAGED if staged else t.b.TUNA_MODE_FUSED, t_layout=t.b.TUNA_T_EXACT)
        assert rc == (t.b.TUNA_ERR_COUNT_MISMATCH if wrong else 0)
        done = t.fake.fake_length(S1)
        out.append([[k[0] for k in t.kernels(first) if not k[0].startswith("k_build")], None])
        nothing = t.problem(np.zeros((4, 4)))
        at = t.fake.fake_notes()
        assert t.call(nothing, 2, S2) == 0                     # (its first kernel is behind what the host has waited for)
        out[-1][1] = t.fake.fake_before(at, S1) >= done
    return out


def case_no_places(t, P, radix, before):
    """The return code and kernels of a call whose blocks never wait in T: behind one of `before`, [ranks, radix], that leaves memory; with none,
    as the call that allocates nothing."""
    prob = t.problem(np.full((P, P), 40))
    if before:
        assert t.call(t.problem(np.full((before[0], before[0]), 40)), before[1], S1) == 0
    first = t.fake.fake_notes()
    rc = t.call(prob, radix, S1) if before else t.lib.tuna_alltoallv_noalloc(*prob[1], P, 0, radix, radix, S1)
    return [rc, [k[0] for k in t.kernels(first) if not k[0].startswith("k_build")]]


def case_small_workspace(t, kind, P, radix):
    """A call on a caller's workspace of 4 MiB, which holds its metadata and not T: its kernels, and whether the host has waited for them."""
    counts = {"one pass": np.full((P, P), 300), "pipelined": _engine_counts(P) + 8000, "two passes": _engine_counts(P) + 8000}[kind]
    prob = t.problem(counts, gap=1)
    assert t.call(t.problem(np.full((4, 4), 40)), 2, S1) == 0                  # (a context's first call has no early kernels)
    room = np.zeros((4 << 20) + 256, np.uint8)
    assert t.lib.tuna_set_workspace(room.ctypes.data + -room.ctypes.data % 256, 4 << 20) == 0
    first = t.fake.fake_notes()
    if kind == "two passes":
        t.fake.fake_no_streams()
    assert t.call(prob, radix, S1, t_layout=t.b.TUNA_T_EXACT) == t.b.TUNA_ERR_WORKSPACE_TOO_SMALL
    return [[k[0] for k in t.kernels(first)], t.fake.fake_waited(S1) >= t.fake.fake_length(S1)]


def case_single_launch(t, calls):
    """Whether each of `calls`, [kind, radix], all of 12 ranks and with inputs of their own, asked k_tiny_call (which declines everything here)."""
    out, keep = [], []
    for kind, radix in calls:
        keep.append(t.problem(np.full((12, 12), 9000 if kind == "large" else 40)))
        lay = keep[-1][0]
        if kind in ("far in S", "far in R"):
            (lay.sdispls if kind == "far in S" else lay.rdispls)[3:] += 1 << 32
        first = t.fake.fake_notes()
        assert t.call(keep[-1], radix, S1, mode=t.b.TUNA_MODE_FUSED if kind == "own options" else t.b.TUNA_MODE_AUTO) == 0
        out.append("k_tiny_call" in [k[0] for k in t.kernels(first)])
    return out


def case_early_use(t, P, radix, calls, noalloc):
    """Whether each of `calls` on one schedule -- "direct", "engine", "staged", "slots" -- launched early kernels: behind validation and ahead of
    what needs its result."""
    short, engine = t.problem(np.full((P, P), 40), gap=1), t.problem(_engine_counts(P), gap=1)
    out = []
    for kind in ["direct"] + calls:
        prob = engine if kind == "engine" else short
        first = t.fake.fake_notes()
        if noalloc:
            assert t.lib.tuna_alltoallv_noalloc(*prob[1], P, 0, radix, radix, S1) == 0
        else:
            assert t.call(prob, radix, S1, mode=t.b.TUNA_MODE_STAGED if kind == "staged" else t.b.TUNA_MODE_FUSED,
                          t_layout=t.b.TUNA_T_SLOTS if kind == "slots" else t.b.TUNA_T_EXACT) == 0
        kernels = [k[0] for k in t.kernels(first)]
        validated = max(i for i, k in enumerate(kernels) if k.startswith("k_validate"))
        # (k_t_bases and the hops' partial sums tell a direct call that found its places early from one that did not)
        out.append(kernels[validated + 1].startswith(("k_t_places", "k_row_totals")) and "k_phase_sums" not in kernels)
    return out[1:]


def case_rows_of_validation(t, units, P, radix):
    """The call that allocates nothing on a device of so many compute units: where the rows that validation writes end, and where the schedule's
    tables begin."""
    t.fake.fake_units(units)
    prob, first = t.problem(np.full((P, P), 4)), t.fake.fake_notes()
    assert t.lib.tuna_alltoallv_noalloc(*prob[1], P, 0, radix, radix, S1) == 0
    names = [k[0] for k in t.kernels(first)]
    return [t.fake.fake_end(first + names.index("k_validate")), t.fake.fake_ptr(first + names.index("k_build_tables"))]


def case_stream_gone(t, kind, P, radix, plan, first):
    """The return code of a call, or of the making of a plan, on a stream after the one that the schedule was first used on has been destroyed, or
    is being recorded."""
    prob = t.problem(_engine_counts(P) if kind == "engine" else np.full((P, P), 300), gap=1)
    fields = {"mode": t.b.TUNA_MODE_STAGED if kind == "staged" else t.b.TUNA_MODE_FUSED, "t_layout": t.b.TUNA_T_SLOTS if kind == "slots" else t.b.TUNA_T_EXACT}
    assert t.call(prob, radix, S1, **fields) == 0
    if first == "destroyed":
        t.fake.fake_destroy(S1)
    else:
        t.fake.fake_record(S1, 1)
    if plan:
        handle = ctypes.c_void_p(None)
        return t.lib.tuna_alltoallv_init_ex(None, *prob[1], P, 0, radix, radix, ctypes.byref(t.options(**fields)), S2, ctypes.byref(handle))
    return t.call(prob, radix, S2, **fields)


def case_verdict(t, P, radix):
    """Where the kernels that a call launches ahead of the host look up what validation found, from the status block on."""
    prob = t.problem(np.random.default_rng(P).integers(0, 60, (P, P)))
    assert t.call(prob, radix, S1) == 0
    first = t.fake.fake_notes()
    assert t.call(prob, radix, S1) == 0
    names = [k[0] for k in t.kernels(first)]
    status = t.fake.fake_ptr(first + names.index("k_validate"))
    early = [i for i, k in enumerate(names) if k.startswith("k_t_places") or k == "k_row_totals"]
    assert len(early) == 1
    ptr = t.fake.fake_ptr(first + early[0])
    return ["k_validate_finish" in names, ptr - status if ptr else None]


def case_schedules(t, problems, plan):
    """How many schedules each of `problems` (as in case_routes) makes."""
    out = []
    for P, rpn, rl, rg, longest, q, t_layout, layout in problems:
        prob = t.problem(np.random.default_rng(P).integers(0, longest // q + 1, (P, P)) * q, **layout)
        first = t.fake.fake_notes()
        if plan:
            assert t.lib.tuna_plan_free(t.plan(prob, rl, S1, rpn=rpn, rg=rg, t_layout=t_layout)) == 0
        else:
            assert t.call(prob, rl, S1, rpn=rpn, rg=rg, t_layout=t_layout) == 0
        out.append([k[0] for k in t.kernels(first)].count("k_build_tables"))
        assert t.lib.tuna_release() == 0
    return out


CASES = {k[5:]: f for k, f in list(globals().items()) if k.startswith("case_")}

if __name__ == "__main__":
    lib = Lib(sys.argv[1])
    print(json.dumps(CASES[sys.argv[2]](lib, *json.loads(sys.argv[3]))))

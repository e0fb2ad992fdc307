// Device kernels of the tunable-radix all-to-all for gfx950 (wave64).
//
// All kernels are pure data movement or 32/64-bit integer index arithmetic; none uses MFMA.
// Staging buffers are addressed in 16-byte "chunks": every block is padded to a whole number of
// chunks in staging, so staging accesses are always aligned dwordx4 and the only unaligned
// accesses are to the caller's send / receive buffers.
#pragma once
#include <hip/hip_runtime.h>
#include <climits>
#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "tuna_plan.h"

namespace tuna {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));   // one 16-byte chunk

// Shape of the copy kernels' work, chosen by measurement on MI355X: workgroups of 64, 128, 512 and
// 1024 threads and 2 or 8 chunks per lane were all slower than 256 threads x 4 chunks.
constexpr int kWave = 64;
constexpr int kCopyThreads = 256;                        // 4 waves, each an independent work unit
constexpr int kChunksPerLane = 4;
constexpr int kUnitChunks = kWave * kChunksPerLane;      // 256 chunks = 4 KiB per wave unit
constexpr int kWideChunksPerLane = 8;
constexpr int kWideUnitChunks = kWave * kWideChunksPerLane;   // 8 KiB: the last phase of a schedule as a word-granular tiled hop
constexpr int kRankAlignChunks = 8;                      // every rank's region of a staging buffer or of a class of exact-size T starts on a 128-byte line
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kExchangeRanks = 8;                        // ranks per thread of the elementwise size kernels

enum CopyMode { kPack = 0, kExchange = 1, kUnpack = 2, kFused = 3 };
// per-segment flags in the copy kernel's window: bits 0-3 = bytes of the first chunk that lie
// before the block (fused rounds), then:
constexpr int kFlagFill = 16;    // destination is a T slot: the tail lane fills up the 128-byte line
constexpr int kFlagSrcT = 32;    // source is a T slot: reading past the block's end is always safe

constexpr int kMaxClasses = 64 * 63 / 2;     // class_count(TUNA_MAX_PHASES)

// Device-side status block: the validation pass writes the head and the class sums, every phase its own entries of the
// other arrays; head and class sums are read back after validation, in one copy.
struct Status {
    unsigned int flags;            // bit 0: negative count, bit 1: recvcounts != transpose(sendcounts), (bit 3: receive regions not dense)
                                   // bit 2: negative displacement of a non-empty block, (bit 4: one into R of 4 GiB and more)
    unsigned int align_bits;       // OR of all counts and displacements, low 7 bits (they decide the granularity)
    int max_count;                 // M
    int tiny_done;                 // k_tiny_call: 1 = the whole call was done by that one kernel, 0 = it declined (nothing moved)
    unsigned long long total_bytes;    // sum of sendcounts
    unsigned long long total_chunks;   // sum of ceil(count / 16)
    unsigned long long send_extent;    // max over non-empty blocks of sdispls + count: bytes of sendbuf that hold blocks
    unsigned long long reserved1;
    unsigned long long short_blocks;   // blocks of fewer than kShortBlockBytes bytes, empty ones included
    unsigned long long windows;        // with blocks of more than kWindowMinBytes: most bytes that one receiver gets from
                                       // kValTile aligned neighbouring senders (high half) and one sender sends to as many
                                       // receivers (low half); blocks count up to kWindowBlock
    unsigned long long cls_chunks[kMaxClasses];   // exact-size T: chunks of every class (f, y), summed by the validation pass
    unsigned long long phase_bytes[64];   // payload bytes moved per phase
    unsigned long long phase_chunks[64];  // staged chunks per phase
    unsigned int phase_units[64][2];      // wave units per phase: [0] receive-side layout, [1] send-side layout
    unsigned int self_units;              // wave units of the ranks' own blocks when the copy engine moves them
    unsigned int reserved2;
    // What an immediate call's validation found, once more, for kernels of the call that run ahead of the host (no_places): unlike the
    // head it is left alone by plans and sizing queries, which do not wait for a call in flight.
    struct Verdict {
        unsigned int flags;
        int max_count;
        unsigned long long total_bytes;
    } verdict;
};

// The per-phase table of moving blocks (segments) on the device, one array per field: in message order or in that of the slot indices
// (PlanScalars.by_index).
struct SegDev {
    const int32_t* e;      // slot index j*Q + l
    const int32_t* z;      // digit value: which message, partner distance z*r^x
    const int32_t* src;    // source T slot or -1 (send buffer)
    const int32_t* dst;    // destination T slot or -1 (receive buffer)
    const int32_t* srcph;  // phase in which the block arrived in T, or -1 (send buffer)
    const int32_t* srcseg; // its position in that phase's table
    const int32_t* scls;   // exact-size T: class (arrival phase, this phase) the block is read from, or -1
    const int32_t* dcls;   // exact-size T: class (this phase, next move) the block is stored into, or -1
};

// Exact-size T.  A block that arrives in phase f and moves again in phase y waits in T from f to y: the
// blocks of one such class (f, y) lie together, rank after rank, each rank's part back to back in
// the order of the segments (padded to 16 bytes per block, to a 128-byte line per rank).  Where a class lies in T
// is decided on the host from the classes' sizes (the validation pass sums them) and lifetimes: classes
// whose lifetimes do not overlap share memory, so T holds what waits in it at one time, not what ever
// passed through it.  All offsets are in 16-byte chunks.
struct ExactT {
    const long long* cbase;  // [classes]: first chunk of each class in T (from the host)
    long long* tbase;        // [classes][P]: first chunk in T of rank p's part of a class
    int* csub;               // [classes][P]: chunks of rank p's part of a class
    int* tpos;               // [phases][P][P]: chunk offset, inside its rank's part of its class, of every block that the phase stored: by segment
                             // where phases find their blocks themselves (k_t_places), else by slot index
    int* tpre;               // [P][ld]: the same offsets for the phase being run, by segment
    int ld;
    int phase;               // index of the phase being run
    // the T-bound blocks of the phase being run, grouped by class: tord[tcls[3k+1] .. +tcls[3k+2]) are the
    // segment indices of class tcls[3k], ascending
    const int32_t* tord;
    const int32_t* tcls;
    int ncls;                // classes the phase being run stores into
};

// Distance pair of a slot index.
__device__ __forceinline__ void split_slot_index(int e, int Q, int N, int& j, int& l) {
    if (N == 1) { j = 0; l = e; }
    else { j = e / Q; l = e - j * Q; }
}

// One staging layout (send side or receive side) of the current phase.
struct LayoutDev {
    int* pre;                      // [P][ld]: exclusive prefix of chunk counts over the rank's segments; [nseg] = total
    int* tot;                      // [P]: chunks per rank
    long long* rank_base;          // [P+1]: first chunk of each rank in the staging buffer
    int* unit_base;                // [P+1]: first wave unit of each rank
    int4* units;                   // {rank, first segment, first chunk (rank-local), chunks in unit}
    int* n_units;                  // total units
    int ld;                        // row stride of pre (>= P + 1)
    int unit_chunks;               // chunks (or pieces) per wave unit: kUnitChunks, or kWideUnitChunks for the units of k_copy_tiled<4, 8>
};

// One-kernel phases: where every block a rank receives in the phase is read from and written to,
// resolved once per phase by k_resolve_hop, in the receive-side message order of the rank.  The copy
// kernel then needs one round of loads (prefix, source, destination, size) before its payload loads
// instead of three dependent ones (table, displacement or T position, payload).
struct HopDev {
    unsigned long long* src;       // [P][ld]: source address; kHopInT: an offset into T instead
    unsigned long long* dst;       // [P][ld]: destination address; kHopInT: an offset into T; kHopFill: a T slot whose last line is filled up
    int* size;                     // [P][ld]: bytes the destination takes: the exact count into R, whole chunks into T
    int ld;
};
constexpr unsigned long long kHopInT = 1ull << 62;
constexpr unsigned long long kHopFill = 1ull << 63;
constexpr int kHopLanes = 16;      // lanes of a copy wave that fetch their hop entries before the prefix is known

// ------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        int u = __shfl_up(v, d, kWave);
        if (lane >= d) v += u;
    }
    return v;
}

// op over the values of a wave (LANES = 64), or of each row of 16 lanes (16), in its last lane: by lane moves of the vector unit,
// no LDS.  The other lanes hold parts.
template <int CTRL, int ROWS, class T> __device__ __forceinline__ T lane_move(T v, T none) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two registers");
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xf, false);
    } else {
        const unsigned int lo = (unsigned int)__builtin_amdgcn_update_dpp((int)(unsigned int)none, (int)(unsigned int)v, CTRL, ROWS, 0xf, false);
        const unsigned int hi = (unsigned int)__builtin_amdgcn_update_dpp((int)(none >> 32), (int)(v >> 32), CTRL, ROWS, 0xf, false);
        return (T)hi << 32 | lo;
    }
}
template <int LANES, class T, class Op> __device__ __forceinline__ T last_lane(T v, T none, Op op) {
    v = op(v, lane_move<0x111, 0xf>(v, none));            // from 1, 2, 4, 8 lanes below in the row
    v = op(v, lane_move<0x112, 0xf>(v, none));
    v = op(v, lane_move<0x114, 0xf>(v, none));
    v = op(v, lane_move<0x118, 0xf>(v, none));
    if (LANES == kWave) {
        v = op(v, lane_move<0x142, 0xa>(v, none));        // the last lane of the row before to rows 1 and 3,
        v = op(v, lane_move<0x143, 0xc>(v, none));        // of the first half to the second
    }
    return v;
}
struct AddOp { template <class T> __device__ T operator()(T a, T b) const { return a + b; } };
struct MaxOp { template <class T> __device__ T operator()(T a, T b) const { return a > b ? a : b; } };
struct OrOp { template <class T> __device__ T operator()(T a, T b) const { return a | b; } };

// Sender of the message with digit value z that rank (n, g) receives in a phase: the rank at
// distance +z*r^x in the phase's dimension (Algorithm "TuNA": recvrank = p + z r^x).
__device__ __forceinline__ int partner_up(int n, int g, int Q, int N, int dim, int dist) {
    if (dim == 0) { int gg = g + dist; if (gg >= Q) gg -= Q; return n * Q + gg; }
    int nn = n + dist; if (nn >= N) nn -= N; return nn * Q + g;
}

// ------------------------------------------------------------------------------------------
// k_build_tables: the rank-independent tables of the digit phases, built on the device.  One
// thread per slot index e: its digit value z in this phase (Algorithm "TuNA", lines 8-11: the
// blocks whose x-th base-r digit equals z), its position in message order, the T slot it is read
// from / stored to by the map t = o - 1 - dx (r-1) - dz (Section "Estimating temporary buffer
// size"), or -1 for the send / receive buffer.
// ------------------------------------------------------------------------------------------
constexpr int kBuildPhases = 24;
struct BuildPhase {
    PhaseScalars ps;
    int32_t* mem;           // e, z, src, dst, srcph, srcseg, scls, dcls (SegDev), `stride` entries each
    int32_t* zt;
    int32_t* tord;          // ExactT
    int32_t* tcls;
    int stride;
};
struct BuildArgs {
    PlanScalars pl;
    BuildPhase ph[kBuildPhases];
    int first;              // index of ph[0] in the schedule
    int rows;               // phases here
    unsigned long long* mask;           // move_mask of every slot index
    unsigned long long* zero;           // n_zero words to clear on the way
    int n_zero;
};
// The lists of k_build_classes, by a workgroup of k_build_tables: where segments lie in the order of the slot indices the list of a
// class needs no finished table.  f: the phase, y: the one that forwards the class.
__device__ __forceinline__ void class_list(const BuildArgs& a, const BuildPhase& b, int f, int y) {
    __shared__ int s_n[2][4];
    __shared__ unsigned long long s_seen;
    const PlanScalars& pl = a.pl;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    int before = 0, own = 0;
    unsigned long long seen = 0;                         // classes before this one that have segments
    if (tid == 0) s_seen = 0;
    __syncthreads();
    for (int e = tid; e < pl.P; e += 256) {
        SegInfo s;
        int pos;
        if (!slot_entry(pl, b.ps, e, &s, &pos)) continue;
        if (s.nxt_phase > f && s.nxt_phase < y) { ++before; seen |= 1ull << (s.nxt_phase - f - 1); }
        own += s.nxt_phase == y;
    }
    before = last_lane<kWave>(before, 0, AddOp()); own = last_lane<kWave>(own, 0, AddOp());
    if (lane == kWave - 1) { s_n[0][wv] = before; s_n[1][wv] = own; }
    if (seen) atomicOr(&s_seen, seen);
    __syncthreads();
    before = s_n[0][0] + s_n[0][1] + s_n[0][2] + s_n[0][3];
    own = s_n[1][0] + s_n[1][1] + s_n[1][2] + s_n[1][3];
    seen = s_seen;
    if (own == 0) return;
    if (tid < 3) b.tcls[3 * __popcll(seen) + tid] = tid == 0 ? class_id(f, y, pl.nph) : tid == 1 ? before : own;
    int at = before;
    for (int e0 = 0; e0 < pl.P; e0 += 256) {
        SegInfo s;
        int pos = 0;
        const bool in = e0 + tid < pl.P && slot_entry(pl, b.ps, min(e0 + tid, pl.P - 1), &s, &pos) && s.nxt_phase == y;
        const unsigned long long mine = __ballot(in);
        __syncthreads();                                 // s_n of the step before is consumed
        if (lane == 0) s_n[0][wv] = __popcll(mine);
        __syncthreads();
        int here = at;
        for (int w = 0; w < 4; ++w) { here += w < wv ? s_n[0][w] : 0; at += s_n[0][w]; }
        if (in) b.tord[here + __popcll(mine & ((1ull << lane) - 1))] = pos;
    }
}
// grid (ceil(P / 256), rows); the first row also fills `mask`.  More rows, one per class of the schedule behind those, stand in for k_build_classes: a
// launch less for a call that may keep no schedule (with validation's results copied instead of folded by a kernel 87 -> 60 us, P = 200, r = 16).
__global__ void __launch_bounds__(256) k_build_tables(const BuildArgs a) {
    const PlanScalars& pl = a.pl;
    if ((int)blockIdx.y >= a.rows) {
        if (blockIdx.x) return;
        int f = 0, k = blockIdx.y - a.rows;
        while (k >= pl.nph - 1 - f) { k -= pl.nph - 1 - f; ++f; }
        class_list(a, a.ph[f], f, f + 1 + k);
        return;
    }
    const BuildPhase& b = a.ph[blockIdx.y];
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < a.n_zero; i += blockDim.x) a.zero[i] = 0;
    if (e >= pl.P) return;
    if (blockIdx.y == 0 && a.first == 0) a.mask[e] = move_mask(pl, e);
    SegInfo s;
    int pos = 0;
    if (slot_entry(pl, b.ps, e, &s, &pos)) {
        b.zt[e] = s.z;
        int32_t* m = b.mem + pos;
        const size_t ld = (size_t)b.stride;
        m[0] = s.e; m[ld] = s.z; m[2 * ld] = s.src_slot; m[3 * ld] = s.dst_slot; m[4 * ld] = s.src_phase; m[5 * ld] = s.src_seg;
        const int cur = b.ps.dim == 0 ? b.ps.x : pl.w_l + b.ps.x;
        m[6 * ld] = s.src_phase >= 0 ? class_id(s.src_phase, cur, pl.nph) : -1;
        m[7 * ld] = s.nxt_phase >= 0 ? class_id(cur, s.nxt_phase, pl.nph) : -1;
    } else {
        b.zt[e] = 0;
    }
}

// k_build_classes: the T-bound segments of every phase grouped by the class they are stored into, in message order (ExactT,
// tord and tcls).  Grid (classes a phase can have, phases), one wave per class: it counts the segments of the classes before
// its own and lists its own.  (On the host, and the lists copied to the device, it cost a call that may keep nothing 15 us.)
__global__ void __launch_bounds__(kWave) k_build_classes(const BuildArgs a) {
    const int f = a.first + blockIdx.y, first = class_id(f, f + 1, a.pl.nph), cid = first + blockIdx.x, lane = threadIdx.x;
    if (f + 1 + (int)blockIdx.x >= a.pl.nph) return;
    const BuildPhase& b = a.ph[blockIdx.y];
    const int32_t* dcls = b.mem + 7 * (size_t)b.stride;
    const int nseg = b.ps.nseg;
    int before = 0, own = 0;
    unsigned long long seen = 0;                         // classes before this one that have segments
    for (int s = lane; s < nseg; s += kWave) {
        const int c = dcls[s];
        if (c >= first && c < cid) { ++before; seen |= 1ull << (c - first); }
        own += c == cid;
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        before += __shfl_xor(before, d, kWave);
        own += __shfl_xor(own, d, kWave);
        seen |= __shfl_xor(seen, d, kWave);
    }
    if (own == 0) return;
    if (lane < 3) b.tcls[3 * __popcll(seen) + lane] = lane == 0 ? cid : lane == 1 ? before : own;
    int at = before;
    for (int s0 = 0; s0 < nseg; s0 += kWave) {
        const unsigned long long mine = __ballot(s0 + lane < nseg && dcls[min(s0 + lane, nseg - 1)] == cid);
        if (mine >> lane & 1) b.tord[at + __popcll(mine & ((1ull << lane) - 1))] = s0 + lane;
        at += __popcll(mine);
    }
}

// ------------------------------------------------------------------------------------------
// k_plain_copy: one aligned 16-byte chunk per thread, nothing else.  The practical HBM copy
// ceiling of the device and the known-size reference that hardware byte counters are scaled by.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_plain_copy(const v4u* __restrict__ src, v4u* __restrict__ dst, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// ------------------------------------------------------------------------------------------
// k_fill_uniform: the count and displacement matrices of a dense problem whose blocks all have
// `bytes` bytes (the calibration problems of the cost model); one thread per matrix entry.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_fill_uniform(int32_t* __restrict__ sendcounts, int64_t* __restrict__ sdispls,
                                                      int32_t* __restrict__ recvcounts, int64_t* __restrict__ rdispls,
                                                      int P, int bytes) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)P * P) return;
    sendcounts[i] = bytes; recvcounts[i] = bytes;
    sdispls[i] = (int64_t)i * bytes; rdispls[i] = (int64_t)i * bytes;
}

// ------------------------------------------------------------------------------------------
// k_validate: one pass over the P x P matrices in 64 x 64 tiles.  Finds M (Algorithm "TuNA",
// line 1: the maximum block size over all ranks, here one device reduction instead of an
// allreduce), the totals the workspace is sized from, checks counts >= 0 and
// recvcounts == transpose(sendcounts) through an LDS tile so both matrices are read row-wise
// (a wave reads 64 consecutive entries of one row).  With `mask` it also sums the chunks of every class of exact-size T.
// A non-empty block with a negative displacement is flagged too.  Workgroups of (64, 16) threads, two per compute unit,
// stride over the tiles and write one row of partial results each.  WHOLE: all four matrices; else sendcounts alone (a sizing query).
// Bound by its reads (24 bytes per pair) from P = 4096 on and by latency below, so a tile is one step: a thread has its four rows of all four
// matrices and of the masks in flight at once, and there is one barrier per tile (two buffers).  Against two steps with a barrier
// behind each, and from 23 x 23 tiles on eight of four waves (us of the kernel): P = 256, r = 4 15.4 / 10.6, P = 1024 20.1 / 14.1, P =
// 2048, r = 46 35.2 / 23.5, P = 4096 98 / 79 (5.1 TB/s), P = 8192 315 / 288; 4 us of the first for sums by lane moves instead of the LDS.
// The class sums are LDS atomics on one of `copies` copies per lane: neighbouring blocks mostly belong
// to one class, and on one copy a wave's additions queued up behind each other (P = 4096, r = 8: 159 -> 124 us).
// With a ticket (few workgroups) the partial rows, class sums included, lie in pinned host memory, each ends with the
// ticket, and the host waits for those and adds the rows up: no kernel to clear the sums, none to fold the rows, no copy of
// the result (see run_validate; P = 256, r = 4 138 -> 117 us per call with the above).
// The tile's columns and rows are summed too; the largest sums say whether long blocks lie side by side
// (clustered).  Not before a block of more than kWindowMinBytes was seen: problems of shorter ones only do not ask.
// ------------------------------------------------------------------------------------------
constexpr int kValTile = 64;
constexpr int kValRows = 16;                // waves of a workgroup
constexpr int kValPartial = 8;              // 64-bit words per workgroup in the partial-result array
constexpr int kValCopies = 32;
constexpr int kValFoldRows = 64, kValFoldClasses = 24;      // most workgroups and classes that the host folds
constexpr int kValRow = kValPartial + kValFoldClasses + 1;  // words of such a row, the ticket behind the others
// A wave's stores to pinned host memory, then the number that tells a waiting host that they are there: it need not wait
// for the kernel's end, its signal and the runtime's look at it.  By a whole wave, as its last stores: a call that is refused
// returns on the ticket, and the context's next one, on whatever stream, is ordered behind nothing else.
__device__ __forceinline__ void send_ticket(unsigned long long* word, unsigned long long ticket) {
    __threadfence_system();
    if ((threadIdx.x & (kWave - 1)) == 0) __hip_atomic_store(word, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
constexpr int kShortBlockBytes = 256;       // below this a block is mostly edges to the destination-tiled hop
constexpr int kWindowMinBytes = 64;
constexpr int kWindowBlock = 1 << 25;       // kValTile of them fit 32 bits
// the larger ones of two pairs of sums (Status.windows)
__host__ __device__ inline unsigned long long max_windows(unsigned long long a, unsigned long long b) {
    const unsigned long long low = 0xffffffffull, ar = a >> 32, br = b >> 32, as = a & low, bs = b & low;
    return (ar > br ? ar : br) << 32 | (as > bs ? as : bs);
}
template <bool WHOLE>
__global__ void __launch_bounds__(kValTile * kValRows, 8) k_validate(const int32_t* __restrict__ sendcounts,
                                                                     const int32_t* __restrict__ recvcounts,
                                                                     const int64_t* __restrict__ sdispls,
                                                                     const int64_t* __restrict__ rdispls,
                                                                     int P, unsigned long long* __restrict__ partial, int copies,
                                                                     int Q, int N, const unsigned long long* __restrict__ mask, int nph,
                                                                     Status* __restrict__ st, unsigned long long ticket, int clear_totals) {
    constexpr int kRows = kValTile / kValRows;            // rows of a tile per thread
    __shared__ int tile[2][kValTile][kValTile + 1];
    __shared__ unsigned int sums[2][2][kValTile];         // bytes per receiver, per sender of a tile
    __shared__ unsigned long long red[kValRows][8];
    __shared__ int long_seen[2];                          // (per buffer: a wave may be a tile ahead of one that still asks)
    extern __shared__ unsigned long long lcls[];          // class_count(nph) sums of this workgroup, `copies` of each (with `mask`)
    const int tx = threadIdx.x, ty = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int ncls = mask ? class_count(nph) : 0;
    for (int i = ty * kValTile + tx; i < ncls * copies; i += kValRows * kValTile) lcls[i] = 0;
    if (ty < 4) sums[ty >> 1][ty & 1][tx] = 0;
    if (tx < 2 && ty == 0) long_seen[tx] = 0;
    // the totals that k_phase_sums adds to, and the units that k_long_units counts (without a ticket k_validate_finish clears
    // them), not for a sizing query: the totals there belong to the context's last call.  First of all: right in front of the
    // ticket these stores cost a call 2 us
    if (ticket && clear_totals && blockIdx.x == 0 && ty == 0) st->phase_bytes[tx] = st->phase_chunks[tx] = st->phase_units[tx][0] = 0;
    __syncthreads();
    unsigned int window = 0;                              // largest sum of a receiver (first wave) or a sender (second wave)
    const int tpr = (P + kValTile - 1) / kValTile;       // tiles per row
    const int ntile = tpr * tpr;
    unsigned int flags = 0, abits = 0;
    int mx = 0, buf = 0;
    unsigned long long bytes = 0, chunks = 0, extent = 0;
    unsigned int shortb = 0;
    for (int t = blockIdx.x; t < ntile; t += gridDim.x, buf ^= 1) {        // a workgroup strides over tiles
        const int bi = (t / tpr) * kValTile, bj = (t % tpr) * kValTile;
        const int j = bj + tx, i2 = bi + tx;              // the receiver of a row's entry of sendcounts, the sender of one of recvcounts
        // every load of the tile, from clamped indices
        int cv[kRows], rv[kRows];
        long long dv[kRows], rd[kRows], rx = 0;
        unsigned int mv[kRows];                           // (no more than 32 phases: fewer than 2^30 ranks)
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const size_t at = (size_t)min(bi + ty + kValRows * u, P - 1) * P + min(j, P - 1);
            cv[u] = sendcounts[at];
            if (WHOLE) dv[u] = sdispls[at];
        }
        if (mask) {
            const int jn = min(j, P - 1) / Q, jg = min(j, P - 1) - jn * Q;    // the destination's node and local id
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int i = min(bi + ty + kValRows * u, P - 1), in = i / Q;
                int dn = in - jn; if (dn < 0) dn += N;
                int dg = i - in * Q - jg; if (dg < 0) dg += Q;
                mv[u] = (unsigned int)mask[dn * Q + dg];
            }
        }
        if (WHOLE) {
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const size_t at = (size_t)min(bj + ty + kValRows * u, P - 1) * P + min(i2, P - 1);
                rv[u] = recvcounts[at];
                rd[u] = rdispls[at];
            }
            // what the last lane of row u has behind it, in the lanes u, u + kRows, ...
            rx = rdispls[(size_t)min(bj + ty + kValRows * (tx & (kRows - 1)), P - 1) * P + min(bi + kValTile, P - 1)];
        }
        unsigned int to = 0;                              // bytes that this thread's senders have for receiver j
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int a = ty + kValRows * u;
            int c = 0;
            if (bi + a < P && j < P) {
                c = cv[u];
                if (c < 0) { flags |= 1u; c = 0; }
                abits |= (unsigned int)c;
                if (WHOLE) {
                    abits |= (unsigned int)dv[u] & 127u;
                    if (c > 0) {
                        if (dv[u] >= 0) extent = max(extent, (unsigned long long)dv[u] + (unsigned long long)c);
                        else flags |= 4u;
                    }
                }
                mx = max(mx, c);
                bytes += (unsigned long long)c;
                shortb += c < kShortBlockBytes ? 1u : 0u;
                const unsigned long long ch = (unsigned long long)((c + 15) >> 4);
                chunks += ch;
                if (mask && c > 0) {
                    // the block waits in T between every two consecutive phases in which it moves
                    unsigned int m = mv[u];
                    int f = __ffs((int)m) - 1;
                    m &= m - 1;
                    while (m) {
                        const int y = __ffs((int)m) - 1;
                        m &= m - 1;
                        atomicAdd(&lcls[class_id(f, y, nph) * copies + (tx & (copies - 1))], ch);
                        f = y;
                    }
                }
            }
            to += (unsigned int)min(c, kWindowBlock);
            tile[buf][a][tx] = c;
        }
        if (!WHOLE) continue;
        if (mx > kWindowMinBytes) long_seen[buf] = 1;     // (in every tile from the first long block on)
        __syncthreads();                                  // the only one per tile: the next one's entries go to the other buffer
        unsigned int from = 0;                            // bytes that sender i2 has for this thread's receivers
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int a = ty + kValRows * u;
            const int c = tile[buf][tx][a];
            from += (unsigned int)min(c, kWindowBlock);
            const bool in = bj + a < P && i2 < P;
            if (in) {
                if (rv[u] < 0) flags |= 1u;
                else if (rv[u] != c) flags |= 2u;         // recvcounts[jr][i] must equal sendcounts[i][jr]
                abits |= (unsigned int)rd[u] & 127u;
                const int high = (int)(rd[u] >> 32);
                if (rv[u] > 0 && high) flags |= high < 0 ? 4u : 16u;
            }
            // dense receive regions: every block starts where its predecessor in source order ends (flag 8 when not; the
            // destination-tiled hop needs it).  A wave holds 64 neighbours of one row.
            long long dn = __shfl_down(rd[u], 1, kWave);
            const long long behind = __shfl(rx, u, kWave);
            if (tx == kValTile - 1) dn = behind;
            if (in && i2 + 1 < P && dn != rd[u] + (long long)max(rv[u], 0)) flags |= 8u;
        }
        if (long_seen[buf]) {                              // windows of neighbouring blocks
            atomicAdd(&sums[buf][0][tx], to);
            atomicAdd(&sums[buf][1][tx], from);
        }
        // the sums of the tile before, which every wave added to in front of the barrier above
        if (ty < 2) { window = max(window, sums[buf ^ 1][ty][tx]); sums[buf ^ 1][ty][tx] = 0; }
    }
    __syncthreads();
    if (ty < 2) window = max(window, sums[buf ^ 1][ty][tx]);
    // wave reduction, workgroup reduction through LDS, then one row of partial results per workgroup
    unsigned long long fa = last_lane<kWave>(flags << 8 | (abits & 127u), 0u, OrOp());
    fa = fa >> 8 << 32 | (fa & 127u);
    unsigned long long m = last_lane<kWave>((unsigned int)mx, 0u, MaxOp()), sb = last_lane<kWave>(shortb, 0u, AddOp());
    unsigned long long by = last_lane<kWave>(bytes, 0ull, AddOp()), ch = last_lane<kWave>(chunks, 0ull, AddOp());
    unsigned long long ex = last_lane<kWave>(extent, 0ull, MaxOp());
    window = last_lane<kWave>(window, 0u, MaxOp());
    if (tx == kWave - 1) {                               // one wave per value of ty
        unsigned long long* r = red[ty];
        r[0] = fa; r[1] = m; r[2] = by; r[3] = ch; r[4] = ex; r[6] = sb; r[7] = window;
    }
    __syncthreads();
    unsigned long long* o = partial + (size_t)blockIdx.x * (ticket ? kValRow : kValPartial);
    if (ty == 0) {                                        // one lane per wave's row
        static_assert(kValRows == 16, "a row of lanes");
        const unsigned long long* r = red[tx & (kValRows - 1)];
        const unsigned long long wi = red[0][7] << 32 | red[1][7];
        fa = last_lane<kValRows>(r[0], 0ull, OrOp()); m = last_lane<kValRows>(r[1], 0ull, MaxOp());
        by = last_lane<kValRows>(r[2], 0ull, AddOp()); ch = last_lane<kValRows>(r[3], 0ull, AddOp());
        ex = last_lane<kValRows>(r[4], 0ull, MaxOp()); sb = last_lane<kValRows>(r[6], 0ull, AddOp());
        // one row of partial results per workgroup, folded by k_validate_finish or the host: thousands of atomics
        // on the same few addresses would take longer than reading the matrices
        if (tx == kValRows - 1) { o[0] = fa; o[1] = m; o[2] = by; o[3] = ch; o[4] = ex; o[5] = 0; o[6] = sb; o[7] = wi; }
    }
    // the class sums: in the row, or one atomic per class and workgroup that holds any of it (cls_chunks starts at zero)
    for (int i = ty * kValTile + tx; i < ncls; i += kValRows * kValTile) {
        unsigned long long v = 0;
#pragma unroll 8
        for (int k = 0; k < copies; ++k) v += lcls[i * copies + ((i + k) & (copies - 1))];
        if (ticket) o[kValPartial + i] = v;                   // (first wave: kValFoldClasses < kWave)
        else if (v) atomicAdd(&st->cls_chunks[i], v);
    }
    if (ticket && ty == 0) send_ticket(o + kValRow - 1, ticket);
}

// k_zero64: n 64-bit words to zero (the class sums before a validation pass).
__global__ void __launch_bounds__(256) k_zero64(unsigned long long* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// k_validate_finish: folds the workgroups' partial results into the status block (one workgroup).  With `mirror` it also
// writes the block's head and the ncls class sums there, pinned host memory, and sends the ticket, and clears the sums for
// the next call: in place of a copy command and a launch of k_zero64.
__global__ void __launch_bounds__(256) k_validate_finish(const unsigned long long* __restrict__ partial, int n,
                                                         Status* __restrict__ st, int clear_totals, Status* __restrict__ mirror,
                                                         int ncls, unsigned long long* __restrict__ word, unsigned long long ticket) {
    __shared__ unsigned long long red[4][8];
    // the totals that k_phase_sums adds to, and the units that k_long_units counts; the other paths write them whole
    if (clear_totals && threadIdx.x < 64) st->phase_bytes[threadIdx.x] = st->phase_chunks[threadIdx.x] = st->phase_units[threadIdx.x][0] = 0;
    unsigned long long fa = 0, m = 0, by = 0, ch = 0, ex = 0, sb = 0, wi = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long* o = partial + (size_t)i * kValPartial;
        fa |= o[0]; m = max(m, o[1]); by += o[2]; ch += o[3]; ex = max(ex, o[4]); sb += o[6];
        wi = max_windows(wi, o[7]);
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        fa |= __shfl_xor(fa, d, kWave);
        m = max(m, (unsigned long long)__shfl_xor(m, d, kWave));
        by += __shfl_xor(by, d, kWave);
        ch += __shfl_xor(ch, d, kWave);
        ex = max(ex, (unsigned long long)__shfl_xor(ex, d, kWave));
        sb += __shfl_xor(sb, d, kWave);
        wi = max_windows(wi, __shfl_xor(wi, d, kWave));
    }
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    if (lane == 0) { red[wv][0] = fa; red[wv][1] = m; red[wv][2] = by; red[wv][3] = ch; red[wv][4] = ex; red[wv][6] = sb; red[wv][7] = wi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        fa = m = by = ch = ex = sb = wi = 0;
        for (int w = 0; w < 4; ++w) {
            fa |= red[w][0]; m = max(m, red[w][1]); by += red[w][2]; ch += red[w][3]; ex = max(ex, red[w][4]);
            sb += red[w][6]; wi = max_windows(wi, red[w][7]);
        }
        if (clear_totals) st->verdict = Status::Verdict{(unsigned int)(fa >> 32), (int)m, by};
        st->flags = (unsigned int)(fa >> 32);
        st->align_bits = (unsigned int)(fa & 127u);
        st->max_count = (int)m;
        st->total_bytes = by;
        st->total_chunks = ch;
        st->send_extent = ex;
        st->short_blocks = sb;
        st->windows = wi;
        if (mirror) {
            mirror->flags = (unsigned int)(fa >> 32);
            mirror->align_bits = (unsigned int)(fa & 127u);
            mirror->max_count = (int)m;
            mirror->total_bytes = by;
            mirror->total_chunks = ch;
            mirror->send_extent = ex;
            mirror->short_blocks = sb;
            mirror->windows = wi;
        }
    }
    if (mirror && threadIdx.x < kWave) {
        for (int i = threadIdx.x; i < ncls; i += kWave) { mirror->cls_chunks[i] = st->cls_chunks[i]; st->cls_chunks[i] = 0; }
        send_ticket(word, ticket);
    }
}

// ------------------------------------------------------------------------------------------
// k_rotate_init: the index-only initial rotation (Algorithm "TuNA", lines 4-5; Algorithm
// "Coalesced TuNA_l^g", line 5).  No payload moves: cur[p][j*Q + l] becomes the size of the
// block rank p = (n, g) holds at distance (j, l), i.e. its block for rank ((n-j)%N, (g-l)%Q).
// With `up` the row is rotated the other way, cur[p][j*Q + l] = counts[p][((n+j)%N, (g+l)%Q)]: applied to
// recvcounts that is the size of the block rank p receives from the rank at distance (j, l) -- for a schedule
// of one phase, where every block arrives in its first and only hop, exactly what the metadata exchange of
// that phase leaves in the receiver's size array (Algorithm "TuNA", line 14), without the exchange.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_rotate_init(const int32_t* __restrict__ sendcounts,
                                                     int32_t* __restrict__ cur, int P, int Q, int N, int up) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;      // grid (ceil(P / 256), ceil(P / kExchangeRanks))
    if (e >= P) return;
    const int j = e / Q, l = e - j * Q;
    const int p0 = blockIdx.y * kExchangeRanks;
    int v[kExchangeRanks];
#pragma unroll
    for (int k = 0; k < kExchangeRanks; ++k) {
        const int p = p0 + k;
        v[k] = 0;
        if (p < P) {
            const int n = p / Q, g = p - n * Q;
            int dn = up ? n + j : n - j; if (dn < 0) dn += N; if (dn >= N) dn -= N;
            int dg = up ? g + l : g - l; if (dg < 0) dg += Q; if (dg >= Q) dg -= Q;
            v[k] = sendcounts[(size_t)p * P + dn * Q + dg];
        }
    }
#pragma unroll
    for (int k = 0; k < kExchangeRanks; ++k)
        if (p0 + k < P) cur[(size_t)(p0 + k) * P + e] = v[k];
}

// ------------------------------------------------------------------------------------------
// k_self_copy: the block a rank keeps for itself goes straight from S to R (Section "Estimating
// temporary buffer size": one block is destined for the rank itself).  One workgroup per rank; own_block is what other launches
// that take the own blocks along run for a rank.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void own_block(const unsigned char* __restrict__ S, const int32_t* __restrict__ sendcounts,
                                          const int64_t* __restrict__ sdispls, unsigned char* __restrict__ R,
                                          const int64_t* __restrict__ rdispls, int P, int p) {
    const size_t d = (size_t)p * P + p;
    const int n = sendcounts[d];
    const unsigned char* src = S + sdispls[d];
    unsigned char* dst = R + rdispls[d];
    const int nchunk = n >> 4;
    for (int c = threadIdx.x; c < nchunk; c += 256) {
        uint4 v;
        __builtin_memcpy(&v, src + ((size_t)c << 4), 16);
        __builtin_memcpy(dst + ((size_t)c << 4), &v, 16);
    }
    const int tail = n & 15;
    if ((int)threadIdx.x < tail) dst[(nchunk << 4) + threadIdx.x] = src[(nchunk << 4) + threadIdx.x];
}
__global__ void __launch_bounds__(256) k_self_copy(const unsigned char* __restrict__ S,
                                                   const int32_t* __restrict__ sendcounts,
                                                   const int64_t* __restrict__ sdispls,
                                                   unsigned char* __restrict__ R,
                                                   const int64_t* __restrict__ rdispls, int P) {
    own_block(S, sendcounts, sdispls, R, rdispls, P, blockIdx.x);
}

// ------------------------------------------------------------------------------------------
// k_self_layout: the ranks' own blocks laid out as one more one-kernel phase of a single block per
// rank, source S at sdispls[p][p], destination R at rdispls[p][p], so that the byte-balanced copy
// engine moves them (large own blocks: one workgroup per rank would leave most of the device idle).
// One thread per rank; k_layout_base and k_layout_units then cut the wave units as for any phase.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_self_layout(const unsigned char* __restrict__ S,
                                                     const int32_t* __restrict__ sendcounts,
                                                     const int64_t* __restrict__ sdispls, unsigned char* __restrict__ R,
                                                     const int64_t* __restrict__ rdispls, int P, LayoutDev L, HopDev h) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const size_t d = (size_t)p * P + p;
    const int sz = sendcounts[d];
    const unsigned long long src = (unsigned long long)(S + sdispls[d]);
    const unsigned long long dst = (unsigned long long)(R + rdispls[d]);
    // chunks are cut at the destination's 16-byte boundaries, as in every one-kernel phase
    const int chunks = sz > 0 ? (int)(((unsigned int)(dst & 15ull) + (unsigned int)sz + 15u) >> 4) : 0;
    int* pre = L.pre + (size_t)p * L.ld;
    pre[0] = 0; pre[1] = chunks;
    L.tot[p] = chunks;
    const size_t o = (size_t)p * h.ld;
    h.src[o] = sz > 0 ? src : 0ull; h.dst[o] = sz > 0 ? dst : 0ull; h.size[o] = sz > 0 ? sz : 0;
}

// ------------------------------------------------------------------------------------------
// k_size_exchange: the metadata exchange of one digit phase (Section "Two-phase communication";
// Algorithm "TuNA", line 14): the size of every moving block travels from the sender's size array
// to the receiver's, nxt[q][e] = cur[q + z r^x][e] with z the digit of e; sizes of blocks that stay
// are carried over.  One thread per (rank, slot index): both rows are read and written along e.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_size_exchange(const int32_t* __restrict__ cur, int32_t* __restrict__ nxt,
                                                       const int32_t* __restrict__ zt, int P, int Q, int N, int dim,
                                                       int rx) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= P) return;
    const int dist = zt[e] * rx;                      // 0: the block stays
    const int q0 = blockIdx.y * kExchangeRanks;
    int v[kExchangeRanks];
#pragma unroll
    for (int k = 0; k < kExchangeRanks; ++k) {        // all loads of a thread are in flight together
        const int q = q0 + k;
        v[k] = 0;
        if (q < P) {
            int src = q;
            if (dist) {
                const int qn = q / Q;
                src = partner_up(qn, q - qn * Q, Q, N, dim, dist);
            }
            v[k] = cur[(size_t)src * P + e];
        }
    }
#pragma unroll
    for (int k = 0; k < kExchangeRanks; ++k)
        if (q0 + k < P) nxt[(size_t)(q0 + k) * P + e] = v[k];
}

// ------------------------------------------------------------------------------------------
// k_phase_layout: the size/displacement scans of one digit phase, one workgroup per rank, from the
// sizes the rank holds before the phase (`cur`) and after it (`nxt`, see k_size_exchange):
//  size/displacement scans (the contiguous send buffer of Algorithm "TuNA", line 15, needs each
//  block's offset inside its message): per rank, the moving blocks' sizes in message order are
//  converted to 16-byte chunks and exclusive-scanned (wave shuffles + LDS across the 4 waves,
//  a running carry across batches of 1024 segments) -- once over the sizes the rank receives
//  (receive-side layout) and once over the sizes it sends (send-side layout);
// With `head_displs` (one-kernel phases) the chunks of a block bound for R are cut at the 16-byte
// boundaries of its destination address: a block that starts `a` bytes into a 16-byte line takes
// ceil((a + size) / 16) chunks; head_base is the low 4 bits of the receive buffer address.
// ------------------------------------------------------------------------------------------
struct PhaseLayoutArgs {
    const int32_t* cur;             // [P][P] sizes before the phase
    int32_t* nxt;                   // [P][P] sizes after it
    int inline_exchange;            // 1: this kernel also does the size exchange (few ranks: one launch less)
    const int32_t* zt;              // [P] digit value of slot e in this phase (0: stays)
    SegDev seg;
    int nseg;
    int P, Q, N, dim, rx;
    LayoutDev Ls, Lr;
    int want_send;                  // 0: only the receive-side layout (one-kernel phases)
    int want_tbound;                // 1: also lay out the blocks this phase stores into exact-size T (see ExactT)
    ExactT x;
    unsigned long long* rank_bytes; // [P]: payload bytes every rank moves in this phase
    unsigned long long* phase_bytes;
    unsigned long long* phase_chunks;
    unsigned int* phase_units;      // [2]: wave units of the receive-side and of the send-side layout
    const int64_t* head_displs;
    unsigned int head_base;
};

// Item k of a thread in a batch of kScanThreads * kScanItems segments: every wave owns
// kScanItems * 64 consecutive segments and lane i takes the ones at i, i + 64, ...: one load
// instruction of a wave reads 64 consecutive table entries.
__device__ __forceinline__ int scan_item_index(int k) {
    const int tid = threadIdx.x;
    return (tid / kWave) * (kWave * kScanItems) + k * kWave + (tid & (kWave - 1));
}

// exclusive scan of the batch in that order; run[k] = start of item k, `carry` grows by the batch total
__device__ __forceinline__ void block_scan_batch(const int (&c)[kScanItems], int (&run)[kScanItems], int& carry,
                                                 int* wsum) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    int wtotal = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int incl = wave_incl_scan(c[k]);
        run[k] = wtotal + incl - c[k];
        wtotal += __shfl(incl, kWave - 1, kWave);
    }
    __syncthreads();                                  // wsum of the previous batch is consumed
    if (lane == 0) wsum[wv] = wtotal;
    __syncthreads();
    int woff = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k) {
        const int v = wsum[k];
        if (k < wv) woff += v;
        total += v;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) run[k] += carry + woff;
    carry += total;
}

// exclusive scan over the P per-rank totals of one layout by one workgroup of kScanThreads: every
// thread sums a contiguous range of ranks, the thread sums are scanned across the workgroup, then
// every thread writes the bases of its range
__device__ __forceinline__ void scan_rank_bases(int P, const LayoutDev& L, unsigned long long* phase_chunks,
                                                long long* wc, int* wt,
                                                const unsigned long long* rank_bytes = nullptr,
                                                unsigned long long* phase_bytes = nullptr,
                                                unsigned int* units_out = nullptr) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int per = (P + kScanThreads - 1) / kScanThreads;
    const int p0 = min(P, tid * per), p1 = min(P, p0 + per);
    const int ralign = kRankAlignChunks;
    long long sc = 0;
    int st = 0;
    // a rank's region is rounded up to whole 128-byte lines: units, which are cut every 4 KiB from
    // the region's start, then begin and end on line boundaries and their streaming stores are never
    // split into partial-line writes
    for (int p = p0; p < p1; ++p) {
        const int c = L.tot[p];
        sc += (c + ralign - 1) / ralign * ralign;
        st += (c + L.unit_chunks - 1) / L.unit_chunks;
    }
    long long ic = sc;
    int it = st;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        long long uc = __shfl_up(ic, d, kWave);
        int ut = __shfl_up(it, d, kWave);
        if (lane >= d) { ic += uc; it += ut; }
    }
    if (lane == kWave - 1) { wc[wv] = ic; wt[wv] = it; }
    __syncthreads();
    long long oc = 0, totc = 0;
    int ot = 0, tott = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k) {
        if (k < wv) { oc += wc[k]; ot += wt[k]; }
        totc += wc[k]; tott += wt[k];
    }
    long long run_c = oc + ic - sc;
    int run_t = ot + it - st;
    for (int p = p0; p < p1; ++p) {
        const int c = L.tot[p];
        L.rank_base[p] = run_c;
        if (L.unit_base) L.unit_base[p] = run_t;
        run_c += (c + ralign - 1) / ralign * ralign;
        run_t += (c + L.unit_chunks - 1) / L.unit_chunks;
    }
    if (tid == 0) {
        L.rank_base[P] = totc;
        if (L.unit_base) { L.unit_base[P] = tott; *L.n_units = tott; }
        if (units_out) *units_out = (unsigned int)tott;
        if (phase_chunks) *phase_chunks = (unsigned long long)totc;
    }
    if (phase_bytes) {                                // payload bytes of the phase = sum of the ranks' sums
        unsigned long long b = 0;
        for (int p = p0; p < p1; ++p) b += rank_bytes[p];
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) b += __shfl_xor(b, d, kWave);
        __syncthreads();                              // wc is reused
        if (lane == 0) wc[wv] = (long long)b;
        __syncthreads();
        if (tid == 0) {
            unsigned long long t = 0;
#pragma unroll
            for (int k = 0; k < kScanThreads / kWave; ++k) t += (unsigned long long)wc[k];
            *phase_bytes = t;
        }
    }
}

__global__ void __launch_bounds__(kScanThreads) k_phase_layout(const PhaseLayoutArgs a) {
    __shared__ int wsum[kScanThreads / kWave];
    __shared__ unsigned long long wbytes[kScanThreads / kWave];
    const int P = a.P;
    const int p = blockIdx.x;
    const int pn = p / a.Q, pg = p - pn * a.Q;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int32_t* crow = a.cur + (size_t)p * P;
    int32_t* nrow = a.nxt + (size_t)p * P;
    if (a.inline_exchange) {
        // the metadata exchange (see k_size_exchange), here by the receiving rank's own workgroup:
        // blocks that do not move keep their size, the others arrive with the scan's gather below
        for (int e = tid; e < P; e += kScanThreads)
            if (a.zt[e] == 0) nrow[e] = crow[e];
    }
    int* pre_r = a.Lr.pre + (size_t)p * a.Lr.ld;
    int* pre_s = a.Ls.pre + (size_t)p * a.Ls.ld;
    int carry_r = 0, carry_s = 0;
    unsigned long long bytes = 0;
    for (int base = 0; base < a.nseg; base += kScanThreads * kScanItems) {
        int cr[kScanItems], cs[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int s = base + scan_item_index(k);
            int szr = 0, szs = 0, head = 0;
            if (s < a.nseg) {
                const int e = a.seg.e[s];
                if (a.inline_exchange) {
                    const int ps = partner_up(pn, pg, a.Q, a.N, a.dim, a.seg.z[s] * a.rx);
                    szr = a.cur[(size_t)ps * P + e];
                    nrow[e] = szr;
                } else {
                    szr = nrow[e];
                }
                if (a.want_send) szs = crow[e];
                if (a.head_displs && szr > 0 && a.seg.dst[s] < 0) {
                    int j, l;
                    split_slot_index(e, a.Q, a.N, j, l);
                    int sn = pn + j; if (sn >= a.N) sn -= a.N;
                    int sg = pg + l; if (sg >= a.Q) sg -= a.Q;
                    head = (int)(((unsigned int)a.head_displs[(size_t)p * P + sn * a.Q + sg] + a.head_base) & 15u);
                }
            }
            bytes += (unsigned long long)(a.want_send ? szs : szr);
            cr[k] = (head + szr + 15) >> 4;
            cs[k] = (szs + 15) >> 4;
        }
        int run[kScanItems];
        block_scan_batch(cr, run, carry_r, wsum);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int s = base + scan_item_index(k);
            if (s < a.nseg) pre_r[s] = run[k];
        }
        if (a.want_send) {
            block_scan_batch(cs, run, carry_s, wsum);
#pragma unroll
            for (int k = 0; k < kScanItems; ++k) {
                const int s = base + scan_item_index(k);
                if (s < a.nseg) pre_s[s] = run[k];
            }
        }
    }
    if (a.want_tbound) {
        // Exact-size T: the blocks this phase stores, class by class (a class = the blocks that move next in
        // the same later phase); within a class in message order.  Every block's chunk offset inside this
        // rank's part of its class goes to tpre (by segment, for this phase's own stores) and to tpos (by slot
        // index, for the phase that forwards the block); the part's size goes to csub.
        __syncthreads();                                  // the sizes this workgroup exchanged itself are in nrow
        int* pre_t = a.x.tpre + (size_t)p * a.x.ld;
        int* pos_t = a.x.tpos + ((size_t)a.x.phase * P + p) * P;
        for (int cl = 0; cl < a.x.ncls; ++cl) {
            const int cid = a.x.tcls[3 * cl], c0 = a.x.tcls[3 * cl + 1], cn = a.x.tcls[3 * cl + 2];
            int carry_t = 0;
            for (int base = 0; base < cn; base += kScanThreads * kScanItems) {
                int ct[kScanItems], sg[kScanItems], se[kScanItems];
#pragma unroll
                for (int k = 0; k < kScanItems; ++k) {
                    const int i = base + scan_item_index(k);
                    ct[k] = 0; sg[k] = -1; se[k] = 0;
                    if (i < cn) {
                        sg[k] = a.x.tord[c0 + i];
                        se[k] = a.seg.e[sg[k]];
                        ct[k] = (nrow[se[k]] + 15) >> 4;
                    }
                }
                int run[kScanItems];
                block_scan_batch(ct, run, carry_t, wsum);
#pragma unroll
                for (int k = 0; k < kScanItems; ++k)
                    if (sg[k] >= 0) { pre_t[sg[k]] = run[k]; pos_t[se[k]] = run[k]; }
            }
            if (tid == 0) a.x.csub[(size_t)cid * P + p] = carry_t;
        }
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) bytes += __shfl_xor(bytes, d, kWave);
    // one sum per rank, added up by k_layout_base: thousands of atomics on one address would take
    // longer than the scans
    __syncthreads();
    if (lane == 0) wbytes[tid / kWave] = bytes;
    __syncthreads();
    if (tid == 0) {
        unsigned long long t = 0;
#pragma unroll
        for (int k = 0; k < kScanThreads / kWave; ++k) t += wbytes[k];
        a.rank_bytes[p] = t;
    }
    if (tid == 0) {
        pre_r[a.nseg] = carry_r; a.Lr.tot[p] = carry_r;
        if (a.want_send) { pre_s[a.nseg] = carry_s; a.Ls.tot[p] = carry_s; }
    }
}

// A class of exact-size T: rank p's part starts at the class's first chunk plus the parts of the ranks before it, each
// rounded up to a 128-byte line.  One workgroup of kScanThreads.
__device__ __forceinline__ void class_base(const ExactT& x, int cid, long long first, int P, long long* wc) {
    const int* sub = x.csub + (size_t)cid * P;
    long long* base = x.tbase + (size_t)cid * P;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int per = (P + kScanThreads - 1) / kScanThreads;
    const int p0 = min(P, tid * per), p1 = min(P, p0 + per);
    long long sc = 0;
    for (int p = p0; p < p1; ++p) sc += (sub[p] + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks;
    long long ic = sc;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const long long uc = __shfl_up(ic, d, kWave);
        if (lane >= d) ic += uc;
    }
    if (lane == kWave - 1) wc[wv] = ic;
    __syncthreads();
    long long oc = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k)
        if (k < wv) oc += wc[k];
    long long run = first + oc + ic - sc;
    for (int p = p0; p < p1; ++p) {
        base[p] = run;
        run += (sub[p] + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks;
    }
}

// ------------------------------------------------------------------------------------------
// k_layout_base: exclusive scan over the P per-rank totals of a layout -> each rank's first chunk
// in its staging buffer and its first wave unit.  One workgroup per layout the host lists (receive
// side, send side), then one per class of exact-size T that the phase stores into: there the scan
// runs over the ranks' parts of the class and gives every rank's first chunk in T.  A separate
// launch rather than a "last workgroup" step inside k_phase_layout: the kernel boundary is the one
// device-wide release the totals need.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kScanThreads) k_layout_base(int P, LayoutDev L0, LayoutDev L1, int n_layouts,
                                                              unsigned long long* __restrict__ phase_chunks,
                                                              int chunks_from, ExactT x,
                                                              const unsigned long long* __restrict__ rank_bytes,
                                                              unsigned long long* __restrict__ phase_bytes,
                                                              unsigned int* __restrict__ phase_units) {
    __shared__ long long wc[kScanThreads / kWave];
    __shared__ int wt[kScanThreads / kWave];
    const int which = blockIdx.x;
    if (which < n_layouts) {
        scan_rank_bases(P, which == 0 ? L0 : L1, which == chunks_from ? phase_chunks : nullptr, wc, wt,
                        rank_bytes, which == chunks_from ? phase_bytes : nullptr,
                        phase_units + which);             // layout 0 is the receive side, 1 the send side
        return;
    }
    const int cid = x.tcls[3 * (which - n_layouts)];
    class_base(x, cid, x.cbase[cid], P, wc);
}

// ------------------------------------------------------------------------------------------
// k_layout_units: cut every rank's staged chunks into wave units of L.unit_chunks and record, per
// unit, the rank and the first segment that overlaps it (binary search in the rank's prefix
// row, which is staged in LDS when it fits: lds_ints = nseg + 1, else 0 and the search reads
// global memory).  grid (P, layouts): one workgroup per rank and layout (y = 0 receive side,
// 1 send side).
// ------------------------------------------------------------------------------------------
constexpr int kUnitsLdsMaxInts = 12288;     // 48 KiB of the workgroup's LDS
__global__ void __launch_bounds__(256) k_layout_units(int nseg, LayoutDev Lr, LayoutDev Ls, int lds_ints) {
    extern __shared__ int s_row[];
    const LayoutDev& L = blockIdx.y == 0 ? Lr : Ls;
    const int p = blockIdx.x;
    const int tot = L.tot[p];
    const int uc = L.unit_chunks;
    const int nu = (tot + uc - 1) / uc;
    if (nu == 0) return;                       // uniform over the workgroup
    const int* pre = L.pre + (size_t)p * L.ld;
    if (lds_ints) {
        for (int i = threadIdx.x; i < lds_ints; i += blockDim.x) s_row[i] = pre[i];
        __syncthreads();
        pre = s_row;
    }
    const int ub = L.unit_base[p];
    for (int t = threadIdx.x; t < nu; t += blockDim.x) {
        const int c0 = t * uc;
        int lo = 0, hi = nseg;                 // largest s in [0, nseg) with pre[s] <= c0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= c0) lo = mid; else hi = mid;
        }
        L.units[ub + t] = make_int4(p, lo, c0, min(uc, tot - c0));
    }
}

// ------------------------------------------------------------------------------------------
// The copy engine.  pack / exchange / unpack are the same byte-balanced variable-length copy
// with a different "other side":
//   pack     staging(send)  <- S at sdispls, or T slot      (Algorithm "TuNA", line 15, sender side)
//   exchange staging(recv)  <- staging(send) of the partner (the point-to-point transfer itself)
//   unpack   staging(recv)  -> R at rdispls, or T slot      (Algorithm "TuNA", lines 16-20)
//   fused    S / T of the sender -> R / other copy of T at the receiver, tiled over the receiver's
//            layout (all three in one hop, no staging)
// Work unit = one wavefront x 256 consecutive 16-byte chunks (4 KiB) of one rank's staging
// region.  The wave is self-contained -- no workgroup barrier anywhere: lane i loads the chunk
// prefix and the table entry of segment s0 + i, the lanes whose segment overlaps the unit
// resolve its other-side address (T slot arithmetic, a position in exact-size T, or one
// displacement load), the 64 entries
// go to the wave's private LDS window, and every lane finds the segment of each of its 4 chunks
// by a binary search over that window.  Lanes of a wave touch consecutive chunks on the staging
// side (aligned, non-temporal dwordx4) and consecutive bytes of a block on the other side.
// One-shot grid: 4 units per workgroup; the host launches an upper bound of units and waves
// beyond the device-side unit count exit at once.  A launch for a batch of rounds may instead use
// one grid row per rank, as wide as the units a rank can have in the batch.
// ------------------------------------------------------------------------------------------
struct CopyArgs {
    // tiled (staging) side
    v4u* stage;                         // staging buffer being tiled (unused when fused)
    LayoutDev L;                        // its layout
    SegDev seg;
    int nseg;
    // other side: caller buffer + T (pack, unpack, fused source)
    const int32_t* counts;              // recvcounts: exact sizes of the blocks that are final (unpack, fused)
    unsigned char* user;                // S (pack) or R (unpack)
    const int64_t* displs;              // sdispls (pack), rdispls (unpack); unused when fused (k_resolve_hop read them)
    unsigned long long user_limit;      // pack: address one past the last byte of S that holds a block
    unsigned char* T;                   // temporary buffer: slot s of rank p at ((p*slots + s) * slot_bytes)
    long long slots;
    long long slot_bytes;
    // other side: send staging (exchange)
    const v4u* stage_src;
    LayoutDev Ls;
    // fused: every block's source and destination, resolved by k_resolve_hop
    HopDev hop;
    // exact-size T (DENSE kernels): the blocks that wait in T lie back to back, class by class, instead of in slots
    ExactT x;
    // a launch may cover only the rounds of one batch: the segments [seg_lo, seg_hi) of every rank
    int seg_lo, seg_hi;
    // 1: such a launch has a grid of (units a rank can have in the batch / 4, P) -- row y covers the units
    // of rank y that overlap the batch; 0: one-dimensional grid over all units
    int batch_rows;
    int P, Q, N, dim, rx;
};

template <int GRAN>
__device__ __forceinline__ v4u load_block_chunk(const unsigned char* src, int nb) {
    v4u v = {0u, 0u, 0u, 0u};
    if (GRAN >= 16 || nb >= 16) {
        __builtin_memcpy(&v, src, 16);
    } else if (GRAN == 4) {
        const uint32_t* s4 = reinterpret_cast<const uint32_t*>(src);
        if (nb > 0) v.x = s4[0];
        if (nb > 4) v.y = s4[1];
        if (nb > 8) v.z = s4[2];
    } else {
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 15; ++b)
            if (b < nb) w[b >> 2] |= (uint32_t)src[b] << (8 * (b & 3));
        v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
    }
    return v;
}

template <int GRAN>
__device__ __forceinline__ void store_block_chunk(unsigned char* dst, v4u v, int nb) {
    if (GRAN >= 16 || nb >= 16) {
        __builtin_memcpy(dst, &v, 16);
    } else if (GRAN == 4) {
        uint32_t* d4 = reinterpret_cast<uint32_t*>(dst);
        if (nb > 0) d4[0] = v.x;
        if (nb > 4) d4[1] = v.y;
        if (nb > 8) d4[2] = v.z;
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int b = 0; b < 15; ++b)
            if (b < nb) dst[b] = (unsigned char)(w[b >> 2] >> (8 * (b & 3)));
    }
}

// Address of the block a table entry describes, on the caller-buffer / T side of rank (n, g).
// far_is_source = false: the block's destination rank ((n - j) % N, (g - l) % Q) indexes displs
// (send side); true: its source rank ((n + j) % N, (g + l) % Q) (receive side).
__device__ __forceinline__ unsigned long long block_address(int slot, bool far_is_source, int p, int n, int g,
                                                            int j, int l, int P, int Q, int N,
                                                            unsigned char* user, const int64_t* displs,
                                                            unsigned char* T, long long slots, long long slot_bytes,
                                                            const int32_t* counts = nullptr, int* count = nullptr) {
    if (slot >= 0) return (unsigned long long)(T + ((long long)p * slots + slot) * slot_bytes);
    int pn, pg;
    if (!far_is_source) {
        pn = n - j; if (pn < 0) pn += N;
        pg = g - l; if (pg < 0) pg += Q;
    } else {
        pn = n + j; if (pn >= N) pn -= N;
        pg = g + l; if (pg >= Q) pg -= Q;
    }
    const size_t idx = (size_t)p * P + pn * Q + pg;
    if (counts) *count = counts[idx];          // the caller's count for the same pair (exact size into R)
    return (unsigned long long)(user + displs[idx]);
}

// Exact-size T: where rank p stores segment s of the phase being run, and where rank p holds the
// block with slot index e that phase `ph` stored.
__device__ __forceinline__ unsigned long long exact_t_dst(unsigned char* T, const ExactT& x, int P, int p, int s, int dcls) {
    return (unsigned long long)(T + ((x.tbase[(size_t)dcls * P + p] + (long long)x.tpre[(size_t)p * x.ld + s]) << 4));
}
__device__ __forceinline__ unsigned long long exact_t_src(unsigned char* T, const ExactT& x, int P, int ph, int p, int e,
                                                          int scls) {
    return (unsigned long long)(T + ((x.tbase[(size_t)scls * P + p] + (long long)x.tpos[((size_t)ph * P + p) * P + e]) << 4));
}

// ------------------------------------------------------------------------------------------
// k_resolve_hop: for a one-kernel phase, the source and the destination of every block every rank
// receives (Algorithm "TuNA", lines 15-20 collapsed into one hop: the block goes from where its sender
// holds it -- S at sdispls[sender][destination], or the sender's T -- straight to where its receiver
// keeps it -- R at rdispls[receiver][source], or the receiver's T), in the receiver's message order.
// One thread per (segment, receiving rank).  TP = 1: a workgroup takes 256 segments of one rank, grid
// (ceil(nseg / 256), P).  TP = 16: a workgroup takes 16 segments of each of 16 ranks, grid (ceil(nseg / 16),
// ceil(P / 16)), for phases of many rounds: there neighbouring segments have neighbouring senders, the
// never-moved blocks are looked up in a column of sdispls, and a tile of 16 x 16 touches 31 of its lines
// where 256 segments of one rank touch 256.  Addresses in T are stored as offsets (kHopInT) because a
// persistent plan resolves them before its T is allocated.
// ------------------------------------------------------------------------------------------
struct ResolveArgs {
    HopDev hop;                         // (first: DirectArgs)
    const int32_t* nxt;                 // [P][P] block sizes after the phase's size exchange (the receiver's view); k_resolve_hop only
    const int32_t* sendcounts;          // block sizes for the kernels that find their blocks themselves (block_bytes)
    const int32_t* recvcounts;
    int rx1;                            // r^(x+1) of the phase
    int near_s;                         // 1: the bytes of a block that never moved lie nearer in sendcounts (kNearSendRadix)
    SegDev seg;
    int nseg;
    int P, Q, N, dim, rx;
    const unsigned char* S;
    const int64_t* sdispls;
    unsigned char* R;
    const int64_t* rdispls;
    long long slots;                    // T in slots: slot s of rank p at offset (p * slots + s) * slot_bytes
    long long slot_bytes;
    ExactT x;                           // T in exact size
    int exact_sizes;                    // 1: every size is the block's byte count (k_hop_direct copies exactly that), also into T
};

constexpr int kResolveTile = 16;

template <bool DENSE, int TP>
__global__ void __launch_bounds__(256) k_resolve_hop(const ResolveArgs a) {
    static_assert(TP == 1 || TP == kResolveTile, "one rank or a tile of ranks per workgroup");
    const int s = TP == 1 ? blockIdx.x * 256 + threadIdx.x : blockIdx.x * (256 / TP) + (threadIdx.x % (256 / TP));
    const int p = TP == 1 ? blockIdx.y : blockIdx.y * TP + threadIdx.x / (256 / TP);
    if (s >= a.nseg || p >= a.P) return;
    const int n = p / a.Q, g = p - n * a.Q;
    const int e = a.seg.e[s];
    const int sz = a.nxt[(size_t)p * a.P + e];
    const size_t o = (size_t)p * a.hop.ld + s;
    int j, l;
    split_slot_index(e, a.Q, a.N, j, l);
    const int ssrc = a.seg.src[s], sdst = a.seg.dst[s];
    if (sz <= 0) {
        // an empty block owns no chunk and is never copied; a final one still records where it would lie in
        // R, so that the destination-tiled hop sees the blocks around it as one contiguous run
        unsigned long long d0 = 0;
        if (sdst < 0) {
            int sn = n + j; if (sn >= a.N) sn -= a.N;
            int sg = g + l; if (sg >= a.Q) sg -= a.Q;
            d0 = (unsigned long long)(a.R + a.rdispls[(size_t)p * a.P + sn * a.Q + sg]);
        }
        a.hop.src[o] = 0; a.hop.dst[o] = d0; a.hop.size[o] = 0;
        return;
    }
    // the sender: the rank at distance z r^x upwards in the phase's dimension
    const int q = partner_up(n, g, a.Q, a.N, a.dim, a.seg.z[s] * a.rx);
    unsigned long long src, dst;
    if (ssrc < 0) {                      // never moved: in the sender's S, addressed by its destination rank
        const int qn = q / a.Q, qg = q - qn * a.Q;
        int dn = qn - j; if (dn < 0) dn += a.N;
        int dg = qg - l; if (dg < 0) dg += a.Q;
        src = (unsigned long long)(a.S + a.sdispls[(size_t)q * a.P + dn * a.Q + dg]);
    } else if (DENSE) {
        const size_t row = (size_t)a.seg.srcph[s] * a.P + q;
        src = (((unsigned long long)(a.x.tbase[(size_t)a.seg.scls[s] * a.P + q] + (long long)a.x.tpos[row * a.P + e])) << 4) | kHopInT;
    } else {
        src = (unsigned long long)(((long long)q * a.slots + ssrc) * a.slot_bytes) | kHopInT;
    }
    int size = sz;
    if (sdst < 0) {                      // final: into R at the slot of its source rank, exactly `sz` bytes
        int sn = n + j; if (sn >= a.N) sn -= a.N;
        int sg = g + l; if (sg >= a.Q) sg -= a.Q;
        dst = (unsigned long long)(a.R + a.rdispls[(size_t)p * a.P + sn * a.Q + sg]);
    } else {
        if (!a.exact_sizes) size = ((sz + 15) >> 4) << 4;    // T takes whole chunks
        if (DENSE)
            dst = (((unsigned long long)(a.x.tbase[(size_t)a.seg.dcls[s] * a.P + p] + (long long)a.x.tpre[(size_t)p * a.x.ld + s])) << 4) | kHopInT;
        else
            dst = (unsigned long long)(((long long)p * a.slots + sdst) * a.slot_bytes) | kHopInT | kHopFill;
    }
    a.hop.src[o] = src; a.hop.dst[o] = dst; a.hop.size[o] = size;
}

// ------------------------------------------------------------------------------------------
// k_hop_direct: a one-kernel phase whose blocks are all short (Section "Performance analysis of TuNA": the
// small-message regime).  The byte-balanced engine cuts work into 4 KiB units and searches a window of block
// boundaries per unit; with short blocks the prefix scans, unit lists and searches are most of a phase.  Here a
// workgroup takes the blocks of 16 neighbouring receivers x SEGS neighbouring segments, one lane resolves one
// block -- where its sender holds it, where its receiver keeps it, how long it is -- and LPB lanes move it, 16
// bytes each, so LPB x 16 bytes is the longest block the kernel takes.  No scan, no unit list and, except for a
// plan's (RESOLVED), no hop arrays: 40 bytes per block that would be written and read back.
//   Bound by memory: the entries of the matrices it looks up and the payload, both in whole lines.  Blocks that
// never moved are looked up down a column of sdispls and lie, for neighbouring receivers, side by side in a
// sender's S: the 16 receivers of a tile share those lines; the SEGS blocks of one receiver lie side by side in R.
//   A block of 16 bytes and more is moved in 16-byte accesses at its own alignment, the last one ending with the
// block and overlapping the one before it (the same bytes are stored twice); a shorter one by the lane that
// resolved it in two overlapping accesses of 8 or 4 bytes, or byte by byte.  Only bytes of the block are read.
//   Measured per call against one thread per block (up to 64 bytes) and the engine (above), both from hop arrays:
// 33 M blocks of 64 bytes and as many empty ones (P = 8192, linear) 6.91 -> 1.57 ms; uniform [0, 16] B, P = 2048, two
// phases 0.44 -> 0.27 ms; uniform [0, 248] B, P = 4096, linear 1.64 -> 1.24 ms.  Blocks of more than 64 bytes and payloads
// beyond the caches are better off in k_hop_rows (block_kernel).
//   TALL tiles (16 receivers x few segments, LPB = 1 and 4) share the lines of S and sdispls between receivers: that pays
// when a round has few blocks, as in the linear schedule (64-byte blocks: 1.57 against 2.0 ms), or neighbouring segments are of other rounds,
// as in the first phase in the order of the slot indices (direct_tall).  With many blocks of one round side by side neighbouring receivers read
// other rows, and long rows of one receiver are better (uniform [0, 16] B, two phases in message order: 0.26 against 0.33 ms).
//   STREAM: 1 = streaming stores (chunk-granular data; -4 %, but +5 % and more where blocks share 16-byte chunks),
// 2 = streaming loads too (whole lines; another -4 %).
//   Payload bytes and 16-byte chunks are summed per receiver and stored as one partial result per tile column
// (a.part); k_phase_sums adds them up.
// ------------------------------------------------------------------------------------------
constexpr int kDirectMaxBytes = 256;        // longest block of the LPB = 16 kernel
// the tile of one workgroup and step: receivers per wave, blocks per lane (of neighbouring receivers), waves side by
// side along the receivers (the others along the segments)
struct DirectShape { int wave_ranks, sets, waves_r; };
constexpr DirectShape direct_shape(int lpb, bool tall) {
    return tall ? (lpb == 1 ? DirectShape{1, 4, 4} : lpb == 4 ? DirectShape{4, 1, 4} : DirectShape{1, 1, 4})
                : (lpb == 1 ? DirectShape{1, 4, 1} : DirectShape{2, 1, 4});
}
constexpr int direct_segs(DirectShape s) { return kWave / s.wave_ranks * (4 / s.waves_r); }
constexpr int direct_ranks(DirectShape s) { return s.wave_ranks * s.sets * s.waves_r; }
// What a kernel with hop arrays reads comes first, in one 64-byte line: a wave that is launched waits for its arguments line after line.  Three
// lines / two / one, us per start, up to 1 KiB: 60 ranks, r = 2 30.2 / 29.0 / 27.9, 150, r = 16 15.9 / - / 15.0, 256, r = 2 83.1 / 81.3 / 79.4, 400, r = 3
// 134.7 / - / 132.0; up to 200 bytes, 500, r = 4 49.6 / - / 48.9.
struct DirectArgs {
    unsigned char* T;
    unsigned long long user_limit;      // address one past the last byte of S that holds a block
    int seg_lo, seg_hi;
    union {
        int iters;                      // steps of segments per workgroup (k_hop_direct)
        int segs;                       // segments per wave, at most 64 (k_hop_rows)
    };
    int own;                            // so many rows of workgroups in front move the ranks' own blocks (k_hop_direct, k_hop_rows)
    ResolveArgs r;                      // hop: only when RESOLVED
    uint2* part;                        // [grid.x][P]: payload bytes and chunks of the tile column, per receiver (null: not wanted)
};
static_assert(offsetof(DirectArgs, r) + offsetof(ResolveArgs, nxt) == 64, "one line");

typedef v4u v4u_any __attribute__((aligned(1)));
typedef unsigned long long u64_any __attribute__((aligned(1)));
typedef unsigned int u32_any __attribute__((aligned(1)));
#define TUNA_GLOBAL __attribute__((address_space(1)))
template <class T> __device__ __forceinline__ T load_global(unsigned long long a) { return *(const TUNA_GLOBAL T*)a; }
template <class T, class V> __device__ __forceinline__ void store_global(unsigned long long a, V v) { *(TUNA_GLOBAL T*)a = v; }

// A block of fewer than 16 bytes (up to 16 in the LPB = 1 kernel), by one lane.  The loads are made without a
// branch, from `dummy` where the block is of another kind: a load under a branch is waited for at the branch's end,
// so the loads of several blocks would go out one after the other.  Blocks of 1 to 3 bytes are left to short_store.
struct ShortBlock { unsigned long long w0, w1; unsigned int x0, x1; };
__device__ __forceinline__ ShortBlock short_load(unsigned long long src, int n, unsigned long long dummy) {
    const bool one = n >= 4 && n < 8;
    ShortBlock b;
    b.w0 = load_global<u64_any>(n >= 8 ? src : dummy);
    b.w1 = load_global<u64_any>(n > 8 ? src + n - 8 : dummy);
    b.x0 = load_global<u32_any>(one ? src : dummy);
    b.x1 = load_global<u32_any>(one && n > 4 ? src + n - 4 : dummy);
    return b;
}
__device__ __forceinline__ void short_store(unsigned long long dst, unsigned long long src, int n, const ShortBlock& b) {
    if (n >= 8) {
        store_global<u64_any>(dst, b.w0);
        if (n > 8) store_global<u64_any>(dst + n - 8, b.w1);
    } else if (n >= 4) {
        store_global<u32_any>(dst, b.x0);
        if (n > 4) store_global<u32_any>(dst + n - 4, b.x1);
    } else if (n > 0) {
        const unsigned char c0 = load_global<unsigned char>(src), c1 = load_global<unsigned char>(src + (n >> 1)), c2 = load_global<unsigned char>(src + n - 1);
        store_global<unsigned char>(dst, c0); store_global<unsigned char>(dst + (n >> 1), c1); store_global<unsigned char>(dst + n - 1, c2);
    }
}

// Where the bytes of a block are written down.  Block (j, l) of rank (n, g) in phase (dim, x), after its hop: it has
// covered the digits up to x of its distance, so it comes from O = (n, g) + that part and is bound for D = O - (j, l)
// (Algorithm "TuNA", line 14, without the exchange: in one memory every size can be looked up where the caller wrote
// it).  The entry of recvcounts is the nearer one where neighbouring blocks have one destination (final blocks, and
// all later phases: runs of r^(x+1) blocks), that of sendcounts where they have one origin: blocks that never moved before, while
// r^(x+1) is below kNearSendRadix (near_s; runs of r^(x+1) in P / r^(x+1) rows of recvcounts against r^x - 1 strided rows of sendcounts).
// Never / below 8 / always, us per call: up to 16 B, P = 2048, r = 3 440 / 430 / 442, r = 4 370 / 366 / 375, r = 8 275 / 274 / 286, r = 46 139 / 138 / 150, P =
// 4000, r = 2 2281 / 2244 / 2301, r = 16 810 / 810 / 853; up to 60, P = 2048, r = 4 631 / 630 / 644, P = 1000, r = 6 140 / 137 / 140; up to 200, P = 1000, r = 46
// 133 / 133 / 139; 500 ranks the same.
constexpr int kNearSendRadix = 8;
__device__ __forceinline__ const int32_t* block_bytes(const int32_t* sendcounts, const int32_t* recvcounts, bool in_s, int n, int g, int j,
                                                      int l, int P, int Q, int N, int dim, int rx1) {
    int on = n, og = g + l;
    if (dim == 0) og = g + (int)((unsigned int)l % (unsigned int)rx1);
    else on = n + (int)((unsigned int)j % (unsigned int)rx1);
    if (og >= Q) og -= Q;
    if (on >= N) on -= N;
    int dn = on - j; if (dn < 0) dn += N;
    int dg = og - l; if (dg < 0) dg += Q;
    const int o = on * Q + og, d = dn * Q + dg;
    return in_s ? sendcounts + (size_t)o * P + d : recvcounts + (size_t)d * P + o;
}

// ------------------------------------------------------------------------------------------
// k_t_places, k_t_bases: exact-size T for phases that find their blocks themselves: the places of the blocks that every
// phase stores into T, of all phases at once -- block sizes come from the caller's matrices (block_bytes), so no phase
// waits for another's size exchange.  k_t_places: one workgroup per receiver and class scans the chunks of the class's
// blocks in the order of the segments, that is of the slot indices (slot_order); the offsets inside the receiver's part go to tpos by segment,
// the part's size to csub.  A copy of the first phase's offsets and sizes by segment, which
// paid in message order, costs now: P = 2048, r = 46 161 -> 182 us per call, uniform [0, 64] B, P = 4096, r = 64 1181 -> 1240.
// k_t_places_slots: the same for larger radices, the sizes read for all slot indices in turn: consecutive ones of one round after
// the other are consecutive entries of a row of recvcounts and of tpos.  They go through the LDS to be scanned
// in the order of the segments and back.  What bounds k_t_places then is the lines it touches
// (P = 2048, r = 46: 435 MB missed in the L2s, 73 us for 16 MB of sizes).  Per call, k_t_places / k_t_places_slots: uniform [0, 16]
// B, P = 2048, r = 46 236 / 184 us; uniform [0, 64] B, P = 4096, r = 64 1.72 / 1.54 ms; uniform [0, 512] B, P = 2048, r = 46 1017 / 972
// us; uniform [0, 16] B, P = 6000, r = 77 2.62 / 2.22 ms; 64-byte blocks, P = 8192, r = 90 5.19 / 4.67 ms; r = 16 255 / 252 us; r = 8 1767 /
// 1734 us and 23.38 / 23.34 ms; but r = 4, whose 15 classes each go through all slot indices, P = 1500
// 586 / 602.  (Neighbouring receivers on one XCD, so that they share those lines in its L2: 195 us at r = 46, but r = 8 +4 %.)
// k_t_bases: one workgroup per class.  Two launches per call in place of four per phase (rotation and size exchange
// included): P = 256, r = 4, four phases 174 -> 138 us per call, uniform [0, 100] B, P = 1500, r = 4 682 -> 598 us.
// ------------------------------------------------------------------------------------------
constexpr int kPlaceClasses = 28;           // 8 phases
constexpr int kPlaceMaxPhases = 24;         // P <= 32768 has at most 16
struct PlacePhase {
    const int32_t* e;       // the phase's table (SegDev)
    const int32_t* src;
    const int32_t* tord;    // its T-bound segments by class (ExactT)
    const int32_t* tcls;
    int phase;              // its index in the schedule
    int first;              // workgroup row of its first class
    int dim, rx1;
};
struct PlaceArgs {
    PlacePhase ph[kPlaceMaxPhases];
    int nph;                // the phases that store into T
    int P, Q, N;
    const int32_t* sendcounts;
    const int32_t* recvcounts;
    ExactT x;
    int most;               // blocks of the largest class
    int own;                // workgroup row that moves the ranks' own blocks (own_block), or -1
    const unsigned char* S;
    const int64_t* sdispls;
    unsigned char* R;
    const int64_t* rdispls;
    int by_value;           // the classes' first chunks are here, not in x.cbase: no copy to the device before the kernels
    long long cbase[kPlaceClasses];
    // the phases' totals, if wanted: payload bytes and chunks of every class row and, behind those, of the final blocks of each of
    // nfin phases, per receiver
    ulonglong2* part;       // [rows + nfin][P]
    int rows, nfin;
    int fin[kPlaceMaxPhases + 1];       // the final blocks of phase x are the slot indices fin[x] .. fin[x + 1] - 1
    Status* st;
    // kernels that run before the host has seen what validation found: nothing is to be done where it says so (no_places)
    int slots_rule;         // full slots are taken (slots_are_full)
    int max_block;
};
// T in the paper's slots of M bytes is at least 90 % full: see choose_exact_t
__host__ __device__ inline bool slots_are_full(unsigned long long total_bytes, int P, int max_count) {
    const double slot_bytes = (double)((max_count + 127) / 128 * 128);
    return (double)total_bytes >= 0.9 * (double)P * (double)P * slot_bytes;
}
// verdict: null where it is not known when the kernels run
__device__ __forceinline__ bool no_places(const PlaceArgs& a, const Status::Verdict* verdict) {
    if (!verdict) return false;
    const Status::Verdict st = *verdict;
    return (st.flags & 7u) || st.total_bytes == 0 || st.max_count > a.max_block || (a.slots_rule && slots_are_full(st.total_bytes, a.P, st.max_count));
}
// Sum over a workgroup of kScanThreads, in its thread 0.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long v, unsigned long long* wsum) {
    v = last_lane<kWave>(v, 0ull, AddOp());
    __syncthreads();                                      // wsum of the sum before is consumed
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) wsum[threadIdx.x / kWave] = v;
    __syncthreads();
    v = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k) v += wsum[k];
    return v;
}
// Payload bytes and chunks, cut at the 16-byte boundaries of R, of the blocks that receiver p gets for good in phase x: this
// thread's share, one in `threads`.
__device__ __forceinline__ void final_shares(const PlaceArgs& a, int p, int x, int thread, int threads, unsigned long long& bytes,
                                             unsigned long long& chunks) {
    const int P = a.P, hi = a.fin[x + 1];
    int pn, pg;
    split_slot_index(p, a.Q, a.N, pn, pg);
    bytes = chunks = 0;
#pragma unroll 4
    for (int e = a.fin[x] + thread; e < hi; e += threads) {
        int j, l;
        split_slot_index(e, a.Q, a.N, j, l);
        int sn = pn + j; if (sn >= a.N) sn -= a.N;
        int sg = pg + l; if (sg >= a.Q) sg -= a.Q;
        const size_t at = (size_t)p * P + sn * a.Q + sg;
        const int n = a.recvcounts[at];
        const unsigned int head = (unsigned int)((unsigned long long)a.R + (unsigned long long)a.rdispls[at]) & 15u;
        bytes += (unsigned long long)(unsigned int)n;
        chunks += n > 0 ? (head + (unsigned int)n + 15u) >> 4 : 0u;
    }
}
__device__ __forceinline__ void final_totals(const PlaceArgs& a, int p, int x) {
    __shared__ unsigned long long s_sum[kScanThreads / kWave];
    unsigned long long bytes, chunks;
    final_shares(a, p, x, threadIdx.x, kScanThreads, bytes, chunks);
    bytes = block_sum(bytes, s_sum);
    chunks = block_sum(chunks, s_sum);
    if (threadIdx.x == 0) a.part[(size_t)(a.rows + x) * a.P + p] = make_ulonglong2(bytes, chunks);
}
// k_row_totals: the totals of a linear schedule's only phase, a wave per receiver.  Validation has cleared them.
__global__ void __launch_bounds__(kScanThreads) k_row_totals(const PlaceArgs a, const Status::Verdict* verdict) {
    __shared__ unsigned long long s_sum[kScanThreads / kWave];
    if (no_places(a, verdict)) return;
    const int lane = threadIdx.x & (kWave - 1), p = blockIdx.x * (kScanThreads / kWave) + threadIdx.x / kWave;
    unsigned long long bytes = 0, chunks = 0;
    if (p < a.P) {
        final_shares(a, p, 0, lane, kWave, bytes, chunks);
        chunks = last_lane<kWave>(chunks, 0ull, AddOp());
        chunks = lane == kWave - 1 ? (chunks + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks : 0;
    }
    bytes = block_sum(bytes, s_sum);
    chunks = block_sum(chunks, s_sum);
    if (threadIdx.x == 0) { atomicAdd(&a.st->phase_bytes[0], bytes); atomicAdd(&a.st->phase_chunks[0], chunks); }
}
// The totals of phase x from those, every receiver's chunks rounded up to a line as the staging layouts round them.
__device__ __forceinline__ void phase_totals(const PlaceArgs& a, int x) {
    __shared__ unsigned long long s_sum[kScanThreads / kWave];
    int lo = 0, hi = 0;                                   // its class rows
    for (int f = 0; f < a.nph; ++f)
        if (a.ph[f].phase == x) { lo = a.ph[f].first; hi = f + 1 < a.nph ? a.ph[f + 1].first : a.rows; }
    unsigned long long bytes = 0, chunks = 0;
    for (int p = threadIdx.x; p < a.P; p += kScanThreads) {
        ulonglong2 v = a.part[(size_t)(a.rows + x) * a.P + p];
        unsigned long long c = v.y;
        bytes += v.x;
#pragma unroll 4
        for (int k = lo; k < hi; ++k) { v = a.part[(size_t)k * a.P + p]; bytes += v.x; c += v.y; }
        chunks += (c + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks;
    }
    bytes = block_sum(bytes, s_sum);
    chunks = block_sum(chunks, s_sum);
    if (threadIdx.x == 0) { a.st->phase_bytes[x] = bytes; a.st->phase_chunks[x] = chunks; }
}
__device__ __forceinline__ int place_phase(const PlaceArgs& a, int row) {
    int f = 0;
    while (f + 1 < a.nph && a.ph[f + 1].first <= row) ++f;
    return f;
}
__global__ void __launch_bounds__(kScanThreads) k_t_places(const PlaceArgs a, const Status::Verdict* verdict) {
    __shared__ int wsum[kScanThreads / kWave];
    __shared__ unsigned long long s_sum[kScanThreads / kWave];
    const int p = blockIdx.x, P = a.P;
    if ((int)blockIdx.y == a.own) { own_block(a.S, a.sendcounts, a.sdispls, a.R, a.rdispls, P, p); return; }
    if (no_places(a, verdict)) return;
    if ((int)blockIdx.y >= a.rows) { final_totals(a, p, blockIdx.y - a.rows); return; }
    const int f = place_phase(a, blockIdx.y);
    const PlacePhase& ph = a.ph[f];
    const int32_t* cls = ph.tcls + 3 * (blockIdx.y - ph.first);
    const int cid = cls[0], c0 = cls[1], cn = cls[2];
    int pn, pg;
    split_slot_index(p, a.Q, a.N, pn, pg);
    int* pos_t = a.x.tpos + ((size_t)ph.phase * P + p) * P;
    int carry = 0;
    unsigned long long bytes = 0;
    for (int base = 0; base < cn; base += kScanThreads * kScanItems) {
        int ct[kScanItems], sg[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int i = base + scan_item_index(k);
            sg[k] = ph.tord[c0 + min(i, cn - 1)];
            int j, l;
            split_slot_index(ph.e[sg[k]], a.Q, a.N, j, l);
            const int n = *block_bytes(a.sendcounts, a.recvcounts, ph.src[sg[k]] < 0, pn, pg, j, l, P, a.Q, a.N, ph.dim, ph.rx1);
            ct[k] = i < cn ? (n + 15) >> 4 : 0;
            bytes += i < cn ? (unsigned long long)(unsigned int)n : 0ull;
        }
        int run[kScanItems];
        block_scan_batch(ct, run, carry, wsum);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + scan_item_index(k) < cn) pos_t[sg[k]] = run[k];
    }
    if (a.part) bytes = block_sum(bytes, s_sum);
    if (threadIdx.x != 0) return;
    a.x.csub[(size_t)cid * P + p] = carry;
    if (a.part) a.part[(size_t)blockIdx.y * P + p] = make_ulonglong2(bytes, (unsigned long long)carry);
}
constexpr int kPlaceSlotRanks = 8192;       // 48 KiB of LDS
constexpr int kPlaceSlotRadix = 8;
// dynamic LDS: the blocks of the largest class (a.most), 4 bytes each, and 2 bytes per slot index
__global__ void __launch_bounds__(kScanThreads) k_t_places_slots(const PlaceArgs a, const Status::Verdict* verdict) {
    extern __shared__ int s_val[];                       // bytes by index inside the class
    __shared__ int wsum[kScanThreads / kWave];
    __shared__ unsigned long long s_sum[kScanThreads / kWave];
    constexpr int kNone = 0xffff;
    unsigned short* s_at = reinterpret_cast<unsigned short*>(s_val + a.most);        // by slot index: the index inside the class
    const int p = blockIdx.x, P = a.P;
    if ((int)blockIdx.y == a.own) { own_block(a.S, a.sendcounts, a.sdispls, a.R, a.rdispls, P, p); return; }
    if (no_places(a, verdict)) return;
    if ((int)blockIdx.y >= a.rows) { final_totals(a, p, blockIdx.y - a.rows); return; }
    const int f = place_phase(a, blockIdx.y);
    const PlacePhase& ph = a.ph[f];
    const int32_t* cls = ph.tcls + 3 * (blockIdx.y - ph.first);
    const int cid = cls[0], c0 = cls[1], cn = cls[2];
    int pn, pg;
    split_slot_index(p, a.Q, a.N, pn, pg);
    for (int e = threadIdx.x; e < P; e += kScanThreads) s_at[e] = kNone;
    __syncthreads();
    for (int i = threadIdx.x; i < cn; i += kScanThreads) s_at[ph.e[ph.tord[c0 + i]]] = (unsigned short)i;
    __syncthreads();
    for (int base = 0; base < P; base += kScanThreads * kScanItems) {
        int at[kScanItems], sz[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int e = base + k * kScanThreads + threadIdx.x;
            at[k] = e < P ? s_at[e] : kNone;
            int j, l;
            split_slot_index(min(e, P - 1), a.Q, a.N, j, l);
            const int32_t* from = block_bytes(a.sendcounts, a.recvcounts, false, pn, pg, j, l, P, a.Q, a.N, ph.dim, ph.rx1);
            sz[k] = *(at[k] != kNone ? from : a.recvcounts);
        }
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (at[k] != kNone) s_val[at[k]] = sz[k];
    }
    __syncthreads();
    int* pos_t = a.x.tpos + ((size_t)ph.phase * P + p) * P;
    int carry = 0;
    unsigned long long bytes = 0;
    for (int base = 0; base < cn; base += kScanThreads * kScanItems) {
        int ct[kScanItems], sg[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int i = base + scan_item_index(k);
            ct[k] = i < cn ? (s_val[i] + 15) >> 4 : 0;
            bytes += i < cn ? (unsigned long long)(unsigned int)s_val[i] : 0ull;
            sg[k] = ph.tord[c0 + min(i, cn - 1)];
        }
        int run[kScanItems];
        block_scan_batch(ct, run, carry, wsum);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int i = base + scan_item_index(k);
            if (i < cn) pos_t[sg[k]] = run[k];
        }
    }
    if (a.part) bytes = block_sum(bytes, s_sum);
    if (threadIdx.x != 0) return;
    a.x.csub[(size_t)cid * P + p] = carry;
    if (a.part) a.part[(size_t)blockIdx.y * P + p] = make_ulonglong2(bytes, (unsigned long long)carry);
}
__global__ void __launch_bounds__(kScanThreads) k_t_bases(const PlaceArgs a) {
    __shared__ long long wc[kScanThreads / kWave];
    if ((int)blockIdx.x >= a.rows) { phase_totals(a, blockIdx.x - a.rows); return; }
    const PlacePhase& ph = a.ph[place_phase(a, blockIdx.x)];
    const int cid = ph.tcls[3 * (blockIdx.x - ph.first)];
    class_base(a.x, cid, a.by_value ? a.cbase[cid] : a.x.cbase[cid], a.P, wc);
}

// The blocks that the lanes of a wave have found, SETS each: LPB lanes move one, or its own lane (LPB = 1).  dummy: any 16
// bytes that can be read.
template <int LPB> struct ShortLds { unsigned long long src[4][kWave], dst[4][kWave]; int n[4][kWave]; };
template <> struct ShortLds<1> {};
template <int LPB, int STREAM, int SETS>
__device__ __forceinline__ void move_short(const unsigned long long (&src)[SETS], const unsigned long long (&dst)[SETS], const int (&n)[SETS],
                                           unsigned long long dummy, ShortLds<LPB>& lds) {
    if constexpr (LPB == 1) {
        ShortBlock b[SETS];
#pragma unroll
        for (int u = 0; u < SETS; ++u) b[u] = short_load(src[u], n[u], dummy);
#pragma unroll
        for (int u = 0; u < SETS; ++u) short_store(dst[u], src[u], n[u], b[u]);
    } else {
        static_assert(SETS == 1, "a lane finds one block, LPB lanes move it");
        constexpr int BPS = kWave / LPB;                 // blocks a wave moves per step of its copy loop
        constexpr int FLIGHT = LPB < 8 ? LPB : 8;        // steps whose loads are in flight together
        const int lane = threadIdx.x & (kWave - 1);
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        // the wave's 64 blocks go to its own part of the LDS; no workgroup barrier
        lds.src[wv][lane] = src[0]; lds.dst[wv][lane] = dst[0]; lds.n[wv][lane] = n[0];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int c = (lane & (LPB - 1)) * 16;
#pragma unroll
        for (int k0 = 0; k0 < LPB; k0 += FLIGHT) {
            v4u v[FLIGHT];
            int o[FLIGHT];                               // byte inside the block, or -1
#pragma unroll
            for (int k = 0; k < FLIGHT; ++k) {
                const int b = (k0 + k) * BPS + lane / LPB;
                const int nb = lds.n[wv][b];
                o[k] = nb >= 16 && c < nb ? min(c, nb - 16) : -1;
                const TUNA_GLOBAL v4u_any* from = (const TUNA_GLOBAL v4u_any*)(o[k] >= 0 ? lds.src[wv][b] + (unsigned int)o[k] : dummy);
                v[k] = STREAM == 2 ? __builtin_nontemporal_load(from) : *from;
            }
            // The destinations are read from the LDS here and not kept in registers from above (LPB = 16 98 -> 78 of them, 4
            // -> 6 waves per SIMD): up to 250 bytes, P = 600, r = 4 159 -> 153 us per call, up to 64, P = 2048 708 -> 696.
            asm volatile("" ::: "memory");
#pragma unroll
            for (int k = 0; k < FLIGHT; ++k)
                if (o[k] >= 0) {
                    const unsigned long long d = lds.dst[wv][(k0 + k) * BPS + lane / LPB] + (unsigned int)o[k];
                    if (STREAM) __builtin_nontemporal_store(v[k], (TUNA_GLOBAL v4u_any*)d);
                    else store_global<v4u_any>(d, v[k]);
                }
        }
        // blocks of fewer than 16 bytes: the lane that resolved them
        const int ns = n[0] < 16 ? n[0] : 0;
        if (__ballot(ns > 0)) short_store(dst[0], src[0], ns, short_load(src[0], ns, dummy));
        __builtin_amdgcn_wave_barrier();                 // the next step overwrites the wave's LDS
    }
}

// The own blocks, of up to kDirectMaxBytes, of the kOwnRanks ranks from p0 on, 16 lanes each.
constexpr int kOwnRanks = 16;
__device__ __forceinline__ void own_short(const ResolveArgs& r, int p0) {
    const int p = p0 + threadIdx.x / 16, lane = threadIdx.x & 15;
    if (p >= r.P) return;
    const size_t d = (size_t)p * r.P + p;
    const int n = r.sendcounts[d];
    const unsigned long long src = (unsigned long long)r.S + (unsigned long long)r.sdispls[d], dst = (unsigned long long)r.R + (unsigned long long)r.rdispls[d];
    if (n < 16) {
        if (lane < n) store_global<unsigned char>(dst + lane, load_global<unsigned char>(src + lane));
        return;
    }
    for (int c = lane * 16; c < n; c += 256) {
        const unsigned int o = (unsigned int)min(c, n - 16);
        store_global<v4u_any>(dst + o, load_global<v4u_any>(src + o));
    }
}

template <int LPB, bool TALL, int STREAM, bool DENSE, bool RESOLVED>
__device__ __forceinline__ void hop_direct(const DirectArgs& a) {
    constexpr DirectShape SH = direct_shape(LPB, TALL);
    constexpr int SEGS = kWave / SH.wave_ranks;          // segments per wave and step
    constexpr int SETS = SH.sets;                        // blocks a lane resolves per step
    constexpr int WS = 4 / SH.waves_r;                   // waves side by side along the segments
    __shared__ ShortLds<LPB> lds;
    const ResolveArgs& r = a.r;
    if ((int)blockIdx.y < a.own) { own_short(r, (int)(blockIdx.y * gridDim.x + blockIdx.x) * kOwnRanks); return; }
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int P = r.P, Q = r.Q, N = r.N;
    const int p0 = (blockIdx.y - a.own) * direct_ranks(SH) + (wv / WS) * SH.wave_ranks * SETS + lane / SEGS;
    const int sub = lane & (SEGS - 1);
    const unsigned long long tb = (unsigned long long)a.T;
    unsigned int sum_b[SETS], sum_c[SETS];
#pragma unroll
    for (int u = 0; u < SETS; ++u) sum_b[u] = sum_c[u] = 0;
    for (int it = 0; it < a.iters; ++it) {
        const int s0 = a.seg_lo + ((blockIdx.x * a.iters + it) * WS + wv % WS) * SEGS;
        if (s0 >= a.seg_hi) break;
        const int s = min(s0 + sub, a.seg_hi - 1);
        const bool in = s0 + sub < a.seg_hi;
        unsigned long long src[SETS], dst[SETS];
        int n[SETS];
        // ---- where every block is and goes: loads from valid addresses without branches, so that they go out together
        if (RESOLVED) {
#pragma unroll
            for (int u = 0; u < SETS; ++u) {
                const size_t o = (size_t)min(p0 + u, P - 1) * r.hop.ld + s;
                n[u] = r.hop.size[o]; src[u] = r.hop.src[o]; dst[u] = r.hop.dst[o];
            }
#pragma unroll
            for (int u = 0; u < SETS; ++u) {
                src[u] = (src[u] & ~(kHopInT | kHopFill)) + ((src[u] & kHopInT) ? tb : 0ull);
                dst[u] = (dst[u] & ~(kHopInT | kHopFill)) + ((dst[u] & kHopInT) ? tb : 0ull);
            }
        } else {
            const int e = r.seg.e[s], dist = r.seg.z[s] * r.rx, ssrc = r.seg.src[s], sdst = r.seg.dst[s];
            const int sph = DENSE ? r.seg.srcph[s] : 0, sseg = DENSE ? r.seg.srcseg[s] : 0, scl = DENSE ? r.seg.scls[s] : 0, dcl = DENSE ? r.seg.dcls[s] : 0;
            const bool in_s = ssrc < 0, in_r = sdst < 0;  // read from S (never moved), stored into R (final)
            int j, l;
            split_slot_index(e, Q, N, j, l);
            long long va[SETS], vc[SETS];
            int vb[SETS], vd[SETS], q[SETS];
#pragma unroll
            for (int u = 0; u < SETS; ++u) {
                const int p = min(p0 + u, P - 1);
                int pn, pg;
                split_slot_index(p, Q, N, pn, pg);
                q[u] = partner_up(pn, pg, Q, N, r.dim, dist);
                int qn, qg;
                split_slot_index(q[u], Q, N, qn, qg);
                int dn = qn - j; if (dn < 0) dn += N;
                int dg = qg - l; if (dg < 0) dg += Q;
                int sn = pn + j; if (sn >= N) sn -= N;
                int sg = pg + l; if (sg >= Q) sg -= Q;
                const size_t at_s = (size_t)q[u] * P + dn * Q + dg, at_r = (size_t)p * P + sn * Q + sg;
                n[u] = *(in_r ? r.recvcounts + at_r : block_bytes(r.sendcounts, r.recvcounts, in_s && r.near_s, pn, pg, j, l, P, Q, N, r.dim, r.rx1));
                const int64_t* tbase = reinterpret_cast<const int64_t*>(r.x.tbase);
                va[u] = *(in_s ? r.sdispls + at_s : (DENSE ? tbase + (size_t)scl * P + q[u] : r.sdispls));
                vc[u] = *(in_r ? r.rdispls + at_r : (DENSE ? tbase + (size_t)dcl * P + p : r.rdispls));
                if (DENSE) {
                    vb[u] = *(in_s ? r.seg.e : r.x.tpos + ((size_t)sph * P + q[u]) * P + sseg);
                    vd[u] = *(in_r ? r.seg.e : r.x.tpos + ((size_t)r.x.phase * P + p) * P + s);
                }
            }
#pragma unroll
            for (int u = 0; u < SETS; ++u) {
                const int p = min(p0 + u, P - 1);
                if (DENSE) {
                    src[u] = in_s ? (unsigned long long)r.S + va[u] : tb + ((unsigned long long)(va[u] + vb[u]) << 4);
                    dst[u] = in_r ? (unsigned long long)r.R + vc[u] : tb + ((unsigned long long)(vc[u] + vd[u]) << 4);
                } else {
                    src[u] = in_s ? (unsigned long long)r.S + va[u] : tb + (unsigned long long)(((long long)q[u] * r.slots + ssrc) * r.slot_bytes);
                    dst[u] = in_r ? (unsigned long long)r.R + vc[u] : tb + (unsigned long long)(((long long)p * r.slots + sdst) * r.slot_bytes);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < SETS; ++u) {
            if (!in || p0 + u >= P) n[u] = 0;
            n[u] = min(n[u], 16 * LPB);                  // validation has bounded it: nothing is cut here
            sum_b[u] += (unsigned int)n[u];
            // chunks as the staging layouts count them: cut at the 16-byte boundaries of R
            if (!RESOLVED) sum_c[u] += n[u] > 0 ? ((r.seg.dst[s] < 0 ? (unsigned int)(dst[u] & 15ull) : 0u) + (unsigned int)n[u] + 15u) >> 4 : 0u;
        }
        move_short<LPB, STREAM>(src, dst, n, (unsigned long long)r.seg.e, lds);
    }
    if (!RESOLVED && a.part) {
#pragma unroll
        for (int u = 0; u < SETS; ++u) {
#pragma unroll
            for (int d = SEGS / 2; d > 0; d >>= 1) { sum_b[u] += __shfl_xor(sum_b[u], d, kWave); sum_c[u] += __shfl_xor(sum_c[u], d, kWave); }
            if (sub == 0 && p0 + u < P) a.part[((size_t)blockIdx.x * WS + wv % WS) * P + p0 + u] = make_uint2(sum_b[u], sum_c[u]);
        }
    }
}

template <int LPB, bool TALL, int STREAM, bool DENSE, bool RESOLVED>
__global__ void __launch_bounds__(256) k_hop_direct(const DirectArgs a) { hop_direct<LPB, TALL, STREAM, DENSE, RESOLVED>(a); }

// ------------------------------------------------------------------------------------------
// k_hop_senders: k_hop_direct under a name of its own in phases of many rounds of schedules of several phases (by_senders), whose tiles have a
// sender's blocks side by side.  Many rounds have many senders, and with the segments in the order of the slot indices (slot_order) a phase's
// senders change either from segment to segment -- the first phase, r^x = 1: neighbouring receivers then get neighbouring blocks of a sender, so
// tiles are TALL, 16 receivers x 16 rounds = 31 senders with up to 16 blocks each, stored as 16 runs of T -- or after r^x
// segments, and a row of one receiver's segments is a run of a sender's part of T and of R (direct_tall).  The code is k_hop_direct's; what the
// rule decides is who moves the own blocks (own_in_first) and what the cost model asks, and traces keep these phases apart.
//   Bound by memory, the lines of the matrices and of T's places above all.  Against workgroups that take the blocks that one rank sends
// (its loads together, its stores a receiver each), us per call: uniform [0, 16] B, P = 2048, r = 46 162 / 148, P = 6000, r = 77 1796 / 1509,
// P = 1024, r = 32 76.5 / 73; up to 64 B, P = 4096, r = 64 1203 / 1135, up to 60, P = 2048, r = 16 409 / 391, P = 1024, r = 32 93 / 95; up to 40, r = 13
// 346 / 335; T in slots, up to 16 B, P = 1000, r = 32 77 / 70, up to 60, r = 64 97 / 90, P = 4096, r = 64 1605 / 1627, r = 16 2586 / 2665.
// ------------------------------------------------------------------------------------------
constexpr int kSenderMinRounds = 12, kSenderMaxRounds = 1024;
template <int LPB, int STREAM, bool DENSE, bool TALL>
__global__ void __launch_bounds__(256) k_hop_senders(const DirectArgs a) { hop_direct<LPB, TALL, STREAM, DENSE, false>(a); }

// ------------------------------------------------------------------------------------------
// k_hop_pairs: k_hop_direct for the only phase of a linear schedule, where every block goes from S to R in its only hop: a
// tile of senders x receivers in the order of the ranks instead of receivers x rounds.  The rows of recvcounts, sdispls and
// rdispls that a tile needs are whole lines (a tile of rounds is a parallelogram in them: 11 KB of lines for the 5 KB of 256
// blocks), no table is read, and the ranks' own blocks are on the diagonal: no launch for them.
//   Bound by memory.  k_hop_direct / k_hop_pairs, us per call: up to 16 bytes, P = 1024 57 / 48, 3000 198 / 163, 8192 1455 / 1124;
// up to 60, P = 5000 866 / 823, 32-byte blocks, P = 4096 464 / 401, the FFT's 64-byte ones, P = 8192 1574 / 1474; up to
// 200, P = 1000 82 / 77, 2500 457 / 444, up to 256, P = 1200 159 / 153, 500 55 / 50; P = 50 to 300, whose own blocks k_hop_direct takes
// along too, 40-43 / 41-43, up to 200 bytes, P = 2000 260 / 263.
//   The tile: up to 16 bytes 32 x 32 (2 x 2 blocks per lane instead of 4: 3000 176; 64 senders 173, 16 178).  Up to 64 bytes 16 x 16,
// and 8 x 32 where blocks share no 16 bytes and the runs of S that a tile reads count (FFT 1568 with 16 x 16, 1474; P = 5000 823 and
// 836, Zipf up to 64, P = 6000 803 and 886; 32 x 8 everywhere slower).  Up to 256 bytes 64 x 4, one receiver's stores per wave (16 x 16:
// P = 1000 86, but 2500 422).  The next step's lookups before this one's payload: no difference; but its sizes alone (AHEAD) let a wave
// pass over a step in which nothing is sent without its displacements, 16 bytes a pair: FFT, P = 8192 1461 / 1382, P = 3000 221 / 215, others
// the same, up to 16 bytes, P = 3000, where registers count, 170 / 175.
// ------------------------------------------------------------------------------------------
// the tile of one workgroup and step: senders side by side, and blocks a lane finds (of neighbouring receivers)
struct PairShape { int senders, sets; };
constexpr PairShape pair_shape(int lpb, bool stream) { return lpb == 1 ? PairShape{32, 4} : PairShape{lpb == 16 ? 64 : stream ? 8 : 16, 1}; }
constexpr int pair_ranks(PairShape s) { return 4 * (kWave / s.senders) * s.sets; }      // receivers of a tile
template <int LPB, int STREAM>
__global__ void __launch_bounds__(256) k_hop_pairs(const DirectArgs a) {
    constexpr PairShape SH = pair_shape(LPB, STREAM != 0);
    constexpr int SEND = SH.senders, SETS = SH.sets;
    __shared__ ShortLds<LPB> lds;
    const ResolveArgs& r = a.r;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int P = r.P;
    const int p0 = blockIdx.y * pair_ranks(SH) + (wv * (kWave / SEND) + lane / SEND) * SETS;
    const int sub = lane & (SEND - 1);
    unsigned int sum_b[SETS], sum_c[SETS];
#pragma unroll
    for (int u = 0; u < SETS; ++u) sum_b[u] = sum_c[u] = 0;
    const int first = blockIdx.x * a.iters * SEND, last = min(P, first + a.iters * SEND);
    constexpr bool AHEAD = LPB > 1;
    int next[SETS];                                      // AHEAD: the bytes of the next step's blocks
#pragma unroll
    for (int u = 0; u < SETS; ++u)
        if (AHEAD) next[u] = r.recvcounts[(size_t)min(p0 + u, P - 1) * P + min(first + sub, P - 1)];
    for (int q0 = first; q0 < last; q0 += SEND) {
        const int q = min(q0 + sub, P - 1);
        int n[SETS];
        long long va[SETS], vc[SETS];
        if (AHEAD) {
            bool some = q0 == first;                     // (the first step does not wait for its sizes)
#pragma unroll
            for (int u = 0; u < SETS; ++u) {
                n[u] = next[u];
                next[u] = r.recvcounts[(size_t)min(p0 + u, P - 1) * P + min(q0 + SEND + sub, last - 1)];
                if (q0 != first) some = some || n[u] > 0;
            }
            if (!__ballot(some)) continue;
        }
#pragma unroll
        for (int u = 0; u < SETS; ++u) {
            const int p = min(p0 + u, P - 1);
            if (!AHEAD) n[u] = r.recvcounts[(size_t)p * P + q];
            va[u] = r.sdispls[(size_t)q * P + p];
            vc[u] = r.rdispls[(size_t)p * P + q];
        }
        unsigned long long src[SETS], dst[SETS];
#pragma unroll
        for (int u = 0; u < SETS; ++u) {
            if (q0 + sub >= last || p0 + u >= P) n[u] = 0;
            n[u] = min(n[u], 16 * LPB);                  // validation has bounded it: nothing is cut here
            src[u] = (unsigned long long)r.S + (unsigned long long)va[u];
            dst[u] = (unsigned long long)r.R + (unsigned long long)vc[u];
            if (q0 + sub != p0 + u) {                        // (the own block is no part of the phase)
                sum_b[u] += (unsigned int)n[u];
                sum_c[u] += n[u] > 0 ? ((unsigned int)(dst[u] & 15ull) + (unsigned int)n[u] + 15u) >> 4 : 0u;
            }
        }
        move_short<LPB, STREAM>(src, dst, n, (unsigned long long)r.recvcounts, lds);
    }
    if (!a.part) return;
#pragma unroll
    for (int u = 0; u < SETS; ++u) {
#pragma unroll
        for (int d = SEND / 2; d > 0; d >>= 1) { sum_b[u] += __shfl_xor(sum_b[u], d, kWave); sum_c[u] += __shfl_xor(sum_c[u], d, kWave); }
        if (sub == 0 && p0 + u < P) a.part[(size_t)blockIdx.x * P + p0 + u] = make_uint2(sum_b[u], sum_c[u]);
    }
}

// pieces segment s owns, and the dead pieces in front of them
__device__ __forceinline__ int tiled_pieces(unsigned long long a, int n, bool has_prev, unsigned long long e_prev,
                                            int* dead) {
    const unsigned long long e = a + (unsigned long long)n;
    const bool new_run = !has_prev || e_prev != a;
    const unsigned long long last = (e + 15) >> 4;
    const unsigned long long first = new_run ? (a >> 7) << 3 : (a + 15) >> 4;
    *dead = (new_run && has_prev) ? (int)((((e_prev + 127) >> 7) << 3) - ((e_prev + 15) >> 4)) : 0;
    return last > first ? (int)(last - first) : 0;
}

// ------------------------------------------------------------------------------------------
// k_hop_rows: a one-kernel phase of blocks of up to 64 KiB, any alignment and granularity, and any sizes that leave its
// waves balanced (rows_balanced).  One wave takes
// `segs` neighbouring segments of one receiver, 5 to 7 KB of payload: lane i finds block s0 + i (source, destination,
// bytes), a wave scan lays the blocks out as rows of aligned 16-byte pieces of the destination (tiled_pieces), and the
// wave moves 8 pieces per lane at a time.  What the destination-tiled hop needs a resolve pass, a layout pass and unit
// lists for -- 40 bytes of hop arrays per block written and read, and four kernels per phase -- lies in one wave's
// registers and LDS here; the blocks a receiver gets side by side are consecutive segments, so the wave's pieces are one
// run of R or of a class of T.
//   Bound by memory (both sides at 5.3 to 5.7 TB/s at 16 GiB, 6.5 TB/s for a plain copy).  A piece inside its block is one
// 16-byte load at the source's alignment and one aligned streaming store.  The first and the last bytes of a block that
// are no whole piece are stored by 16-byte accesses that begin or end with the block and overlap the whole pieces beside
// them (the same bytes twice), so no piece is put together from two blocks and no store is ever narrower; blocks under
// 16 bytes are stored by the lane that found them.  Byte-granular problems run the same code: accesses at odd addresses
// are as fast as aligned ones (16-byte loads 1 byte off: 5.6 TB/s in a copy, like aligned ones).
//   Measured against the destination-tiled hop and the engine's with their metadata kernels: per call, 16 GiB of 1 KiB
// blocks 6.75 -> 6.35 ms linear and 22.9 -> 22.1 ms at r = 8; 512-byte blocks on average, byte-granular, P = 1000, per
// start 333 -> 210 us; uniform [0, 512] B, P = 2048, r = 46 1.24 -> 0.99 ms; 512-byte blocks, P = 2048, r = 16
// 2.57 -> 2.05 ms; 256-byte blocks, P = 2048 as 64 x 32, r = 16 1.73 -> 1.25 ms.  8 pieces per lane against 4: -4 to -9 %.
// Streaming stores against cached ones: -8 to -15 %; streaming loads
// only where blocks are whole lines (512 bytes: -5 %; 1 KiB blocks at 4-byte alignment: up to +6 %).  Four receivers x
// the same segments per workgroup instead of one receiver: 1 KiB blocks +3 %; rows of workgroups cut so that one XCD sees
// the same senders for all receivers: +1 to +13 %.
// ------------------------------------------------------------------------------------------
constexpr int kRowsPieces = 8;              // pieces per lane and step
constexpr int kRowsBytes = 5200;            // payload of one wave, by the mean block (rows_segs)
constexpr int kRowsLongBytes = 7000;        // of longer blocks
constexpr int kRowsMaxBytes = 1 << 16;      // a wave moves whole blocks: longer ones would leave the others waiting

// Where block (segment s, receiver p) is read from and stored to, and its bytes: from the hop arrays, or from the
// tables, matrices and T positions, all loads from valid addresses and without branches so that they go out together.
// Into T a block takes whole chunks.
template <bool DENSE, bool RESOLVED>
__device__ __forceinline__ void find_block(const DirectArgs& a, int p, int s, unsigned long long& src, unsigned long long& dst, int& n,
                                           int& exact, bool& final) {
    const ResolveArgs& r = a.r;
    const unsigned long long tb = (unsigned long long)a.T;
    bool in_s;
    if (RESOLVED) {
        const size_t o = (size_t)p * r.hop.ld + s;
        const unsigned long long hs = r.hop.src[o], hd = r.hop.dst[o];
        n = r.hop.size[o];
        in_s = !(hs & kHopInT);
        final = !(hd & kHopInT);
        src = (hs & ~(kHopInT | kHopFill)) + (in_s ? 0ull : tb);
        dst = (hd & ~(kHopInT | kHopFill)) + (final ? 0ull : tb);
        exact = n;
    } else {
        const int P = r.P, Q = r.Q, N = r.N;
        const int e = r.seg.e[s], dist = r.seg.z[s] * r.rx, ssrc = r.seg.src[s], sdst = r.seg.dst[s];
        const int sph = DENSE ? r.seg.srcph[s] : 0, sseg = DENSE ? r.seg.srcseg[s] : 0, scl = DENSE ? r.seg.scls[s] : 0, dcl = DENSE ? r.seg.dcls[s] : 0;
        in_s = ssrc < 0;
        final = sdst < 0;
        int j, l, pn, pg, qn, qg;
        split_slot_index(e, Q, N, j, l);
        split_slot_index(p, Q, N, pn, pg);
        const int q = partner_up(pn, pg, Q, N, r.dim, dist);
        split_slot_index(q, Q, N, qn, qg);
        int dn = qn - j; if (dn < 0) dn += N;
        int dg = qg - l; if (dg < 0) dg += Q;
        int sn = pn + j; if (sn >= N) sn -= N;
        int sg = pg + l; if (sg >= Q) sg -= Q;
        const size_t at_s = (size_t)q * P + dn * Q + dg, at_r = (size_t)p * P + sn * Q + sg;
        n = *(final ? r.recvcounts + at_r : block_bytes(r.sendcounts, r.recvcounts, in_s && r.near_s, pn, pg, j, l, P, Q, N, r.dim, r.rx1));
        exact = n;
        if (!final) n = (n + 15) & ~15;
        if (DENSE) {
            const int64_t* tbase = reinterpret_cast<const int64_t*>(r.x.tbase);
            const long long va = *(in_s ? r.sdispls + at_s : tbase + (size_t)scl * P + q);
            const long long vc = *(final ? r.rdispls + at_r : tbase + (size_t)dcl * P + p);
            const int vb = *(in_s ? r.seg.e : r.x.tpos + ((size_t)sph * P + q) * P + sseg);
            const int vd = *(final ? r.seg.e : r.x.tpos + ((size_t)r.x.phase * P + p) * P + s);
            src = in_s ? (unsigned long long)r.S + va : tb + ((unsigned long long)(va + vb) << 4);
            dst = final ? (unsigned long long)r.R + vc : tb + ((unsigned long long)(vc + vd) << 4);
        } else {
            const long long va = *(in_s ? r.sdispls + at_s : r.sdispls);
            const long long vc = *(final ? r.rdispls + at_r : r.rdispls);
            src = in_s ? (unsigned long long)r.S + va : tb + (unsigned long long)(((long long)q * r.slots + ssrc) * r.slot_bytes);
            dst = final ? (unsigned long long)r.R + vc : tb + (unsigned long long)(((long long)p * r.slots + sdst) * r.slot_bytes);
        }
    }
    // whole chunks are read past the block's end, but never past the part of S that holds blocks
    if (in_s && n > 0 && src + (unsigned long long)n > a.user_limit) n = (int)(a.user_limit - src);
}

// LINES: every block is whole 128-byte lines (streaming loads)
template <bool LINES, bool DENSE, bool RESOLVED>
__global__ void __launch_bounds__(256) k_hop_rows(const DirectArgs a) {
    constexpr int CPL = kRowsPieces;
    __shared__ int s_pre[4][kWave], s_off0[4][kWave], s_n[4][kWave];
    __shared__ unsigned long long s_src[4][kWave], s_dst[4][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int P = a.r.P;
    if ((int)blockIdx.y < a.own) {
        const int own = blockIdx.y * gridDim.x + blockIdx.x;
        if (own < P) own_block(a.r.S, a.r.sendcounts, a.r.sdispls, a.r.R, a.r.rdispls, P, own);
        return;
    }
    const int p = blockIdx.y - a.own;
    const int grp = blockIdx.x * 4 + wv;
    const int s0 = a.seg_lo + grp * a.segs;
    if (s0 >= a.seg_hi) return;                          // no barrier below: a wave may leave alone
    const bool in = lane < a.segs && s0 + lane < a.seg_hi;
    unsigned long long src, dst;
    int n, exact;
    bool final;
    find_block<DENSE, RESOLVED>(a, p, min(s0 + min(lane, a.segs - 1), a.seg_hi - 1), src, dst, n, exact, final);
    if (!in || n < 0) n = exact = 0;
    if (!RESOLVED && a.part) {
        unsigned int b = (unsigned int)exact, c = n > 0 ? ((final ? (unsigned int)(dst & 15ull) : 0u) + (unsigned int)exact + 15u) >> 4 : 0u;
#pragma unroll
        for (int d = kWave / 2; d > 0; d >>= 1) { b += __shfl_xor(b, d, kWave); c += __shfl_xor(c, d, kWave); }
        if (lane == 0) a.part[(size_t)grp * P + p] = make_uint2(b, c);
    }
    // ---- the wave's blocks as rows of aligned 16-byte pieces of the destination (tiled_pieces); the part of a block
    // in front of its first whole piece is its head
    unsigned long long e_prev = __shfl_up(dst + (unsigned long long)n, 1, kWave);
    int dead;
    const int own = tiled_pieces(dst, n, lane > 0, e_prev, &dead);
    const bool new_run = lane == 0 || e_prev != dst;
    const int cnt = in ? dead + own : 0;
    const int incl = wave_incl_scan(cnt);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    s_pre[wv][lane] = incl - cnt;
    s_off0[wv][lane] = (new_run ? -(int)((unsigned int)dst & 127u) : (int)((0u - (unsigned int)dst) & 15u)) - (dead << 4);
    s_n[wv][lane] = n; s_src[wv][lane] = src; s_dst[wv][lane] = dst;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const unsigned long long dummy = (unsigned long long)a.r.seg.e;
    // ---- heads, and blocks of fewer than 16 bytes, by the lane that found the block
    const bool head = n >= 16 && (dst & 15ull);
    const v4u hv = load_global<v4u_any>(head ? src : dummy);
    const int ns = n < 16 ? n : 0;
    const bool any_short = __ballot(ns > 0) != 0;
    if (any_short) short_store(dst, src, ns, short_load(src, ns, dummy));
    bool stored = false;
    int top = 1;
    while (2 * top < a.segs) top *= 2;
    for (int base = 0; base < total; base += kWave * CPL) {
        int lo[CPL];
#pragma unroll
        for (int k = 0; k < CPL; ++k) lo[k] = 0;
        for (int step = top; step > 0; step >>= 1) {
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const int c = base + k * kWave + lane;
                if (s_pre[wv][lo[k] + step] <= c) lo[k] += step;      // entries behind the last block hold the total
            }
        }
        v4u v[CPL];
        unsigned long long d[CPL];
        bool act[CPL];
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int c = base + k * kWave + lane;
            const int nb = s_n[wv][lo[k]];
            const int off = s_off0[wv][lo[k]] + ((c - s_pre[wv][lo[k]]) << 4);
            act[k] = off >= 0 && off < nb && nb >= 16;
            const int o = min(off, nb - 16);             // the last piece ends with the block
            const unsigned long long sa = s_src[wv][lo[k]] + (unsigned long long)(long long)o;
            d[k] = s_dst[wv][lo[k]] + (unsigned long long)(long long)o;
            const TUNA_GLOBAL v4u_any* from = (const TUNA_GLOBAL v4u_any*)(act[k] ? sa : dummy);
            v[k] = LINES ? __builtin_nontemporal_load(from) : *from;
        }
        if (!stored) {
            stored = true;
            if (head) store_global<v4u_any>(dst, hv);
        }
#pragma unroll
        for (int k = 0; k < CPL; ++k)
            if (act[k]) __builtin_nontemporal_store(v[k], (TUNA_GLOBAL v4u_any*)d[k]);
    }
}

// ------------------------------------------------------------------------------------------
// k_long_units, k_hop_long: a one-kernel phase of long blocks (long_blocks).  k_long_units cuts every block at the 128-byte
// lines of its destination into units of 4 KiB, each written down as where it is read, where it is stored and how long it
// is; k_hop_long moves one unit per wave and looks nothing else up before its payload.  The units are in no particular
// order: a workgroup takes room in the list for its own, so one launch per phase is all the metadata there is.
//   Bound by memory.  What decides is how compact the part of memory is that is under way at one time: a plain copy of 1.8
// GiB by workgroups of four waves runs at 6.4 TB/s with 1 KiB per wave, 6.2 with 4 and 5.5 with 8; workgroups of one wave
// reach 6.35 with 4 KiB and 6.3 with 8 KiB if only 16 and 8 of them are resident, and lose 5 to 10 % with 32 (the units
// of 8 KiB of k_copy_tiled: 5.4).  Hence one wave per workgroup, 4 KiB, 10 resident (kLongResident, held there by unused
// LDS; 60 ranks, up to 1 MiB, radix 2 and linear, us per call: 8 resident 1954 / 682, 10 1940 / 683, 12 1980 / 695, 16 2037 /
// 695, 20 2087 / 698; 8 KiB, 6 resident 1984 / 666, but 200 ranks, 80 KiB 1186 against 1139).  Streaming loads from
// kLongStreamBytes on (683 / 779; 134 MB 90 / 83, 245 MB 125 / 111).
//   Against the engine's and the destination-tiled hop with their metadata kernels: 60 ranks, up to 1 MiB, 786 -> 681 us per
// call (5.3 -> 5.8 TB/s, metadata and validation included), 708 -> 635 per start; 100 ranks, 200 KB, r = 10 1420 -> 1248; 200 ranks, byte-granular up to 150 KB
// 1374 -> 1060 per start; 20 ranks, up to 200 KB (40 MB) 79-94 -> 56.
// ------------------------------------------------------------------------------------------
constexpr int kLongPieces = 4;
constexpr int kLongUnit = kWave * 16 * kLongPieces;          // bytes
// The workgroups take their room in the list one after the other.  (Measured beyond it since, the hops that run there / these: 600 to
// 1024 ranks, 24 to 48 KiB 3.16 / 3.08 ms, 7.9 / 7.2, 19.1 / 17.0 per call, byte-granular 34 KiB, 800 ranks 9.6 / 7.8.)
constexpr int kLongMaxRanks = 512;
constexpr int kLongResident = 10;                            // workgroups per compute unit
constexpr double kLongStreamBytes = 268435456.0;
// in a unit's y: it is not the first of its block; in either: an offset into T, which a plan has not got yet
constexpr unsigned long long kLongAddress = (1ull << 48) - 1, kLongInside = 1ull << 62, kLongInT = 1ull << 63;
struct LongArgs {
    DirectArgs d;
    ulonglong2* units;      // x: source; y: destination, bytes << 48; kLongInside, kLongInT
    unsigned int* count;    // starts at zero
    unsigned long long* bytes;          // of the phase (Status; null: not wanted)
    unsigned long long* chunks;
    int own;                // 1: the ranks' own blocks too
};
template <bool DENSE>
__global__ void __launch_bounds__(kScanThreads) k_long_units(const LongArgs a) {
    __shared__ int s_pre[kScanThreads + 1], wsum[kScanThreads / kWave];
    __shared__ unsigned long long s_src[kScanThreads], s_dst[kScanThreads], w_b[kScanThreads / kWave], w_c[kScanThreads / kWave];
    __shared__ int s_n[kScanThreads];
    __shared__ unsigned int s_base;
    const ResolveArgs& r = a.d.r;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int p = blockIdx.y, nseg = r.nseg, all = nseg + a.own;
    unsigned long long bytes = 0, chunks = 0;
    for (int base = 0; base < all; base += kScanThreads) {
        const int s = base + tid;
        unsigned long long src, dst;
        int n, exact;
        bool final;
        find_block<DENSE, false>(a.d, p, min(s, nseg - 1), src, dst, n, exact, final);
        unsigned long long in_t = 0;
        if (s < nseg) {
            if (r.seg.src[s] >= 0) src |= kLongInT;
            if (!final) in_t = kLongInT;
            bytes += (unsigned long long)exact;
            if (exact > 0) chunks += ((final ? (unsigned int)(dst & 15ull) : 0u) + (unsigned int)exact + 15u) >> 4;
        } else if (s < all) {
            const size_t o = (size_t)p * r.P + p;
            exact = r.sendcounts[o];
            src = (unsigned long long)r.S + r.sdispls[o];
            dst = (unsigned long long)r.R + r.rdispls[o];
        } else {
            exact = 0;
        }
        const int cnt = exact > 0 ? (int)(((unsigned int)(dst & 127ull) + (unsigned int)exact + kLongUnit - 1) / kLongUnit) : 0;
        const int incl = wave_incl_scan(cnt);
        if (lane == kWave - 1) wsum[wv] = incl;
        s_src[tid] = src; s_dst[tid] = dst | in_t; s_n[tid] = exact;
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / kWave; ++w) { before += w < wv ? wsum[w] : 0; total += wsum[w]; }
        s_pre[tid] = before + incl - cnt;
        // this workgroup's share of the tile's units
        const int per = (total + gridDim.x - 1) / gridDim.x, lo = min(total, per * (int)blockIdx.x), hi = min(total, lo + per);
        if (tid == 0) {
            s_pre[kScanThreads] = total;
            s_base = hi > lo ? atomicAdd(a.count, (unsigned int)(hi - lo)) : 0u;
        }
        __syncthreads();
        for (int u = lo + tid; u < hi; u += kScanThreads) {
            int b = 0;
#pragma unroll
            for (int step = kScanThreads / 2; step > 0; step >>= 1) b += s_pre[b + step] <= u ? step : 0;
            const int k = u - s_pre[b], cut = (int)(s_dst[b] & 127ull);
            const long long from = k ? (long long)k * kLongUnit - cut : 0, to = min((long long)s_n[b], (long long)(k + 1) * kLongUnit - cut);
            a.units[s_base + (unsigned int)(u - lo)] =
                make_ulonglong2(s_src[b] + (unsigned long long)from,
                                (s_dst[b] + (unsigned long long)from) | (unsigned long long)(to - from) << 48 | (k ? kLongInside : 0ull));
        }
        __syncthreads();                                     // the next tile overwrites the LDS
    }
    if (blockIdx.x) return;
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) { bytes += __shfl_xor(bytes, d, kWave); chunks += __shfl_xor(chunks, d, kWave); }
    if (lane == 0) { w_b[wv] = bytes; w_c[wv] = chunks; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kScanThreads / kWave; ++w) { bytes += w_b[w]; chunks += w_c[w]; }
        chunks = (chunks + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks;
        if (bytes && a.bytes) { atomicAdd(a.bytes, bytes); atomicAdd(a.chunks, chunks); }
    }
}

template <bool STREAM>
__global__ void __launch_bounds__(kWave) k_hop_long(const ulonglong2* __restrict__ units, const unsigned int* __restrict__ count,
                                                    unsigned int known, unsigned char* T) {
    const int lane = threadIdx.x;
    const unsigned int total = count ? *count : known;
    for (unsigned int u = blockIdx.x; u < total; u += gridDim.x) {
        const ulonglong2 unit = units[u];
        const unsigned long long src = (unit.x & ~kLongInT) + (unit.x & kLongInT ? (unsigned long long)T : 0ull);
        const unsigned long long dst = (unit.y & kLongAddress) + (unit.y & kLongInT ? (unsigned long long)T : 0ull);
        const int n = (int)(unit.y >> 48) & (2 * kLongUnit - 1), head = (int)((0u - (unsigned int)dst) & 15u);
        v4u v[kLongPieces];
        if (n == kLongUnit && head == 0) {
#pragma unroll
            for (int k = 0; k < kLongPieces; ++k) {
                const TUNA_GLOBAL v4u_any* from = (const TUNA_GLOBAL v4u_any*)(src + (unsigned int)((k * kWave + lane) * 16));
                v[k] = STREAM ? __builtin_nontemporal_load(from) : *from;
            }
#pragma unroll
            for (int k = 0; k < kLongPieces; ++k)
                __builtin_nontemporal_store(v[k], (TUNA_GLOBAL v4u*)(dst + (unsigned int)((k * kWave + lane) * 16)));
        } else if (n >= 16 || (unit.y & kLongInside)) {
            // the ends of a block: 16 bytes that begin or end with it and overlap the pieces beside them; a unit of fewer
            // than 16 bytes has bytes of its block in front
            if (head && lane == 0) store_global<v4u_any>(dst, load_global<v4u_any>(src));
#pragma unroll
            for (int k = 0; k < kLongPieces; ++k) {
                const int off = head + (k * kWave + lane) * 16;
                const long long o = min(off, n - 16);
                v[k] = load_global<v4u_any>(off < n ? src + (unsigned long long)o : (unsigned long long)units);
            }
#pragma unroll
            for (int k = 0; k < kLongPieces; ++k) {
                const int off = head + (k * kWave + lane) * 16;
                const long long o = min(off, n - 16);
                if (off < n) __builtin_nontemporal_store(v[k], (TUNA_GLOBAL v4u_any*)(dst + (unsigned long long)o));
            }
        } else if (lane == 0) {
            short_store(dst, src, n, short_load(src, n, (unsigned long long)units));
        }
    }
}

// k_phase_sums: the partial sums of the phases that ran as k_hop_direct or k_hop_rows, rows[x] rows of P entries for
// phase x, into the status block: payload bytes, and staged chunks with every receiver's share rounded up to a line
// as the staging layouts round it.  Four threads per receiver, grid (ceil(P / 64), phases); k_validate_finish cleared
// the totals.  (Up to 512 ranks they mostly come from the counts instead, before the phases run: launch_early.)
struct PhaseParts { const uint2* part[64]; int rows[64]; };
__global__ void __launch_bounds__(256) k_phase_sums(PhaseParts parts, int P, Status* __restrict__ st) {
    __shared__ unsigned long long s_b[4][kWave], s_c[4][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int p = blockIdx.x * kWave + lane, x = blockIdx.y;
    const uint2* part = parts.part[x];
    const int rows = parts.rows[x];
    unsigned long long b = 0, c = 0;
    if (p < P) {
#pragma unroll 8
        for (int i = wv; i < rows; i += 4) { const uint2 v = part[(size_t)i * P + p]; b += v.x; c += v.y; }
    }
    s_b[wv][lane] = b; s_c[wv][lane] = c;
    __syncthreads();
    if (wv) return;
    b += s_b[1][lane] + s_b[2][lane] + s_b[3][lane];
    c += s_c[1][lane] + s_c[2][lane] + s_c[3][lane];
    c = (c + kRankAlignChunks - 1) / kRankAlignChunks * kRankAlignChunks;
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) { b += __shfl_xor(b, d, kWave); c += __shfl_xor(c, d, kWave); }
    if (lane == 0 && b) { atomicAdd(&st->phase_bytes[x], b); atomicAdd(&st->phase_chunks[x], c); }
}

// Compiled for 8 waves per SIMD (a workgroup is one wave per SIMD).  The host lowers the number of
// resident workgroups per launch where fewer are faster by asking for unused dynamic LDS.  Unpack
// keeps its payload in registers across the address resolution; left alone the compiler then takes
// 84 registers (5 waves), held to 8 waves it needs 64 and spills nothing (byte-granular calls excepted).
// The one-kernel variant needs 62 to 72 registers by itself.  Where it fits into 64 without spilling
// (4-byte granular, exact-size T) it is held to 8 waves too: scheduled for occupancy, gathers of many
// short pieces run 6 % faster (measured at r = P on 16 GiB); the variants that would spill are left alone.
template <int MODE, int GRAN, bool DENSE>
__global__ void __launch_bounds__(kCopyThreads) __attribute__((amdgpu_waves_per_eu(((MODE == kUnpack && GRAN >= 4) || (MODE == kFused && GRAN == 4 && DENSE)) ? 8 : 1, 8)))
k_copy(const CopyArgs a) {
    __shared__ int s_pre[kCopyThreads / kWave][kWave];
    __shared__ int s_size[kCopyThreads / kWave][kWave];
    __shared__ unsigned long long s_addr[kCopyThreads / kWave][kWave];
    __shared__ unsigned long long s_addr2[MODE == kFused ? kCopyThreads / kWave : 1][kWave];
    __shared__ int s_flag[kCopyThreads / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int unit = blockIdx.x * (kCopyThreads / kWave) + wv;
    if (a.batch_rows) {
        // the batch's chunks [lo, hi) of rank blockIdx.y lie in its units lo / 256 .. (hi - 1) / 256
        const int* brow = a.L.pre + (size_t)blockIdx.y * a.L.ld;
        const int lo = brow[a.seg_lo], hi = brow[a.seg_hi];
        const int u = lo / kUnitChunks + unit;
        if (hi <= lo || (long long)u * kUnitChunks >= hi) return;
        unit = a.L.unit_base[blockIdx.y] + u;
    } else if (unit >= *a.L.n_units) {
        return;                                  // no barrier below: a wave may leave alone
    }
    const int4 ud = a.L.units[unit];
    const int p = __builtin_amdgcn_readfirstlane(ud.x);
    int sw = __builtin_amdgcn_readfirstlane(ud.y);
    const int c0 = __builtin_amdgcn_readfirstlane(ud.z);
    const int cend = c0 + __builtin_amdgcn_readfirstlane(ud.w);
    const int n = p / a.Q, g = p - n * a.Q;
    const int* prow = a.L.pre + (size_t)p * a.L.ld;
    v4u* stage = MODE == kFused ? nullptr : a.stage + a.L.rank_base[p];
    int* wpre = s_pre[wv];
    int* wsize = s_size[wv];
    unsigned long long* waddr = s_addr[wv];
    unsigned long long* waddr2 = s_addr2[MODE == kFused ? wv : 0];
    int* wflag = s_flag[wv];

    // batch of rounds: the rank's chunks [blo, bhi) belong to this launch
    int blo = 0, bhi = INT_MAX;
    if (a.seg_hi - a.seg_lo < a.nseg) {
        blo = prow[a.seg_lo];
        bhi = prow[a.seg_hi];
        if (c0 >= bhi || cend <= blo) return;
    }
    int c[kChunksPerLane];
    bool pend[kChunksPerLane];
#pragma unroll
    for (int k = 0; k < kChunksPerLane; ++k) {
        c[k] = c0 + k * kWave + lane;
        pend[k] = c[k] < cend && c[k] >= blo && c[k] < bhi;
    }
    for (;;) {
        // ---- window: segments sw .. sw+63, one per lane --------------------------------------
        const int s = sw + lane;
        int pre_i, pre_w;                            // pre_w is wave-uniform: the first prefix of the next window
        // table fields this mode needs, fetched together with the prefix
        int se = 0, sz_ = 0, ssrc = -1, sdst = -1, sph = -1, scl = -1;
        unsigned long long addr = 0, addr2 = 0;
        int size = 0, flag = 0;
        if (MODE == kFused) {
            // One-kernel phases: source, destination and size of every block were resolved by k_resolve_hop.
            // Every lane loads from an index clamped into range instead of under a branch, so that the
            // loads sit in one basic block and go out back to back.
            const int s_tab = min(s, a.nseg - 1);
            const size_t hi_ = (size_t)p * a.hop.ld + s_tab;
            const int pre_raw = prow[min(s, a.nseg)];
            const int pre_w_raw = prow[min(sw + kWave, a.nseg)];
            // A unit of 256 chunks seldom overlaps more than a few blocks: the first kHopLanes lanes fetch
            // their entries at once, together with the prefix (the condition depends on no loaded value);
            // the others only when the prefix shows that the unit reaches that far (many tiny blocks).
            const bool early = lane < kHopLanes;
            unsigned long long hs_ = 0, hd_ = 0;
            if (early) { hs_ = a.hop.src[hi_]; hd_ = a.hop.dst[hi_]; size = a.hop.size[hi_]; }
            pre_i = s <= a.nseg ? pre_raw : INT_MAX;
            pre_w = sw + kWave <= a.nseg ? pre_w_raw : INT_MAX;
            const int reach = __popcll(__ballot(pre_i < cend));
            if (reach > kHopLanes) {
                if (!early && lane < reach) { hs_ = a.hop.src[hi_]; hd_ = a.hop.dst[hi_]; size = a.hop.size[hi_]; }
            }
            const unsigned long long tb = (unsigned long long)a.T;
            addr = (hs_ & ~(kHopInT | kHopFill)) + ((hs_ & kHopInT) ? tb : 0ull);
            addr2 = (hd_ & ~(kHopInT | kHopFill)) + ((hd_ & kHopInT) ? tb : 0ull);
            // chunks are cut at the destination's 16-byte boundaries: `head` bytes of the first chunk lie
            // before the block (0 in T, where blocks start on chunk or line boundaries)
            flag = (int)(addr2 & 15ull) | ((hs_ & kHopInT) ? kFlagSrcT : 0) | ((hd_ & kHopFill) ? kFlagFill : 0);
        } else {
            pre_i = s <= a.nseg ? prow[s] : INT_MAX;
            pre_w = sw + kWave <= a.nseg ? prow[sw + kWave] : INT_MAX;
        }
        int pre_n = __shfl_down(pre_i, 1, kWave);
        if (lane == kWave - 1) pre_n = pre_w;
        if (MODE != kFused && s < a.nseg) {
            if (MODE != kExchange) se = a.seg.e[s];
            if (MODE == kExchange) sz_ = a.seg.z[s];
            if (MODE == kPack) {
                ssrc = a.seg.src[s];
                if (DENSE) { sph = a.seg.srcph[s]; scl = a.seg.scls[s]; }
            }
            if (MODE == kUnpack) {
                sdst = a.seg.dst[s];
                if (DENSE) scl = a.seg.dcls[s];
            }
        }
        const int wend = pre_w;                      // chunks below wend resolve in this window
        // unpack reads its own staging region: the payload loads of this window need only its bounds and
        // go out before the addresses are resolved, so the two latencies overlap
        bool act[kChunksPerLane];
        v4u v[kChunksPerLane];
#pragma unroll
        for (int k = 0; k < kChunksPerLane; ++k) {
            act[k] = pend[k] && c[k] < wend;
            if (MODE == kUnpack && act[k]) v[k] = __builtin_nontemporal_load(stage + c[k]);
        }
        const bool need = MODE != kFused && s < a.nseg && pre_i < cend && pre_n > pre_i && pre_n > c0;
        if (need) {
            if (MODE == kExchange) {
                const int ps = partner_up(n, g, a.Q, a.N, a.dim, sz_ * a.rx);
                addr = (unsigned long long)(a.stage_src + a.Ls.rank_base[ps] + a.Ls.pre[(size_t)ps * a.Ls.ld + s]);
                size = (pre_n - pre_i) << 4;
            } else {
                // `size` = bytes of the block the destination may receive.  Staging and T slots are
                // padded to whole chunks (lines), so they take whole chunks; a store into R must end
                // exactly with the block.  A load may always run up to 15 bytes past a block's end in
                // T or staging; in S only while it stays inside the part of S that holds blocks.
                size = (pre_n - pre_i) << 4;
                int bj, bl;
                split_slot_index(se, a.Q, a.N, bj, bl);
                if (MODE == kPack) {
                    if (DENSE && ssrc >= 0)
                        addr = exact_t_src(a.T, a.x, a.P, sph, p, se, scl);
                    else
                        addr = block_address(ssrc, false, p, n, g, bj, bl, a.P, a.Q, a.N, a.user, a.displs, a.T,
                                             a.slots, a.slot_bytes);
                    if (ssrc >= 0) flag |= kFlagSrcT;
                }
                if (MODE == kUnpack) {
                    // a final block's size is the receiver's own recvcounts entry (validated equal to
                    // the sender's count), read next to its displacement
                    if (DENSE && sdst >= 0)           // exact-size T: blocks lie back to back, nothing to fill
                        addr = exact_t_dst(a.T, a.x, a.P, p, s, scl);
                    else
                        addr = block_address(sdst, true, p, n, g, bj, bl, a.P, a.Q, a.N, a.user, a.displs, a.T,
                                             a.slots, a.slot_bytes, a.counts, &size);
                    if (!DENSE && sdst >= 0) flag |= kFlagFill; // T-bound: the tail lane completes the 128-byte line
                }
            }
        }
        wpre[lane] = pre_i;
        wsize[lane] = size;
        wflag[lane] = flag;
        waddr[lane] = addr;
        if (MODE == kFused) waddr2[lane] = addr2;
        // the window is private to this wave; its LDS writes are ordered before the reads below
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // entries that can hold a chunk of this unit: the leading lanes with pre_i < cend
        const int nlive = __popcll(__ballot(pre_i < cend));
        int steps = 0;
        while ((1 << steps) < nlive) ++steps;

        unsigned long long oa[kChunksPerLane], oa2[kChunksPerLane];
        int nb[kChunksPerLane], fill[kChunksPerLane];
        // The four searches of a lane advance together, without branches: every step is four independent
        // LDS reads and one wait instead of a dependent chain per chunk.  Lanes without a chunk search
        // for whatever c[k] holds; their result is masked out below.
        int lo[kChunksPerLane], hi[kChunksPerLane];  // wpre[lo] <= c < wpre[hi] (hi == nlive: sentinel)
#pragma unroll
        for (int k = 0; k < kChunksPerLane; ++k) { lo[k] = 0; hi[k] = nlive; }
        for (int it = 0; it < steps; ++it) {
#pragma unroll
            for (int k = 0; k < kChunksPerLane; ++k) {
                const int mid = (lo[k] + hi[k]) >> 1;
                const bool up = wpre[mid] <= c[k];
                const bool move = mid > lo[k];
                lo[k] = (move && up) ? mid : lo[k];
                hi[k] = (move && !up) ? mid : hi[k];
            }
        }
#pragma unroll
        for (int k = 0; k < kChunksPerLane; ++k) {
            const int lim = wsize[lo[k]];
            const int fl = wflag[lo[k]];
            int off = (c[k] - wpre[lo[k]]) << 4;     // first byte of the chunk, relative to the block
            int end = off + 16;
            if (MODE == kFused) {                     // chunk grid anchored at the destination line
                const int h = fl & 15;
                end = off + 16 - h;
                off = max(off - h, 0);
            }
            const unsigned long long src = waddr[lo[k]] + (unsigned long long)(long long)off;
            oa[k] = act[k] ? src : 0ull;
            if (MODE == kFused) oa2[k] = act[k] ? waddr2[lo[k]] + (unsigned long long)(long long)off : 0ull;
            else oa2[k] = 0;
            nb[k] = act[k] ? min(end, lim) - off : 0;
            // last chunk of a T-bound block in a slot: number of further chunks up to the 128-byte line end
            fill[k] = (!DENSE && act[k] && (fl & kFlagFill) && (end >= lim)) ? ((128 - (end & 127)) & 127) >> 4 : 0;
            pend[k] = pend[k] && !act[k];
            // Rare: a whole-chunk load from S is safe only inside the part of S that holds blocks.  The
            // last few bytes of S are loaded exactly and stored at once; the chunk then takes no part in
            // the batched loads and stores below (and none of its state stays live across them).
            if ((MODE == kPack || MODE == kFused) && act[k] && !(fl & kFlagSrcT) && src + 16 > a.user_limit) {
                const int ns = (int)min((unsigned long long)nb[k], a.user_limit - src);
                const v4u t = load_block_chunk<GRAN>(reinterpret_cast<const unsigned char*>(src), min(ns, 15));
                if (MODE == kPack) {
                    __builtin_nontemporal_store(t, stage + c[k]);
                } else {
                    unsigned char* dst = reinterpret_cast<unsigned char*>(oa2[k]);
                    store_block_chunk<GRAN>(dst, t, min(ns, 15));
                    for (int f = 1; f <= fill[k]; ++f) *reinterpret_cast<v4u*>(dst + 16 * f) = t;
                }
                act[k] = false;
                fill[k] = 0;
            }
        }
        // ---- whole-chunk loads, all in flight before the first store --------------------------
#pragma unroll
        for (int k = 0; k < kChunksPerLane; ++k) {
            if (MODE != kUnpack && act[k]) {
                if (MODE == kExchange) v[k] = *reinterpret_cast<const v4u*>(oa[k]);   // neighbours share its edge lines
                // blocks that are whole 128-byte lines share no line with a neighbour: streaming loads
                // (measured on 256-byte blocks: pack +7 to +19 %, one-kernel phases +3 to +6 %; with blocks
                // that share their edge lines they lose up to 15 %)
                else if (GRAN == 128) v[k] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(oa[k]));
                else __builtin_memcpy(&v[k], reinterpret_cast<const unsigned char*>(oa[k]), 16);
            }
        }
        // ---- stores: whole chunks into staging and T, exact bytes into R -------------------------
#pragma unroll
        for (int k = 0; k < kChunksPerLane; ++k) {
            if (act[k]) {
                if (MODE == kUnpack || MODE == kFused) {
                    unsigned char* dst = reinterpret_cast<unsigned char*>(MODE == kFused ? oa2[k] : oa[k]);
                    // with exact-size T whole chunks stream into R and into T (measured: +3 to +9 %);
                    // slots of M bytes are written through the cache, where the fill completes their lines,
                    // and telling the two apart per chunk costs more registers than it gains.  Byte-granular
                    // calls keep plain stores: the address may have any alignment.
                    if (DENSE && GRAN >= 4 && nb[k] >= 16) {
                        typedef v4u v4u_word_aligned __attribute__((aligned(4)));
                        __builtin_nontemporal_store(v[k], reinterpret_cast<v4u_word_aligned*>(dst));
                    } else {
                        store_block_chunk<GRAN>(dst, v[k], nb[k]);
                    }
                } else {
                    __builtin_nontemporal_store(v[k], stage + c[k]);
                }
            }
        }
        // ---- line fill: after the last chunk of a T-bound block the rest of its 128-byte line is
        // written too (content is don't-care), so that T only ever sees whole-line writes.  One
        // store instruction per block tail: lanes 0..f-1 write the f missing chunks.
        if (!DENSE && (MODE == kUnpack || MODE == kFused)) {
#pragma unroll
            for (int k = 0; k < kChunksPerLane; ++k) {
                const unsigned long long dsta = MODE == kFused ? oa2[k] : oa[k];
                unsigned long long m = __ballot(act[k] && fill[k] > 0);
                while (m) {
                    const int leader = __ffsll((long long)m) - 1;
                    m &= m - 1;
                    const unsigned int lo32 = __builtin_amdgcn_readlane((unsigned int)dsta, leader);
                    const unsigned int hi32 = __builtin_amdgcn_readlane((unsigned int)(dsta >> 32), leader);
                    const int f = __builtin_amdgcn_readlane(fill[k], leader);
                    if (lane < f) {
                        const v4u zero = {0u, 0u, 0u, 0u};
                        unsigned char* base = reinterpret_cast<unsigned char*>(((unsigned long long)hi32 << 32) | lo32);
                        *reinterpret_cast<v4u*>(base + 16 * (lane + 1)) = zero;
                    }
                }
            }
        }
        if (wend >= cend) break;
        sw += kWave;
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------------------------------------------
// The destination-tiled hop.  What a rank receives in a one-kernel phase lands in a few long contiguous
// runs: the final blocks in R (Algorithm "TuNA", lines 16-18) when the receive regions are dense -- every
// rank's blocks back to back in source order, the usual layout --, the others in exact-size T, where
// the blocks of a class lie back to back.  The copy engine cuts such a phase into 16-byte chunks per
// block; a block that does not start on a 16-byte boundary shares a chunk with its predecessor, the
// chunk count drifts against the addresses, and a wave's 64-lane store never covers whole 128-byte
// lines: measured, streaming stores that begin and end inside lines cost 13 % of the hop's rate
// (blocks of whole lines, destination 4 or 16 bytes off a line: 4.9 and 4.7 TB/s against 5.6 to 5.8
// aligned).  Here the unit of work is the destination itself: a run is cut into its 16-byte pieces
// from the 128-byte line it starts in to the line it ends in, every piece belongs to exactly one lane,
// a piece that holds the end of one block and the start of the next is assembled by that lane from
// both, and every wave store covers eight whole lines.
//
// k_tiled_layout (one workgroup per rank, the scan machinery of k_phase_layout): from the resolved
// destinations and sizes (k_resolve_hop) the number of pieces every segment owns.  Segment s with
// destination a, size n, end E = a + n continues a run when its predecessor in message order ends at a
// (empty blocks lie where they would lie, so they continue runs too); it then owns the pieces from
// ceil(a / 16) to ceil(E / 16) -- the piece that holds its first bytes, if shared, belongs to a
// predecessor.  A segment that starts a run owns the pieces from the start of a's 128-byte line, and
// in front of them come the dead pieces that complete the previous run's last line, so that every run
// starts at a multiple of 8 pieces.  The prefix row has the same form as a chunk prefix row:
// k_layout_base and k_layout_units cut it into wave units of 256 pieces.  The staged chunks of the statistics
// are summed beside it: pieces are not chunks.
// ------------------------------------------------------------------------------------------
struct TiledLayoutArgs {
    HopDev hop;
    int nseg, P;
    LayoutDev Lr;
    int* rank_chunks;                   // [P]: staged chunks of every rank, counted as the chunk scan and k_phase_sums count them
    unsigned long long* rank_bytes;     // [P]: payload bytes every rank receives in the phase; nullptr: already known
};

__global__ void __launch_bounds__(kScanThreads) k_tiled_layout(const TiledLayoutArgs a) {
    __shared__ int wsum[kScanThreads / kWave];
    __shared__ unsigned long long wbytes[kScanThreads / kWave];
    __shared__ int wchunks[kScanThreads / kWave];
    const int p = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const size_t o = (size_t)p * a.hop.ld;
    int* pre_r = a.Lr.pre + (size_t)p * a.Lr.ld;
    int carry = 0, chunks = 0;
    unsigned long long bytes = 0;
    for (int base = 0; base < a.nseg; base += kScanThreads * kScanItems) {
        int cr[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int s = base + scan_item_index(k);
            cr[k] = 0;
            if (s < a.nseg) {
                // a destination in T is an offset with the in-T bit set; T starts on a 256-byte boundary, so the
                // raw values align and follow each other exactly like the addresses they stand for
                const unsigned long long d = a.hop.dst[o + s];
                const int n = a.hop.size[o + s];
                unsigned long long e_prev = 0;
                if (s > 0) e_prev = a.hop.dst[o + s - 1] + (unsigned long long)a.hop.size[o + s - 1];
                int dead;
                const int own = tiled_pieces(d, n, s > 0, e_prev, &dead);
                cr[k] = dead + own;
                bytes += (unsigned long long)n;
                chunks += n > 0 ? ((int)(d & 15ull) + n + 15) >> 4 : 0;
            }
        }
        int run[kScanItems];
        block_scan_batch(cr, run, carry, wsum);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int s = base + scan_item_index(k);
            if (s < a.nseg) pre_r[s] = run[k];
        }
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) { bytes += __shfl_xor(bytes, d, kWave); chunks += __shfl_xor(chunks, d, kWave); }
    __syncthreads();
    if (lane == 0) { wbytes[tid / kWave] = bytes; wchunks[tid / kWave] = chunks; }
    __syncthreads();
    if (tid == 0) {
        unsigned long long t = 0;
        int c = 0;
#pragma unroll
        for (int k = 0; k < kScanThreads / kWave; ++k) { t += wbytes[k]; c += wchunks[k]; }
        if (a.rank_bytes) a.rank_bytes[p] = t;
        a.rank_chunks[p] = c;
        pre_r[a.nseg] = carry; a.Lr.tot[p] = carry;
    }
}

// ------------------------------------------------------------------------------------------
// k_copy_tiled: the payload kernel of the destination-tiled hop.  Work unit = one wavefront x
// 64 CPL consecutive pieces of one rank (k_tiled_layout; CPL = 4, or 8 for a word-granular last phase: what
// a wave spends on its edge pieces does not grow with the unit, measured 4.6 % per start at r = P on the
// 16 GiB workload, while phases without edge pieces lose 2 % with the larger unit); no workgroup barrier.  Lane i of a window loads
// the prefix and the resolved source, destination and size of segment s0 + i and derives the address of
// the segment's first own piece; every lane finds the segment of each of its CPL pieces by the same
// branch-free search as the copy engine.  A piece that lies inside its block is one 16-byte load at
// the source's own alignment and one aligned streaming store.  A piece at a block's edge is put together
// word by word (GRAN = 4: every size and address is a multiple of 4) from its block and the one behind it
// in the run (a walk over the window's entries, and over the hop arrays behind the window, when more blocks
// than that meet in one piece) and stored whole
// when all four words belong to blocks, else word by word (the ends of a run: bytes outside every block
// are never written).  With GRAN = 16 every piece is inside a block or outside all of them.  Blocks bound
// for T take whole chunks; a load never leaves the part of S that holds blocks.
// ------------------------------------------------------------------------------------------
struct TiledCopyArgs {
    LayoutDev L;
    HopDev hop;
    int nseg;
    unsigned char* T;
    unsigned long long user_limit;      // address one past the last byte of S that holds a block
};

template <int GRAN, int CPL>
__global__ void __launch_bounds__(kCopyThreads) k_copy_tiled(const TiledCopyArgs a) {
    __shared__ int s_pre[kCopyThreads / kWave][kWave];
    __shared__ int s_size[kCopyThreads / kWave][kWave];
    __shared__ int s_off0[kCopyThreads / kWave][kWave];
    __shared__ int s_lim[kCopyThreads / kWave][kWave];
    __shared__ unsigned long long s_src[kCopyThreads / kWave][kWave];
    __shared__ unsigned long long s_dst[kCopyThreads / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int unit = blockIdx.x * (kCopyThreads / kWave) + wv;
    if (unit >= *a.L.n_units) return;                // no barrier below: a wave may leave alone
    const int4 ud = a.L.units[unit];
    const int p = __builtin_amdgcn_readfirstlane(ud.x);
    int sw = __builtin_amdgcn_readfirstlane(ud.y);
    const int c0 = __builtin_amdgcn_readfirstlane(ud.z);
    const int cend = c0 + __builtin_amdgcn_readfirstlane(ud.w);
    const int* prow = a.L.pre + (size_t)p * a.L.ld;
    const size_t ho = (size_t)p * a.hop.ld;
    int* wpre = s_pre[wv];
    int* wsize = s_size[wv];
    int* woff0 = s_off0[wv];
    int* wlim = s_lim[wv];
    unsigned long long* wsrc = s_src[wv];
    unsigned long long* wdst = s_dst[wv];
    const unsigned long long tb = (unsigned long long)a.T;
    int c[CPL];
    bool pend[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
        c[k] = c0 + k * kWave + lane;
        pend[k] = c[k] < cend;
    }
    for (;;) {
        // ---- window: segments sw .. sw+63, one per lane; loads from clamped indices.  A unit of 256 pieces seldom
        // overlaps more than a few blocks: the first kHopLanes lanes fetch their entries together with the
        // prefix, the others only when the prefix shows that the unit reaches that far (two entries more than
        // it reaches: the last piece of the unit may hold the first words of the blocks behind it).
        const int s = sw + lane;
        const int s_tab = min(s, a.nseg - 1);
        const int pre_raw = prow[min(s, a.nseg)];
        const int pre_w_raw = prow[min(sw + kWave, a.nseg)];
        const bool early = lane < kHopLanes;
        unsigned long long hs_ = 0, hd_ = 0;
        int size = 0;
        if (early) { hs_ = a.hop.src[ho + s_tab]; hd_ = a.hop.dst[ho + s_tab]; size = a.hop.size[ho + s_tab]; }
        // the end of the block in front of the window, for its first segment
        unsigned long long e_front = 0;
        if (lane == 0 && sw > 0) e_front = a.hop.dst[ho + sw - 1] + (unsigned long long)a.hop.size[ho + sw - 1];
        const int pre_i = s <= a.nseg ? pre_raw : INT_MAX;
        const int pre_w = sw + kWave <= a.nseg ? pre_w_raw : INT_MAX;
        const int nload = min(kWave, max(kHopLanes, __popcll(__ballot(pre_i < cend)) + 2));
        if (nload > kHopLanes) {
            if (!early && lane < nload) { hs_ = a.hop.src[ho + s_tab]; hd_ = a.hop.dst[ho + s_tab]; size = a.hop.size[ho + s_tab]; }
        }
        unsigned long long e_prev = __shfl_up(hd_ + (unsigned long long)size, 1, kWave);
        if (lane == 0) e_prev = e_front;
        // Offset of piece 0 of the segment's row from the block's first byte: a segment that starts a run owns
        // the pieces from its 128-byte line's start, behind the dead pieces that complete the previous run's
        // line; one that continues a run owns them from the first piece that begins inside the block.  Dead
        // pieces and the pieces in front of the block come out with negative offsets and hold none of its bytes.
        int dead;
        (void)tiled_pieces(hd_, size, s_tab > 0, e_prev, &dead);
        const bool new_run = s_tab == 0 || e_prev != hd_;
        const int off0 = (new_run ? -(int)((unsigned int)hd_ & 127u) : (int)((0u - (unsigned int)hd_) & 15u)) - (dead << 4);
        const unsigned long long src_addr = (hs_ & ~(kHopInT | kHopFill)) + ((hs_ & kHopInT) ? tb : 0ull);
        // A block bound for T takes whole chunks: its last piece is loaded whole and may run up to 15 bytes past
        // the block's end.  In T that is padding; in S it is the next block, except at the very end of S: `lim` =
        // the bytes that may be loaded from the block's start on.
        int lim = size;
        if (!(hs_ & kHopInT)) lim = (int)min((unsigned long long)size, a.user_limit > src_addr ? a.user_limit - src_addr : 0ull);
        wpre[lane] = pre_i;
        wsize[lane] = size;
        woff0[lane] = off0;
        wlim[lane] = lim;
        wsrc[lane] = src_addr;
        wdst[lane] = (hd_ & ~(kHopInT | kHopFill)) + ((hd_ & kHopInT) ? tb : 0ull);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int wend = pre_w;                      // pieces below wend resolve in this window
        const int nlive = __popcll(__ballot(pre_i < cend));
        int steps = 0;
        while ((1 << steps) < nlive) ++steps;
        bool act[CPL];
        int lo[CPL], hi[CPL];
#pragma unroll
        for (int k = 0; k < CPL; ++k) { act[k] = pend[k] && c[k] < wend; lo[k] = 0; hi[k] = nlive; }
        for (int it = 0; it < steps; ++it) {
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const int mid = (lo[k] + hi[k]) >> 1;
                const bool up = wpre[mid] <= c[k];
                const bool move = mid > lo[k];
                lo[k] = (move && up) ? mid : lo[k];
                hi[k] = (move && !up) ? mid : hi[k];
            }
        }
        // every piece as a byte offset from its block's start: 32-bit arithmetic from here on
        int off[CPL];
        bool whole[CPL], edge[CPL];
        v4u v[CPL];
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const int idx = lo[k];
            off[k] = woff0[idx] + ((c[k] - wpre[idx]) << 4);
            whole[k] = act[k] && off[k] >= 0 && off[k] + 16 <= wlim[idx];
            edge[k] = act[k] && !whole[k] && off[k] > -16;
            pend[k] = pend[k] && !act[k];
        }
        // ---- loads of the pieces inside their blocks, issued together ----------------------------------------
#pragma unroll
        for (int k = 0; k < CPL; ++k)
            if (whole[k]) __builtin_memcpy(&v[k], reinterpret_cast<const unsigned char*>(wsrc[lo[k]] + (unsigned long long)(long long)off[k]), 16);
        // ---- pieces at block edges: a word lies in the piece's block, in the block behind it, or in none.  The
        // loads go out at once and travel with the ones above; nothing loaded is looked at before the stores.
        // A unit holds a handful of block edges, seldom two in one lane: every lane takes its first edge piece,
        // then its second ..., so that the code below runs once or twice per wave, not once per piece index.
        unsigned int emask = 0;                      // bit 4 k + q: word q of piece k was loaded
        unsigned int raremask = 0;
        if (GRAN < 16) {
            static_assert(CPL <= 8, "emask holds four bits per piece");
            unsigned int todo = 0;
#pragma unroll
            for (int k = 0; k < CPL; ++k) todo |= edge[k] ? 1u << k : 0u;
            while (__ballot(todo != 0)) {
                bool on = todo != 0;
                const int ks = on ? __ffs((int)todo) - 1 : 0;
                todo &= todo - 1;
                int offk = off[0], t = lo[0];
#pragma unroll
                for (int k = 1; k < CPL; ++k) { offk = ks == k ? off[k] : offk; t = ks == k ? lo[k] : t; }
                const int n = wsize[t];
                const int nlim = wlim[t];                    // < n only for the last block of S when it is bound for T
                const bool has_next = sw + t + 1 < a.nseg;
                const bool next_here = has_next && t + 1 < nload;
                const int tn = min(t + 1, kWave - 1);
                const int nn = wsize[tn];
                const bool follows = next_here && wdst[tn] == wdst[t] + (unsigned long long)n;
                const int over = offk + 16 - n;              // bytes of the piece behind this block's end
                // the walk over several blocks is needed when the block behind is not in the window, is empty,
                // or ends inside this piece too
                if (on && over > 0 && has_next && (!next_here || (follows && nn < over && sw + t + 2 < a.nseg))) {
                    raremask |= 1u << ks;
                    on = false;
                }
                const unsigned long long sa = wsrc[t] + (unsigned long long)(long long)offk;
                const unsigned long long sb = wsrc[tn] + (unsigned long long)(long long)(offk - n);
                uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int o = offk + 4 * q, o2 = o - n;
                    const bool mine = o >= 0 && o < n;
                    const bool theirs = follows && o2 >= 0 && o2 < nn;
                    if (on && (mine || theirs)) {
                        if (mine ? o < nlim : o2 < wlim[tn]) w[q] = *reinterpret_cast<const uint32_t*>((mine ? sa : sb) + 4u * q);
                        emask |= 1u << (4 * ks + q);
                    }
                }
#pragma unroll
                for (int kk = 0; kk < CPL; ++kk)
                    if (on && kk == ks) { v[kk][0] = w[0]; v[kk][1] = w[1]; v[kk][2] = w[2]; v[kk][3] = w[3]; }
            }
            // rare: the blocks of a piece reach past the entries the window holds, or several blocks end inside
            // one piece (a row of tiny or empty blocks): a walk over the entries in the window, and over the hop
            // arrays in global memory behind it
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                if (!(raremask & (1u << k))) continue;
                int t = sw + lo[k];
                unsigned long long ta = wdst[lo[k]], te = ta + (unsigned long long)wsize[lo[k]], ts = wsrc[lo[k]];
                long long tl = wlim[lo[k]];                         // bytes of the block that may be loaded
                const unsigned long long d = ta + (unsigned long long)(long long)off[k];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned long long b = d + 4u * q;
                    bool in_run = true;
                    while (b >= te) {                // the word lies behind this block: the next one, if it follows directly
                        ++t;
                        if (t >= a.nseg) { in_run = false; break; }
                        const int wi = t - sw;
                        unsigned long long na, nsa;
                        int nsz;
                        long long nl;
                        if (wi < nload) {            // the window holds the entry
                            na = wdst[wi]; nsa = wsrc[wi]; nsz = wsize[wi]; nl = wlim[wi];
                        } else {
                            const unsigned long long nraw = a.hop.dst[ho + t], nsrc = a.hop.src[ho + t];
                            na = (nraw & ~(kHopInT | kHopFill)) + ((nraw & kHopInT) ? tb : 0ull);
                            nsa = (nsrc & ~(kHopInT | kHopFill)) + ((nsrc & kHopInT) ? tb : 0ull);
                            nsz = a.hop.size[ho + t];
                            nl = nsz;
                            if (!(nsrc & kHopInT)) nl = (long long)min((unsigned long long)nsz, a.user_limit > nsa ? a.user_limit - nsa : 0ull);
                        }
                        if (na != te) { in_run = false; break; }
                        ta = na; te = na + (unsigned long long)nsz; ts = nsa; tl = nl;
                    }
                    if (!in_run) break;              // nothing behind the run's end belongs to a block
                    if (b >= ta) {
                        const unsigned long long o = b - ta;
                        v[k][q] = (long long)o < tl ? *reinterpret_cast<const uint32_t*>(ts + o) : 0u;
                        emask |= 1u << (4 * k + q);
                    }
                }
            }
        }
        // ---- stores: whole pieces and edge pieces with all four words as aligned streaming stores (eight whole
        // lines per wave store), the others word by word (the ends of a run) -----------------------------------
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            if (whole[k] || edge[k]) {
                unsigned char* d = reinterpret_cast<unsigned char*>(wdst[lo[k]] + (unsigned long long)(long long)off[k]);
                const unsigned int em = (emask >> (4 * k)) & 0xfu;
                if (whole[k] || em == 0xfu) {
                    __builtin_nontemporal_store(v[k], reinterpret_cast<v4u*>(d));
                } else {
                    uint32_t* d4 = reinterpret_cast<uint32_t*>(d);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (em & (1u << q)) d4[q] = v[k][q];
                }
            }
        }
        if (wend >= cend) break;
        sw += kWave;
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------------------------------------------
// k_tiny_call: a whole call in one kernel, for problems so small that launches, not bytes, are
// what a call costs (Section "Performance analysis of TuNA": with tiny messages the number of rounds
// decides; here the number of kernel launches does).  One workgroup of 1024 threads does what the
// other kernels do between them, in the same order: the validation pass (counts >= 0, recvcounts ==
// transpose(sendcounts), M, total), the index-only initial rotation (Algorithm "TuNA", lines 4-5), the
// ranks' own blocks, then every digit phase: the metadata exchange (line 14: block sizes travel to the
// receiver's size array) and the hop of every moving block from where its sender holds it (S, or its
// slot of T) to where its receiver keeps it (R at the slot of its source rank, or its slot of T; lines
// 15-20).  T is the paper's B slots of M bytes per rank, laid out twice: a phase reads one copy and
// writes the other (the copy is the parity of a block's hop count, folded into the slot tables of the
// schedule), so no slot is read and written in one phase.  Sixteen lanes move one block at a time;
// workgroup barriers separate the phases.
// What a phase needs besides the payload is read from global memory once, at the start, all loads in
// flight together, and kept in LDS: the rotated sizes, the low 32 bits of both displacement
// matrices and the tables of every phase.  A block's size is looked up where the rotation left it (no
// exchange between the phases).  Where every block of every phase is read from and stored to is then worked out at once, a thread per
// block, and kept in LDS too; T lies there as well where it fits (the device has 160 KB a workgroup), as the 16-byte registers that
// move a block, else in global memory.
// The kernel declines -- writes tiny_done = 0 and moves nothing -- when the counts are invalid, when
// the problem is not tiny after all (payload above kTinyMaxPayload, T above its capacity) or when a
// displacement of a non-empty block does not fit into 32 bits; the host then takes the general path,
// which reports the error or does the work.
// Bound by the instructions of one workgroup and by latency: a call has 15 us of launch and wait, the kernel a round trip for the matrices, one
// for S and R each, and 1 to 2 us per phase.  With 16 lanes that each worked out their block's place, phase by phase, that arithmetic
// was most of the kernel (T in the LDS alone changed nothing).  Us per call, before / now: 16 ranks, up to 256 bytes, r = 2 34.0 /
// 27.7, r = 4 30.9 / 25.8, linear 26.5 / 22.7; 24 ranks, r = 2, up to 60 bytes 50.9 / 40.7; 30 ranks, linear, up to 16 bytes 39.2 / 30.2; 4 x 4
// ranks, up to 100 bytes 37.1 / 28.8.
// Dynamic LDS: tiny_lds_bytes(P, total table entries).
// ------------------------------------------------------------------------------------------
constexpr int kTinyMaxRanks = 40;           // above it every schedule moves more blocks than run_tiny sends here
constexpr int kTinyMaxPhases = 8;
constexpr int kTinyThreads = 1024;
constexpr int kTinyGroups = kTinyThreads / 16;
constexpr unsigned long long kTinyMaxPayload = 1ull << 20;      // bytes
struct TinyPhase {
    const int32_t* e;
    const int32_t* z;
    const int32_t* src;
    const int32_t* dst;
    int nseg, dim, rx, rx1;
};
struct TinyArgs {
    const unsigned char* S;
    const int32_t* sendcounts;
    const int64_t* sdispls;
    unsigned char* R;
    const int32_t* recvcounts;
    const int64_t* rdispls;
    int P, Q, N, nph;
    TinyPhase ph[kTinyMaxPhases];
    unsigned char* T;               // capacity t_capacity bytes
    long long slots;                // T slots per rank (both copies)
    unsigned long long t_capacity;
    int entries;                    // table entries of all phases
    int moving;                     // and blocks, P per entry
    int t_lds;                      // bytes of LDS behind matrices and tables, for T if it fits
    Status* st;                     // the first 64 bytes are written; in pinned host memory, so that the host reads
                                    // them after the stream's synchronisation without a copy of its own
};

// three P x P arrays of 4 bytes (the sizes and two displacement matrices), four ints per table entry and three per block that
// moves, in whole chunks
constexpr size_t tiny_lds_bytes(int P, int table_entries) {
    return (((size_t)3 * P * P + (size_t)4 * table_entries + (size_t)3 * P * table_entries) * 4 + 15) / 16 * 16;
}

// A block of fewer than 16 bytes as one register of 16: the overlapping parts that short_load and short_store work with.
__device__ __forceinline__ v4u short_pack(unsigned long long src, int n, unsigned long long dummy) {
    const ShortBlock b = short_load(src, n, dummy);
    v4u v = {b.x0, b.x1, 0u, 0u};
    if (n >= 8) { v.x = (unsigned int)b.w0; v.y = (unsigned int)(b.w0 >> 32); v.z = (unsigned int)b.w1; v.w = (unsigned int)(b.w1 >> 32); }
    else if (n > 0 && n < 4)
        v.x = load_global<unsigned char>(src) | load_global<unsigned char>(src + (n >> 1)) << 8 | load_global<unsigned char>(src + n - 1) << 16;
    return v;
}
__device__ __forceinline__ void short_unpack(unsigned long long dst, int n, v4u v) {
    if (n >= 8) {
        store_global<u64_any>(dst, (unsigned long long)v.y << 32 | v.x);
        if (n > 8) store_global<u64_any>(dst + n - 8, (unsigned long long)v.w << 32 | v.z);
    } else if (n >= 4) {
        store_global<u32_any>(dst, v.x);
        if (n > 4) store_global<u32_any>(dst + n - 4, v.y);
    } else if (n > 0) {
        store_global<unsigned char>(dst, (unsigned char)v.x);
        store_global<unsigned char>(dst + (n >> 1), (unsigned char)(v.x >> 8));
        store_global<unsigned char>(dst + n - 1, (unsigned char)(v.x >> 16));
    }
}

__global__ void __launch_bounds__(kTinyThreads) k_tiny_call(const TinyArgs a) {
    extern __shared__ __align__(16) int tiny_lds[];
    __shared__ unsigned long long red[kTinyThreads / kWave][4];
    __shared__ int verdict;
    const int P = a.P, Q = a.Q, N = a.N, P2 = P * P;
    int* cur = tiny_lds;                                            // [P][P] sizes by slot index (the rotation's result)
    unsigned int* sd32 = reinterpret_cast<unsigned int*>(cur + P2); // [P][P] sdispls, low 32 bits
    unsigned int* rd32 = sd32 + P2;                                 // [P][P] rdispls, low 32 bits
    int* tab = reinterpret_cast<int*>(rd32 + P2);                   // per phase: e[nseg], z[nseg], src[nseg], dst[nseg]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    constexpr int kWaves = kTinyThreads / kWave;
    // ---- the tables of every phase, four ints per entry: requested first, so that they travel together with the matrices ----
    auto table_entry = [&](int k) {
        for (int x = 0; x < a.nph; ++x) {
            const TinyPhase& ph = a.ph[x];
            if (k < 4 * ph.nseg) {
                const int f = k / ph.nseg, s_ = k - f * ph.nseg;
                return (f == 0 ? ph.e : (f == 1 ? ph.z : (f == 2 ? ph.src : ph.dst))) + s_;
            }
            k -= 4 * ph.nseg;
        }
        return a.sendcounts;                                        // any int that can be read
    };
    const int entry = *table_entry(tid);
    // ---- validation, and the initial rotation (index only) on the way ---------------------------------------
    unsigned int flags = 0, abits = 0;
    int mx = 0;
    unsigned long long bytes = 0, chunks = 0, extent = 0;
    for (int k = tid; k < P2; k += kTinyThreads) {
        const int i = k / P, j = k - i * P;
        int c = a.sendcounts[k];
        const int rc = a.recvcounts[(size_t)j * P + i];
        const int64_t sd = a.sdispls[k], rd = a.rdispls[(size_t)j * P + i];
        if (c < 0) { flags |= 1u; c = 0; }
        if (rc < 0) flags |= 1u;
        else if (rc != c) flags |= 2u;
        abits |= (unsigned int)c | ((unsigned int)sd & 127u) | ((unsigned int)rd & 127u);
        if (c > 0) {
            if (sd < 0 || rd < 0) flags |= 4u;
            else extent = max(extent, (unsigned long long)sd + (unsigned long long)c);
            if (((unsigned long long)sd | (unsigned long long)rd) >> 32) flags |= 8u;      // not an error: beyond this kernel
        }
        mx = max(mx, c);
        bytes += (unsigned long long)c;
        chunks += (unsigned long long)((c + 15) >> 4);
        // rank i = (n, g) holds its block for rank j = (jn, jg) at the slot index of their distance
        const int n = i / Q, g = i - n * Q, jn = j / Q, jg = j - jn * Q;
        int dj = n - jn; if (dj < 0) dj += N;
        int dl = g - jg; if (dl < 0) dl += Q;
        cur[i * P + dj * Q + dl] = c;
        sd32[k] = (unsigned int)sd;
        rd32[j * P + i] = (unsigned int)rd;
    }
    if (tid < 4 * a.entries) tab[tid] = entry;
    for (int k = tid + kTinyThreads; k < 4 * a.entries; k += kTinyThreads) tab[k] = *table_entry(k);
    flags = last_lane<kWave>(flags << 8 | (abits & 127u), 0u, OrOp());
    mx = (int)last_lane<kWave>((unsigned int)mx, 0u, MaxOp());
    bytes = last_lane<kWave>(bytes, 0ull, AddOp());
    chunks = last_lane<kWave>(chunks, 0ull, AddOp());
    extent = last_lane<kWave>(extent, 0ull, MaxOp());
    if (lane == kWave - 1) {
        red[wv][0] = (unsigned long long)flags << 32 | (unsigned int)mx;
        red[wv][1] = bytes; red[wv][2] = chunks; red[wv][3] = extent;
    }
    __syncthreads();
    if (wv == 0) {
        static_assert(kWaves == 16, "a row of lanes");
        const unsigned long long* r = red[lane & (kWaves - 1)];
        const unsigned int fl = last_lane<kWaves>((unsigned int)(r[0] >> 32), 0u, OrOp()), m = last_lane<kWaves>((unsigned int)r[0], 0u, MaxOp());
        const unsigned long long by = last_lane<kWaves>(r[1], 0ull, AddOp()), ch = last_lane<kWaves>(r[2], 0ull, AddOp());
        const unsigned long long ex = last_lane<kWaves>(r[3], 0ull, MaxOp());
        if (lane == kWaves - 1) {
            const long long slot_bytes = ((long long)m + 15) / 16 * 16;
            const unsigned long long t_need = (unsigned long long)P * (unsigned long long)a.slots * (unsigned long long)slot_bytes;
            const bool ok = fl >> 8 == 0 && by <= kTinyMaxPayload && t_need <= a.t_capacity;
            a.st->flags = fl >> 8 & 7u; a.st->align_bits = fl & 127u; a.st->max_count = (int)m; a.st->total_bytes = by; a.st->total_chunks = ch;
            a.st->send_extent = ex; a.st->tiny_done = ok ? 1 : 0;
            verdict = ok ? (int)m : -1;
        }
    }
    __syncthreads();
    if (verdict < 0) return;                             // uniform: declined, nothing has moved
    const long long slot_bytes = ((long long)verdict + 15) / 16 * 16;
    // ---- where every block of every phase is read from, stored to, and its bytes: a thread per block, all phases at once ----
    unsigned int* d_src = reinterpret_cast<unsigned int*>(tab + 4 * a.entries);     // offset into S, or T
    unsigned int* d_dst = d_src + a.moving;                                         // into R, or T
    unsigned int* d_n = d_dst + a.moving;
    constexpr unsigned int kSrcT = 1u << 30, kDstT = 1u << 31;                      // (blocks have no more than kTinyMaxPayload bytes)
    for (int k0 = tid; k0 < a.moving; k0 += kTinyThreads) {
        int x = 0, k = k0, off = 0;
        while (k >= P * a.ph[x].nseg) { k -= P * a.ph[x].nseg; off += 4 * a.ph[x].nseg; ++x; }
        const int nseg = a.ph[x].nseg, dim = a.ph[x].dim, rx = a.ph[x].rx, rx1 = a.ph[x].rx1;
        const int q = k / nseg, s = k - q * nseg;
        const int* t = tab + off + s;
        const int e = t[0], ssrc = t[2 * nseg], sdst = t[3 * nseg];
        int qn, qg, j, l;
        split_slot_index(q, Q, N, qn, qg);
        split_slot_index(e, Q, N, j, l);
        // the block's size: in the rotated sizes of the rank it comes from, the digits up to this phase's away (see
        // block_bytes); no exchange from phase to phase
        int on0 = qn, og0 = qg + l;
        if (dim == 0) og0 = qg + l % rx1;
        else on0 = qn + j % rx1;
        if (og0 >= Q) og0 -= Q;
        if (on0 >= N) on0 -= N;
        const int size = cur[(on0 * Q + og0) * P + e];
        const int sender = partner_up(qn, qg, Q, N, dim, t[nseg] * rx);
        int sn, sg;
        split_slot_index(sender, Q, N, sn, sg);
        int dn = sn - j; if (dn < 0) dn += N;
        int dg = sg - l; if (dg < 0) dg += Q;
        int on = qn + j; if (on >= N) on -= N;
        int og = qg + l; if (og >= Q) og -= Q;
        d_src[k0] = ssrc < 0 ? sd32[sender * P + dn * Q + dg] : (unsigned int)((sender * (int)a.slots + ssrc) * (int)slot_bytes);
        d_dst[k0] = sdst < 0 ? rd32[q * P + on * Q + og] : (unsigned int)((q * (int)a.slots + sdst) * (int)slot_bytes);
        d_n[k0] = (unsigned int)size | (ssrc < 0 ? 0u : kSrcT) | (sdst < 0 ? 0u : kDstT);
    }
    __syncthreads();
    // ---- digit phases; the ranks' own blocks go with the first ----------------------------------------------
    const unsigned long long dummy = (unsigned long long)a.T;       // any 16 bytes that can be read
    v4u* const t_lds = reinterpret_cast<v4u*>(tiny_lds + ((3 * P2 + 4 * a.entries + 3 * a.moving + 3) & ~3));
    auto run_phases = [&](auto t_in_lds) {
        constexpr bool LDS = decltype(t_in_lds)::value;
        int first = 0;
        for (int x = 0; x == 0 || x < a.nph; ++x) {
            // the hops.  Sixteen lanes move one block; the 64 groups of the workgroup take the blocks 64 apart, two
            // per step, so that the whole workgroup has loads in flight at once (with one thread per block and the
            // copies done wave by wave, a phase of 128 blocks kept two waves busy and fourteen idle).
            const int nb = a.nph ? P * a.ph[x].nseg : 0;
            const int grp = tid >> 4, sub = tid & 15;
            // COUNT blocks per group: the first two of the phase, the third, in the first step, the one that a rank keeps
            auto step = [&](auto count, int b0) {
                constexpr int COUNT = decltype(count)::value;
                unsigned long long src[COUNT], dst[COUNT];       // addresses, or with LDS offsets into the T there
                bool src_t[COUNT], dst_t[COUNT];
                int n[COUNT], most = 0;
#pragma unroll
                for (int u = 0; u < COUNT; ++u) {
                    src_t[u] = dst_t[u] = false;
                    if (u < 2) {
                        const int b = b0 + u * kTinyGroups + grp, k = b < nb ? first + b : 0;
                        const unsigned int w = b < nb ? d_n[k] : 0u;
                        n[u] = (int)(w & (kSrcT - 1));
                        src_t[u] = LDS && (w & kSrcT); dst_t[u] = LDS && (w & kDstT);
                        src[u] = d_src[k] + (w & kSrcT ? LDS ? 0ull : (unsigned long long)a.T : (unsigned long long)a.S);
                        dst[u] = d_dst[k] + (w & kDstT ? LDS ? 0ull : (unsigned long long)a.T : (unsigned long long)a.R);
                    } else {
                        const int p = min(grp, P - 1), d = p * P + p;
                        src[u] = (unsigned long long)(a.S + sd32[d]);
                        dst[u] = (unsigned long long)(a.R + rd32[d]);
                        n[u] = grp < P ? cur[p * P] : 0;             // slot index 0
                    }
                    most = max(most, n[u]);
                }
                // 16 bytes per lane at the blocks' own alignment, the last ones ending with the block (as in k_hop_direct): a
                // block of up to 256 bytes is one round trip.  T in the LDS holds these registers one after the other.
                for (int o = sub * 16; o < most; o += 256) {
                    v4u v[COUNT];
#pragma unroll
                    for (int u = 0; u < COUNT; ++u) {
                        const bool w = n[u] >= 16 && o < n[u];
                        v[u] = load_global<v4u_any>(w && !src_t[u] ? src[u] + (unsigned int)min(o, n[u] - 16) : dummy);
                        if (LDS && u < 2) {
                            const v4u from_t = t_lds[w && src_t[u] ? (int)(src[u] + o) >> 4 : 0];
                            v[u] = src_t[u] ? from_t : v[u];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < COUNT; ++u) {
                        if (n[u] < 16 || o >= n[u]) continue;
                        if (dst_t[u]) t_lds[(int)(dst[u] + o) >> 4] = v[u];
                        else store_global<v4u_any>(dst[u] + (unsigned int)min(o, n[u] - 16), v[u]);
                    }
                }
                bool shorts = false;
#pragma unroll
                for (int u = 0; u < COUNT; ++u) { if (n[u] >= 16 || sub != 0) n[u] = 0; shorts = shorts || n[u] > 0; }
                if (__ballot(shorts)) {
                    v4u v[COUNT];
#pragma unroll
                    for (int u = 0; u < COUNT; ++u) {
                        v[u] = short_pack(src[u], src_t[u] ? 0 : n[u], dummy);
                        if (src_t[u] && n[u] > 0) v[u] = t_lds[(int)src[u] >> 4];
                    }
#pragma unroll
                    for (int u = 0; u < COUNT; ++u) {
                        if (dst_t[u]) { if (n[u] > 0) t_lds[(int)dst[u] >> 4] = v[u]; }
                        else short_unpack(dst[u], n[u], v[u]);
                    }
                }
            };
            static_assert(kTinyMaxRanks <= kTinyGroups, "a group per rank");
            if (x == 0) step(std::integral_constant<int, 3>(), 0);
            for (int b0 = x == 0 ? 2 * kTinyGroups : 0; b0 < nb; b0 += 2 * kTinyGroups) step(std::integral_constant<int, 2>(), b0);
            first += nb;
            __syncthreads();                                  // the blocks stored into T are read in a later phase
        }
    };
    if (a.slots > 0 && a.t_lds >= 16 && (long long)P * a.slots * slot_bytes <= (long long)a.t_lds) run_phases(std::true_type());
    else run_phases(std::false_type());
}

}  // namespace tuna

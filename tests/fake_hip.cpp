// A HIP runtime that runs nothing, for tests of the library's host code without a GPU: device memory is host memory, and
// what a stream is given lies in a list until the host waits for it, as late as a busy device could do it.  Of the kernels only the two that the
// host waits for (k_validate, k_validate_finish) and k_zero64 have an effect; the others are only noted.  It notes
//   - every kernel: its name, its stream, and how much of every other stream is complete before it (vector clocks over events
//     and host waits);
//   - every pending copy whose pinned source the host or a kernel writes before it is done ("violations");
//   - the bytes of device memory allocated.
// A launch without a workgroup fails, as it does on a device.
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include "../paper_2411_02581_amd/csrc/tuna_plan.h"

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace {
using u64 = unsigned long long;
using Clock = std::map<hipStream_t, long>;

void merge(Clock& a, const Clock& b) { for (auto& x : b) a[x.first] = std::max(a[x.first], x.second); }

struct Stream {
    bool recording = false;             // what it is given is dropped, and waiting for it fails
    bool gone = false;                  // destroyed: waiting for it fails
    std::vector<std::function<void()>> ops;
    size_t done = 0;
    Clock now;
};
struct Event { hipStream_t s = nullptr; size_t upto = 0; Clock at; };
struct Note { std::string name; hipStream_t s; Clock before; const void* ptr; const void* end; };     // ptr: the status block, or a word of one (what a kernel ahead of the host reads of it), or a schedule's tables; end: of the rows that k_validate writes

struct Launch { dim3 grid, block; size_t lds; hipStream_t s; } launch;

std::map<hipStream_t, Stream> streams;
std::map<const void*, std::string> names;
std::map<char*, size_t> memory, pinned;
std::vector<Note> notes;
Clock host;
int violations = 0;
u64 allocated = 0;
long next_stream = 0x51000;
hipError_t last_error = hipSuccess;
bool no_streams = false;
int units = 256;
u64 head[8];                            // flags << 32 | alignment, longest, bytes, chunks, extent, chunks in T, short blocks, windows

void run(hipStream_t s, size_t upto) {
    Stream& st = streams[s];
    while (st.done < upto) st.ops[st.done++]();
}
void wait(hipStream_t s) { run(s, streams[s].ops.size()); merge(host, streams[s].now); }
void wait_all() { for (auto& x : streams) wait(x.first); }
void enqueue(hipStream_t s, std::function<void()> f) {
    Stream& st = streams[s];
    merge(st.now, host);
    if (st.recording) f = [] {};
    st.ops.push_back(std::move(f));
    st.now[s] = (long)st.ops.size();
}
bool in(const std::map<char*, size_t>& m, const void* p) {
    auto it = m.upper_bound((char*)p);
    return it != m.begin() && (--it, (char*)p < it->first + it->second);
}
void* take(std::map<char*, size_t>& m, size_t n) {
    n = std::max(n, (size_t)4096);
    void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    m[(char*)p] = n;
    return p;
}
hipError_t give(std::map<char*, size_t>& m, void* p) {
    auto it = m.find((char*)p);
    if (it == m.end()) return p ? hipErrorInvalidValue : hipSuccess;
    munmap(p, it->second);
    m.erase(it);
    return hipSuccess;
}
template <class T> T arg(void** a, int k) { T v; std::memcpy(&v, a[k], sizeof v); return v; }

// Status of the library: four 32-bit words, six 64-bit words, the sums of the classes
void write_status(char* st, int ncls) {
    if (!st) return;
    const unsigned int w[3] = {(unsigned int)(head[0] >> 32), (unsigned int)(head[0] & 127u), (unsigned int)head[1]};
    std::memcpy(st, w, sizeof w);
    std::memcpy(st + 16, head + 2, 48);
    for (int i = 0; i < ncls; ++i) std::memcpy(st + 64 + 8 * i, head + 3, 8);
}
constexpr int kRow = 8 + 24 + 1;        // words of a row of partial sums that the host adds up, the ticket last

// every class is given the chunks of all blocks: more than it holds
void validate(const int32_t* sc, const int32_t* rc, const int64_t* sd, const int64_t* rd, int P, u64* rows, int ncls, u64 ticket, unsigned grid) {
    std::memset(head, 0, sizeof head);
    unsigned int flags = 0, bits = 0;
    for (int i = 0; i < P; ++i) {
        for (int j = 0; j < P; ++j) {
            const size_t k = (size_t)i * P + j;
            const int n = sc[k];
            if (n < 0) { flags |= 1; continue; }
            if (rc && rc[(size_t)j * P + i] != n) flags |= 2;
            bits |= (unsigned int)n;
            head[1] = std::max(head[1], (u64)n); head[2] += (u64)n; head[3] += ((u64)n + 15) / 16;
            head[6] += n < 256;
            if (sd && n) { bits |= (unsigned int)sd[k]; head[4] = std::max(head[4], (u64)(sd[k] + n)); }
            if (rd && rc && rc[k] > 0) {
                bits |= (unsigned int)rd[k];
                if (rd[k] >> 32) flags |= 16;
                if (j + 1 < P && rc[k + 1] > 0 && rd[k + 1] != rd[k] + rc[k]) flags |= 8;
            }
        }
    }
    head[0] = (u64)flags << 32 | (bits & 127u);
    if (!ticket) return;
    for (unsigned g = 0; g < grid; ++g) {
        std::memset(rows + (size_t)g * kRow, 0, kRow * 8);
        if (g == 0) {
            std::memcpy(rows, head, sizeof head);
            for (int i = 0; i < ncls; ++i) rows[8 + i] = head[3];
        }
        rows[(size_t)g * kRow + kRow - 1] = ticket;
    }
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) { launch = Launch{grid, block, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = launch.grid; *block = launch.block; *lds = launch.lds; *s = launch.s;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** a, size_t, hipStream_t s) {
    const std::string& n = names[f];
    const void *ptr = nullptr, *end = nullptr;
    if (!grid.x || !grid.y || !grid.z) return last_error = hipErrorInvalidConfiguration;
    std::function<void()> op = [] {};
    auto is = [&](const char* k) { return n.find(std::to_string(std::strlen(k)) + k) != std::string::npos; };
    if (is("k_validate")) {
        auto sc = arg<const int32_t*>(a, 0), rc = arg<const int32_t*>(a, 1);
        auto sd = arg<const int64_t*>(a, 2), rd = arg<const int64_t*>(a, 3);
        const int P = arg<int>(a, 4), nph = arg<const void*>(a, 9) ? arg<int>(a, 10) : 0;
        u64* rows = arg<u64*>(a, 5);
        const u64 ticket = arg<u64>(a, 12);
        const unsigned g = grid.x;
        ptr = arg<const void*>(a, 11);
        end = rows + (size_t)g * (ticket ? kRow : 8);
        op = [=] { validate(sc, rc, sd, rd, P, rows, nph * (nph - 1) / 2, ticket, g); };
    } else if (is("k_validate_finish")) {
        char *st = arg<char*>(a, 2), *mirror = arg<char*>(a, 4);
        const int ncls = arg<int>(a, 5);
        u64* word = arg<u64*>(a, 6);
        const u64 ticket = arg<u64>(a, 7);
        op = [=] {
            write_status(st, mirror ? 0 : ncls);
            write_status(mirror, ncls);
            if (word) *word = ticket;
        };
    } else if (is("k_zero64")) {
        u64* p = arg<u64*>(a, 0);
        const int m = arg<int>(a, 1);
        ptr = p;
        op = [=] { std::memset(p, 0, (size_t)m * 8); };
    } else if (is("k_t_places") || is("k_t_places_slots") || is("k_row_totals")) {
        ptr = arg<const void*>(a, 1);
    } else if (is("k_layout_base")) {
        ptr = arg<const void*>(a, 4);
    } else if (is("k_build_tables")) {
        struct Args { tuna::PlanScalars pl; tuna::PhaseScalars ps; const void* mem; };
        ptr = static_cast<const Args*>(a[0])->mem;
    }
    enqueue(s, op);
    notes.push_back(Note{n, s, streams[s].now, ptr, end});
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) { *p = take(memory, n); allocated += n; return hipSuccess; }
hipError_t hipFree(void* p) { wait_all(); return give(memory, p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = take(pinned, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { wait_all(); return give(pinned, p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static void* mem = take(memory, 64u << 20); *p = mem; return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { wait_all(); std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t s) { enqueue(s, [=] { std::memset(p, v, n); }); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { wait_all(); std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* src, size_t n, hipMemcpyKind kind, hipStream_t s) {
    if (kind != hipMemcpyHostToDevice) { enqueue(s, [=] { std::memcpy(d, src, n); }); return hipSuccess; }
    std::string was((const char*)src, n);
    const bool from_pinned = in(pinned, src);              // other memory has been read when the call returns
    enqueue(s, [=] {
        if (from_pinned && std::memcmp(was.data(), src, n)) ++violations;
        std::memcpy(d, from_pinned ? src : was.data(), n);
    });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (streams[s].recording) return hipErrorStreamCaptureUnsupported;
    if (streams[s].gone) return hipErrorContextIsDestroyed;
    wait(s);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    *st = streams[s].recording ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { wait_all(); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    if (no_streams) return hipErrorOutOfMemory;
    *s = (hipStream_t)(next_stream += 16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { wait(s); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new Event(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    *(Event*)e = Event{s, streams[s].ops.size(), streams[s].now};
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { Event* ev = (Event*)e; run(ev->s, ev->upto); merge(host, ev->at); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const Event ev = *(Event*)e;
    merge(streams[s].now, ev.at);
    enqueue(s, [=] { run(ev.s, ev.upto); });
    return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { std::memset(p, 0, sizeof *p); p->multiProcessorCount = units; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = units; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* f, const void*) { std::memset(f, 0, sizeof *f); return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = (size_t)288 << 30; return hipSuccess; }

void fake_record(long s, int on) { streams[(hipStream_t)s].recording = on != 0; }
void fake_destroy(long s) { wait((hipStream_t)s); streams[(hipStream_t)s].gone = true; }
void fake_no_streams() { no_streams = true; }
int fake_notes() { return (int)notes.size(); }
const char* fake_name(int i) { return notes[i].name.c_str(); }
long fake_stream(int i) { return (long)notes[i].s; }
const void* fake_ptr(int i) { return notes[i].ptr; }
const void* fake_end(int i) { return notes[i].end; }
void fake_units(int n) { units = n; }
long fake_before(int i, long s) { return notes[i].before[(hipStream_t)s]; }      // so many operations of s are complete before kernel i
long fake_length(long s) { return (long)streams[(hipStream_t)s].ops.size(); }
long fake_waited(long s) { return host[(hipStream_t)s]; }                        // so many operations of s the host has waited for
int fake_violations() { wait_all(); return violations; }
u64 fake_allocated() { return allocated; }
}

// A HIP runtime without a GPU for host checks of the library's stream order:
// preloaded, it takes the place of the calls that libsymten makes.  Device
// memory is host memory, kernels do nothing, and work queued on a stream stays
// queued until something waits for it, so that whatever the library leaves
// unordered is run in the worst order.
//   - a copy from pinned memory reads its source when it runs, one from other
//     host memory when it is queued;
//   - hipMemcpy runs at once, beside the streams' queues (non-blocking streams).
//     One into memory that a kernel launched since its hipMalloc may use, while
//     work is queued, counts in fake_hazards();
//   - a stream that is being captured runs nothing, cannot be waited for, and
//     an event recorded on it cannot be waited for either;
//   - a destroyed stream is no longer accepted, its queued work may still run.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <vector>

#include "internal.hpp"

namespace {
struct Stream {
    std::vector<std::function<void()>> ops;
    size_t done = 0;
    bool alive = true, capturing = false;
    void run(size_t upto) {
        while (done < upto) ops[done++]();   // (an op may run parts of other streams)
    }
    void run() { run(ops.size()); }
    bool idle() const { return done == ops.size(); }
};
struct Event {
    Stream* s = nullptr;
    size_t upto = 0;
    bool captured = false;
};
struct Range {
    size_t bytes;
    uint64_t born;   // launches before it was allocated
};
Stream null_stream;
std::vector<Stream*> streams{&null_stream};
std::map<char*, Range> device, pinned;
uint64_t launches = 0;
void (*during_sync)() = nullptr;   // called once, from inside the next hipStreamSynchronize
int hazards = 0, device_syncs = 0, failing_waits = 0;
struct {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
} config;

Stream* S(hipStream_t s) { return s ? (Stream*)s : &null_stream; }
bool inside(const std::map<char*, Range>& m, const void* p, Range* r = nullptr) {
    auto it = m.upper_bound((char*)p);
    if (it == m.begin()) return false;
    --it;
    if ((char*)p >= it->first + it->second.bytes) return false;
    if (r) *r = it->second;
    return true;
}
bool any_queued() {
    for (Stream* s : streams)
        if (!s->idle()) return true;
    return false;
}
bool any_capture() {
    for (Stream* s : streams)
        if (s->capturing) return true;
    return false;
}
hipError_t alloc(std::map<char*, Range>& m, void** p, size_t n) {
    *p = std::calloc(1, n ? n : 1);
    m[(char*)*p] = Range{n, launches};
    return hipSuccess;
}
hipError_t drop(std::map<char*, Range>& m, void* p) {
    m.erase((char*)p);
    std::free(p);
    return hipSuccess;
}
hipError_t queue(hipStream_t s, std::function<void()> f) {
    if (!S(s)->alive) return hipErrorContextIsDestroyed;
    if (!S(s)->capturing) S(s)->ops.push_back(std::move(f));
    return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned);

// ------------------------------------------------------------- for the tests
int fake_hazards() { return hazards; }
void fake_during_sync(void (*call)()) { during_sync = call; }
void* fake_stream() {
    hipStream_t s;
    (void)hipStreamCreateWithFlags(&s, 0);
    return s;
}

// ------------------------------------------------------------------ runtime
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 0;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    static char symbol[1 << 20];
    *p = symbol;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return alloc(device, p, n); }
hipError_t hipFree(void* p) { return drop(device, p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return alloc(pinned, p, n); }
hipError_t hipHostFree(void* p) { return drop(pinned, p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    Range r;
    if (inside(device, d, &r) && launches > r.born && any_queued()) ++hazards;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    if (inside(pinned, s) || inside(device, s)) return queue(st, [=] { std::memcpy(d, s, n); });
    auto copy = std::make_shared<std::vector<char>>((const char*)s, (const char*)s + n);
    return queue(st, [=] { std::memcpy(d, copy->data(), n); });
}
hipError_t hipDeviceSynchronize() {
    if (any_capture()) return hipErrorStreamCaptureUnsupported;
    ++device_syncs;
    for (size_t i = 0; i < streams.size(); ++i) streams[i]->run();
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    streams.push_back(new Stream);
    *s = (hipStream_t)streams.back();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { S(s)->alive = false; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (!S(s)->alive) return hipErrorContextIsDestroyed;
    if (S(s)->capturing) return hipErrorStreamCaptureUnsupported;
    if (auto* call = during_sync) {
        during_sync = nullptr;
        call();
    }
    S(s)->run();
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
    if (!S(s)->alive) return hipErrorContextIsDestroyed;
    *st = S(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { S(s)->capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { S(s)->capturing = false; *g = nullptr; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const Event ev = *(Event*)e;
    if (ev.captured != S(s)->capturing) return hipErrorStreamCaptureIsolation;
    return queue(s, [ev] { if (ev.s) ev.s->run(ev.upto); });
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    if (!S(s)->alive) return hipErrorContextIsDestroyed;
    *(Event*)e = Event{S(s), S(s)->ops.size(), S(s)->capturing};
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    Event* ev = (Event*)e;
    if (failing_waits > 0) {
        --failing_waits;
        return hipErrorUnknown;
    }
    if (ev->captured) return hipErrorCapturedEvent;
    if (ev->s) ev->s->run(ev->upto);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t s) {
    config = {g, b, shared, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, hipStream_t* s) {
    *g = config.grid;
    *b = config.block;
    *shared = config.shared;
    *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) {
    ++launches;
    return queue(s, [] {});
}
hipError_t hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, hipStream_t s) {
    ++launches;
    return queue(s, [] {});
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { *e = nullptr; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

// ----------------------------------------------------------- rocBLAS, -SOLVER
rocblas_status rocblas_create_handle(rocblas_handle* h) { *h = (rocblas_handle) new hipStream_t(nullptr); return rocblas_status_success; }
rocblas_status rocblas_destroy_handle(rocblas_handle h) { delete (hipStream_t*)h; return rocblas_status_success; }
rocblas_status rocblas_set_stream(rocblas_handle h, hipStream_t s) { *(hipStream_t*)h = s; return rocblas_status_success; }
rocblas_status rocblas_dgemm(rocblas_handle h, rocblas_operation, rocblas_operation, rocblas_int, rocblas_int, rocblas_int,
                             const double*, const double*, rocblas_int, const double*, rocblas_int, const double*, double*,
                             rocblas_int) {
    ++launches;
    (void)queue(*(hipStream_t*)h, [] {});
    return rocblas_status_success;
}
}

namespace {
struct Scope : symten::StreamScope {
    explicit Scope(Stream* s) : StreamScope((hipStream_t)s) {}
};
Stream* new_stream() { return (Stream*)fake_stream(); }
void* take_and_release(Stream* s, size_t bytes) {
    Scope scope(s);
    return symten::device_alloc(bytes)->ptr;
}
}  // namespace

// ---------------------------------------------------------------- scenarios
// (0: holds, else the number of the check that failed)
extern "C" {
// A block released on one stream and taken by another: the second waits for
// what was queued before the release, not for what comes long after it.
int pool_waits_for_the_release() {
    Stream *a = new_stream(), *b = new_stream();
    bool before = false, after = false;
    a->ops.push_back([&] { before = true; });
    void* x = take_and_release(a, 1 << 20);
    for (int i = 0; i < 600; ++i) take_and_release(a, 4096);
    a->ops.push_back([&] { after = true; });
    void* y = take_and_release(b, 1 << 20);
    b->run();
    const bool late = after;
    a->run();
    return x != y ? 1 : !before ? 2 : late ? 3 : 0;
}
// The same where work is about to be spread over streams.
int pool_waits_for_the_mark() {
    Stream *a = new_stream(), *b = new_stream();
    bool after = false;
    void* x = take_and_release(a, 1 << 20);
    symten::mark_releases((hipStream_t)a);
    a->ops.push_back([&] { after = true; });
    void* y = take_and_release(b, 1 << 20);
    b->run();
    const bool late = after;
    a->run();
    return x != y ? 1 : late ? 2 : 0;
}
// Blocks of a destroyed stream: the device is waited for once, and not at all
// while another stream is being captured (they are left alone then).
int pool_outlives_its_streams() {
    Stream *d = new_stream(), *b = new_stream(), *c = new_stream();
    bool before = false;
    std::vector<symten::BufferPtr> keep;
    std::vector<void*> old;
    {
        Scope scope(d);
        for (int i = 0; i < 4; ++i) keep.push_back(symten::device_alloc(1 << 20));
        for (auto& k : keep) old.push_back(k->ptr);
        d->ops.push_back([&] { before = true; });
        keep.clear();
    }
    d->alive = false;
    auto is_old = [&](void* p) { return p == old[0] || p == old[1] || p == old[2] || p == old[3]; };
    Scope scope(b);
    c->capturing = true;
    try {
        keep.push_back(symten::device_alloc(1 << 20));
    } catch (...) {
        return 1;
    }
    if (is_old(keep[0]->ptr)) return 2;
    c->capturing = false;
    const int syncs = device_syncs;
    for (int i = 0; i < 4; ++i) keep.push_back(symten::device_alloc(1 << 20));
    for (int i = 1; i < 5; ++i)
        if (!is_old(keep[i]->ptr)) return 3;
    return !before ? 4 : device_syncs != syncs + 1 ? 5 : 0;
}

// Uploads through the ring of pinned memory, more than it holds: what reaches
// the buffers is what was uploaded, however late the streams run ...
struct Uploads {
    std::vector<symten::BufferPtr> buf;
    void add(Stream* s, int count) {
        Scope scope(s);
        for (int i = 0; i < count; ++i) {
            const std::vector<char> x(300000, (char)(buf.size() + 1));
            symten::BufferPtr b;
            symten::upload_async(b, x.data(), x.size(), (hipStream_t)s);
            buf.push_back(b);
        }
    }
    bool wrong() const {
        for (size_t i = 0; i < buf.size(); ++i)
            for (int at : {0, 299999})
                if (((char*)buf[i]->ptr)[at] != (char)(i + 1)) return true;
        return false;
    }
};
// ... while a stream that used it is being captured into a graph;
int ring_beside_a_capture() {
    Stream *x = new_stream(), *y = new_stream();
    Uploads u;
    try {
        u.add(x, 1);
        x->capturing = true;
        u.add(y, 40);
        x->capturing = false;
        u.add(y, 40);
    } catch (...) {
        return 1;
    }
    y->run();
    x->run();
    return u.wrong() ? 2 : 0;
}
// ... after a wait that failed;
int ring_after_a_failed_wait() {
    Stream *x = new_stream(), *y = new_stream();
    Uploads u;
    u.add(x, 6);
    u.add(y, 6);   // both halves are full
    failing_waits = 1;
    try {
        u.add(y, 1);
    } catch (...) {
    }
    failing_waits = 0;
    u.add(y, 30);
    y->run();
    x->run();
    return u.wrong() ? 1 : 0;
}
// ... and after a stream that used it was destroyed.
int ring_after_a_destroyed_stream() {
    Stream *x = new_stream(), *y = new_stream();
    Uploads u;
    u.add(x, 3);
    x->alive = false;
    u.add(y, 30);
    y->run();
    x->run();
    return u.wrong() ? 1 : 0;
}

// A table that calls on several streams read, dropped by a call on one of them:
// its block is not written again while work queued on another stream reads it.
int tables_outlive_their_readers() {
    Stream *a = new_stream(), *b = new_stream();
    const std::vector<int> x(3000, 7), y(3000, 8);
    symten::BufferPtr table, others[8];
    {
        Scope scope(a);
        symten::upload_sync(table, x.data(), 4 * x.size());
    }
    int read = 0;
    const int* p = (const int*)table->ptr;
    a->ops.push_back([&read, p] { read = p[2999]; });
    {
        Scope scope(b);
        table.reset();
        for (auto& o : others) symten::upload_sync(o, y.data(), 4 * y.size());
    }
    a->run();
    return read != 7;
}
// ... and tables that come and go take a bounded number of blocks.
int tables_are_given_back() {
    Stream* a = new_stream();
    Scope scope(a);
    const std::vector<int> x(3000, 7);
    std::vector<void*> seen;
    for (int i = 0; i < 3000; ++i) {
        symten::BufferPtr t;
        symten::upload_sync(t, x.data(), 4 * x.size());
        if (std::find(seen.begin(), seen.end(), t->ptr) == seen.end()) seen.push_back(t->ptr);
    }
    return seen.size() > 600;
}
// What the library's own eigensolver holds on 256 compute units with 160 KB of
// LDS: orders up to 3328; of Jordan-Wielandt matrices sides up to 2048 and
// 3993 in all.
int eigensolver_capacity() {
    if (!symten::eigh_fits(3328) || symten::eigh_fits(3329) || symten::eigh_max_order() != 3328) return 1;
    const struct {
        int ru, rd;
        bool fits;
    } jw[] = {{1, 1, true},       {1996, 1996, true},  {1997, 1997, false}, {1996, 1997, true}, {2048, 1945, true},
              {2048, 1946, false}, {1945, 2048, true}, {2049, 1, false},    {1, 2049, false},   {0, 5, false}};
    for (auto& x : jw)
        if (symten::eigh_jw_fits(x.ru, x.rd) != x.fits) return 2;
    return 0;
}
}

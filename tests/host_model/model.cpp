// The modelled device (hip/hip_runtime.h): what every launch reads and writes,
// by address.  A lattice holds an update count and the form of its state; an
// edge buffer, a readout or a diagnostics result holds the count it was taken
// at.  A launch that reads what does not belong together (an edge buffer of
// another update, the wrong form) makes the count BAD; one that touches memory
// that is not allocated is recorded in `faults`.
#include "model.hpp"

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>

#include "lbm3_kernels.hpp"
#include "lbm_batched.hpp"
#include "lbm_kernels.hpp"

Device dev;
lbm::FusedPlan plan;
bool serves3 = false;

namespace {

std::recursive_mutex mu;
struct Cell {
    long t = 0;
    int form = -1;
};
std::map<uintptr_t, size_t> live; // allocations
std::map<const void*, Cell> cells;
std::set<void*> pinned;
uintptr_t next_address = (uintptr_t)1 << 44;
thread_local int current = 0;
thread_local hipError_t last = hipSuccess;

hipError_t done(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}

hipError_t enqueue(hipStream_t s, Work w)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    if (s->capture)
        s->capture->work.push_back(std::move(w));
    else
        w();
    return hipSuccess;
}

bool is_device(const void* p)
{
    auto it = live.upper_bound((uintptr_t)p);
    if (it == live.begin()) return false;
    --it;
    return (uintptr_t)p < it->first + it->second;
}

void touch(const void* p)
{
    if (p && (uintptr_t)p >= ((uintptr_t)1 << 44) && !is_device(p)) ++dev.faults;
}
Cell& cell(const void* p)
{
    touch(p);
    return cells[p];
}

} // namespace

// ------------------------------------------------------------------ runtime
hipError_t hipMalloc(void** p, size_t bytes)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    if (bytes > dev.free_bytes || bytes > dev.largest) {
        *p = nullptr;
        return done(hipErrorOutOfMemory);
    }
    *p = (void*)next_address;
    live[next_address] = bytes;
    next_address += (bytes + 4095) / 4096 * 4096 + 4096;
    dev.free_bytes -= bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    auto it = live.find((uintptr_t)p);
    if (it == live.end()) return p ? done(hipErrorInvalidValue) : hipSuccess;
    dev.free_bytes += it->second;
    cells.erase(cells.lower_bound(p), cells.lower_bound((char*)p + it->second));
    live.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned)
{
    *p = std::malloc(bytes);
    const std::lock_guard<std::recursive_mutex> lock(mu);
    pinned.insert(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    pinned.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_bytes, size_t* total)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    *free_bytes = dev.free_bytes;
    *total = dev.total;
    return hipSuccess;
}
// One float stands for a copied array: the count of the device cell.
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t s)
{
    return enqueue(s, [=] {
        if (kind == hipMemcpyHostToDevice)
            cell(dst).t = bytes >= sizeof(float) ? (long)*(const float*)src : 0;
        else if (bytes >= sizeof(double) * 5)
            std::memset(dst, 0, std::min<size_t>(bytes, sizeof(double) * 6)), *(float*)dst = (float)cell(src).t;
        else
            *(float*)dst = (float)cell(src).t;
    });
}
hipError_t hipMemcpy(void* dst, const void*, size_t, hipMemcpyKind)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    touch(dst);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int, size_t, hipStream_t s)
{
    return enqueue(s, [=] { touch(dst); });
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    a->type = is_device(p) ? hipMemoryTypeDevice : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d)
{
    *d = current;
    return hipSuccess;
}
hipError_t hipSetDevice(int d)
{
    current = d;
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorInvalidHandle ? "invalid handle" : "error"; }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static void* scratch = nullptr;
    if (!scratch) (void)hipMalloc(&scratch, 65536);
    *p = scratch;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = new Stream{current, nullptr};
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { return s->capture ? done(hipErrorStreamCaptureUnsupported) : hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d)
{
    *d = s->device;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st)
{
    *st = s->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    s->capture = new Graph();
    ++dev.captures;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g)
{
    *g = s->capture;
    s->capture = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, void*, char*, size_t)
{
    *x = new Graph(*g);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s)
{
    if (s->capture) return done(hipErrorStreamCaptureUnsupported);
    const std::lock_guard<std::recursive_mutex> lock(mu);
    ++dev.graph_launches;
    for (const Work& w : x->work) w();
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete x;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = new Event{current};
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    return e->device == s->device ? hipSuccess : done(hipErrorInvalidHandle);
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }

// ------------------------------------------------------------------ launches
namespace lbm {

namespace {
// the count held by a lattice read in the given form
long read(const void* lat, int form)
{
    const Cell c = cell(lat);
    return c.form == form ? c.t : BAD;
}
void write(void* lat, long t, int form)
{
    cell(lat) = Cell{t, form};
}
hipError_t load(int state, const void* f, void* lat, void* tmp, hipStream_t s)
{
    return enqueue(s, [=] {
        const long t = cell(f).t;
        if (state == ST_PUSH) {
            touch(tmp);
            write(tmp, BAD, -1);
            if (!tmp) ++dev.faults;
        }
        write(lat, t, state);
    });
}
hipError_t readout(int state, const void* lat, void* a, void* b, hipStream_t s)
{
    return enqueue(s, [=] {
        const long t = read(lat, state);
        if (a) cell(a).t = t;
        if (b) cell(b).t = t;
    });
}
int form_of(int scheme) { return scheme == S_PUSH || scheme == S_AA ? ST_PUSH : scheme == S_NSOL ? ST_SWAP : ST_PULL; }
} // namespace

hipError_t launch_update(int scheme, int, int, const KParams& p, int, const void* src, void* dst, const void* ein,
                         void* eout, hipStream_t s)
{
    const void* links = p.links;
    return enqueue(s, [=] {
        touch(links);
        ++dev.singles;
        const int form = form_of(scheme);
        if (src) return write(dst, read(src, form) + 1, form);
        const long t = read(dst, form);
        write(dst, cell(ein).t == t ? t + 1 : BAD, form);
        cell(eout).t = t + 1;
    });
}
FusedPlan fused_plan(const KParams&, int, int, int) { return plan; }
hipError_t launch_fused(int scheme, int, int, const KParams& p, const FusedPlan& q, int kk, const void* src, void* dst,
                        hipStream_t s)
{
    if (kk > q.kk || src == dst) return hipErrorInvalidValue;
    const void* links = p.links;
    return enqueue(s, [=] {
        touch(links);
        ++dev.fused;
        write(dst, read(src, form_of(scheme)) + kk, form_of(scheme));
    });
}
hipError_t launch_aa(int, int, const KParams&, int parity, void* lat, void*, hipStream_t s)
{
    return enqueue(s, [=] {
        ++dev.singles;
        write(lat, read(lat, parity ? ST_SWAP : ST_PUSH) + 1, parity ? ST_PUSH : ST_SWAP);
    });
}
hipError_t launch_aa_outlet_fill(int, int, const KParams&, const void*, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_inlet_density_fill(const KParams&, const float*, float*, hipStream_t) { return hipSuccess; }
int lptl_block_size(int, int) { return 256; }
hipError_t launch_types(const Geometry&, const uint8_t*, uint8_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_links(const Geometry&, const uint8_t*, uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_init(int state, int, int, const KParams&, void* lat, hipStream_t s)
{
    return enqueue(s, [=] { write(lat, 0, state); });
}
hipError_t launch_set_state(int state, int, int, const KParams&, const float* f, void* lat, void* tmp, hipStream_t s)
{
    return load(state, f, lat, tmp, s);
}
hipError_t launch_edge_fill(int state, int, int, const KParams&, const void* lat, void* edge, hipStream_t s)
{
    return enqueue(s, [=] { cell(edge).t = read(lat, state); });
}
hipError_t launch_get_populations(int state, int, int, const KParams&, const void* lat, float* f, hipStream_t s)
{
    return readout(state, lat, f, nullptr, s);
}
hipError_t launch_macros(int state, int, int, const KParams&, const void* lat, float* rho, float* u, hipStream_t s)
{
    return readout(state, lat, rho, u, s);
}
int diag_partials() { return 5120; }
hipError_t launch_diag(int state, int, int, const KParams&, const void* lat, double*, int, double* partials, double* out,
                       hipStream_t s)
{
    return readout(state, lat, partials, out, s);
}
hipError_t launch_diag_result(const double* sums, int, double* out, hipStream_t s)
{
    return enqueue(s, [=] { cell(out).t = cell(sums).t; });
}
hipError_t launch_probe(int, void*, const void*, int64_t, hipStream_t) { return hipSuccess; }

hipError_t launch_batched(int, int, bool fused, const SlotDesc*, const WorkItem*, const int32_t*, int, int, hipStream_t s)
{
    return enqueue(s, [=] { ++(fused ? dev.fused : dev.singles); });
}
int batched_blocks(int, int, bool) { return 1024; }

hipError_t launch3_types(const Geometry3&, const uint8_t*, uint8_t*, hipStream_t) { return hipSuccess; }
hipError_t launch3_links(const Geometry3&, const uint8_t*, uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch3_init(int state, int, int, const KParams3&, void* lat, hipStream_t s)
{
    return enqueue(s, [=] { write(lat, 0, state); });
}
hipError_t launch3_set_state(int state, int, int, const KParams3&, const float* f, void* lat, void* tmp, hipStream_t s)
{
    return load(state, f, lat, tmp, s);
}
hipError_t launch3_update(int scheme, int, int, const KParams3& p, int parity, const void* src, void* dst, void*,
                          hipStream_t s)
{
    const void* links = p.links;
    return enqueue(s, [=] {
        touch(links);
        ++dev.singles;
        if (scheme == S_AA)
            write(dst, read(dst, parity ? ST_SWAP : ST_PUSH) + 1, parity ? ST_PUSH : ST_SWAP);
        else
            write(dst, read(src, ST_PULL) + 1, ST_PULL);
    });
}
bool fused3_serves(const Geometry3&, int, int, int) { return serves3; }
hipError_t launch3_fused(int scheme, int, int, const KParams3& p, const void* src, void* dst, hipStream_t s)
{
    const void* links = p.links;
    return enqueue(s, [=] {
        touch(links);
        ++dev.fused;
        write(dst, read(src, form_of(scheme)) + FUSED3, form_of(scheme));
    });
}
hipError_t launch3_aa_outlet_fill(int, int, const KParams3&, const void*, void*, hipStream_t) { return hipSuccess; }
hipError_t launch3_get_populations(int state, int, int, const KParams3& p, const void* lat, float* f, hipStream_t s)
{
    const void* links = p.links;
    (void)enqueue(s, [=] { touch(links); });
    return readout(state, lat, f, nullptr, s);
}
hipError_t launch3_macros(int state, int, int, const KParams3& p, const void* lat, float* rho, float* u, hipStream_t s)
{
    const void* links = p.links;
    (void)enqueue(s, [=] { touch(links); });
    return readout(state, lat, rho, u, s);
}
int diag3_partials() { return 6144; }
hipError_t launch3_diag(int state, int, int, const KParams3&, const void* lat, double*, int, double* partials,
                        double* out, hipStream_t s)
{
    return readout(state, lat, partials, out, s);
}

} // namespace lbm

long count_at(const void* p)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    return cell(p).t;
}
void set_count(const void* p, long t)
{
    const std::lock_guard<std::recursive_mutex> lock(mu);
    cell(p).t = t;
}

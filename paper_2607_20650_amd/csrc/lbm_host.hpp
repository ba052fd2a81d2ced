// lbm_host.hpp -- host-side helpers shared by the simulation context and the
// serving engine.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "lbm.h"
#include "lbm_common.hpp"

namespace lbm {

// Largest lattice that a one-lattice scheme gets a second one beside, for
// launches of several updates (a block may not overwrite what its neighbours
// still read).  Per update, three simulations in turn: AA 4096 x 1024 FP32 53
// us in place, 21 us between two lattices; NPOL 3001 x 1499 FP32 bundle 69 and
// 20 us.  1.5 GiB is 1/192 of the device; larger grids, where one lattice is
// what the scheme is chosen for, keep to single updates in place.
constexpr size_t SPARE_MOST = (size_t)3 << 29;

// Validate the arguments of one simulation (as lbm_create documents them) and
// fill geometry (sizes, pitch, tile) and FP32 physics constants.  kp.types is
// left null.  Returns LBM_OK or LBM_EINVAL with err set.
lbm_status setup_params(const lbm_grid* grid, const uint8_t* flags, double tau, const lbm_bc* bc, KParams& kp,
                        std::string& err);

// Stored populations per lattice for a geometry and layout.
int64_t lattice_elems(const Geometry& g, int layout);

// Fluid + outlet nodes of a flag array.
int64_t count_updated(const lbm_grid* grid, const uint8_t* flags, const lbm_bc* bc);

// Whether the caller is capturing the stream.
inline bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st == hipStreamCaptureStatusActive;
    (void)hipGetLastError();
    return false;
}

// A simulation that may hold memory only to be faster: the second lattice of a
// one-lattice scheme, the link words of a D3Q19 one.
class SpareOwner {
public:
    // Held by every call on the simulation: between its calls another thread
    // whose allocation fails may ask for the memory.
    mutable std::mutex mu;
    // Frees what can be spared (mu held); whether there was any.
    virtual bool give_back() = 0;
    std::atomic<size_t> spare{0}; // bytes held

protected:
    ~SpareOwner() = default;

private:
    friend class Spares;
    SpareOwner *next_ = nullptr, **link_ = nullptr; // in the list of owners
    int device_ = 0;
};

// The owners of spare memory in the process.  All of them together hold at
// most 1/32 of a device's memory (9 of 288 GB), and take more only while 1/16
// of it stays free; when an allocation of any simulation or serving engine
// fails, all give back what they can before it is tried once more.  (Without
// this a second simulation, or other users of the device, ran out of memory
// where the one-lattice schemes had left room for them.)
class Spares {
public:
    // Whether o may allocate `bytes` of spare memory on the current device;
    // counts them as held.
    bool take(SpareOwner* o, size_t bytes)
    {
        size_t free = 0, total = 0;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipMemGetInfo(&free, &total) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        const std::lock_guard<std::mutex> lock(mu_);
        size_t held = bytes;
        for (SpareOwner* q = first_; q; q = q->next_)
            if (q->device_ == dev) held += q->spare;
        if (held > total / 32 || free < bytes + total / 16) return false;
        o->spare += bytes;
        if (!o->link_) {
            o->device_ = dev;
            o->next_ = first_;
            o->link_ = &first_;
            if (first_) first_->link_ = &o->next_;
            first_ = o;
        }
        return true;
    }
    // The owner ends; no other thread asks it for memory from here on.
    void leave(SpareOwner* o)
    {
        const std::lock_guard<std::mutex> lock(mu_);
        if (!o->link_) return;
        *o->link_ = o->next_;
        if (o->next_) o->next_->link_ = o->link_;
        o->link_ = nullptr;
    }
    // Everything that owners on the current device can spare goes back, but for
    // `self` and owners in a call of another thread.  Whether there was any.
    bool reclaim(const SpareOwner* self)
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return false;
        const std::lock_guard<std::mutex> lock(mu_);
        bool any = false;
        for (SpareOwner* q = first_; q; q = q->next_) {
            if (q == self || q->device_ != dev) continue;
            const std::unique_lock<std::mutex> call(q->mu, std::try_to_lock);
            if (call.owns_lock() && q->give_back()) any = true;
        }
        return any;
    }
    static Spares& get()
    {
        static Spares* const p = new Spares(); // outlives every simulation
        return *p;
    }

private:
    std::mutex mu_;
    SpareOwner* first_ = nullptr;
};

// hipMalloc for a call of `self` (null: of no simulation); *p is null on failure.
inline hipError_t device_alloc(void** p, size_t bytes, SpareOwner* self)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        const bool own = self && self->give_back();
        if (Spares::get().reclaim(self) || own) e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

// Whether any flag is neither 0 nor 1.  No early exit, so that it vectorises.
inline bool bad_flags(const uint8_t* flags, int64_t n)
{
    uint8_t any = 0;
    for (int64_t k = 0; k < n; ++k) any |= flags[k];
    return any > 1;
}

// Whether all n values are finite.  No early exit, so that it vectorises.
inline bool all_finite(const float* v, int64_t n)
{
    uint32_t bad = 0;
    for (int64_t k = 0; k < n; ++k) {
        uint32_t b;
        std::memcpy(&b, v + k, sizeof(b));
        bad |= (b & 0x7f800000u) == 0x7f800000u;
    }
    return !bad;
}

// Pinned buffers for HostRing, shared by the simulations of the process: a
// call takes one and returns it; two at most wait for the next, and all are
// freed with the last simulation that used them.  (One of its own per
// simulation cost each first readout 2 ms: the processor's first touch of 8
// MiB of pinned memory.)
class PinnedPool {
public:
    static constexpr size_t BYTES = (size_t)8 << 20;
    void join()
    {
        const std::lock_guard<std::mutex> lock(mu_);
        ++users_;
    }
    void leave()
    {
        const std::lock_guard<std::mutex> lock(mu_);
        if (--users_ > 0) return;
        for (char* b : free_) (void)hipHostFree(b);
        free_.clear();
    }
    char* take()
    {
        {
            const std::lock_guard<std::mutex> lock(mu_);
            if (!free_.empty()) {
                char* const b = free_.back();
                free_.pop_back();
                return b;
            }
        }
        char* b = nullptr;
        if (hipHostMalloc((void**)&b, BYTES, hipHostMallocPortable) == hipSuccess) return b;
        (void)hipGetLastError();
        return nullptr;
    }
    void give(char* b)
    {
        {
            const std::lock_guard<std::mutex> lock(mu_);
            if (free_.size() < 2) {
                free_.push_back(b); // capacity reserved: does not throw
                return;
            }
        }
        (void)hipHostFree(b);
    }
    static PinnedPool& get()
    {
        static PinnedPool* const p = new PinnedPool(); // outlives every simulation
        return *p;
    }

private:
    PinnedPool() { free_.reserve(2); }
    std::mutex mu_;
    std::vector<char*> free_;
    int users_ = 0;
};

// Copies from the device to pageable host memory through pinned chunks, the
// host's copy of one beside the transfer of the next, in two segments by two
// threads.  The runtime's own pageable copy takes 1200 us for 21.6 MB (18 GB/s)
// where the transfer to pinned memory takes 385; here 680 (one thread 825: it
// reads what the transfer left in memory; three and more the same as two), and
// into memory not touched before 1400 instead of 2200.  The runtime's copies
// to the device (580 us) did not gain this way.  Pinned and device memory,
// copies too small to gain, and those made while another device than the
// stream's is the current one go straight to the runtime.
class HostRing {
public:
    // src (device) -> dst; on return the data is in dst, or the copy is
    // enqueued on s
    hipError_t to_host(void* dst, const void* src, size_t bytes, hipStream_t s)
    {
        char* const buf = serves(dst, bytes, s) ? PinnedPool::get().take() : nullptr;
        if (!buf) return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        const hipError_t res = segments(bytes, [=](int w, size_t lo, size_t hi) {
            const size_t chunk = chunk_of(hi - lo), n = (hi - lo + chunk - 1) / chunk;
            for (size_t i = 0; i < n + SLOTS; ++i) {
                char* const slot = buf + (w * SLOTS + i % SLOTS) * CHUNK;
                if (i >= SLOTS && i - SLOTS < n) { // the chunk sent for before in this slot
                    const size_t at = lo + (i - SLOTS) * chunk;
                    const hipError_t e = hipEventSynchronize(ev_[w][i % SLOTS]);
                    if (e != hipSuccess) return e;
                    std::memcpy((char*)dst + at, slot, std::min(chunk, hi - at));
                }
                if (i < n) {
                    const size_t at = lo + i * chunk;
                    hipError_t e = hipMemcpyAsync(slot, (const char*)src + at, std::min(chunk, hi - at),
                                                  hipMemcpyDeviceToHost, s);
                    if (e == hipSuccess) e = hipEventRecord(ev_[w][i % SLOTS], s);
                    if (e != hipSuccess) return e;
                }
            }
            return hipSuccess;
        });
        if (res != hipSuccess) (void)hipStreamSynchronize(s); // nothing writes the buffer any more
        PinnedPool::get().give(buf);
        return res;
    }
    void release()
    {
        for (auto& w : ev_)
            for (hipEvent_t& e : w) {
                if (e) (void)hipEventDestroy(e);
                e = nullptr;
            }
        if (ready_) PinnedPool::get().leave();
        ready_ = false;
    }

private:
    static constexpr size_t CHUNK = (size_t)2 << 20, SLOTS = 2, WORKERS = 2, UNIT = (size_t)1 << 20;
    // from where on it gains (us, the runtime's copy : this: 1.05 MB 87 : 127, 1.9
    // MB 128 : 150, 2.4 MB 164 : 163, 3.7 MB 224 : 191)
    static constexpr size_t LEAST = (size_t)9 << 18;
    static_assert(CHUNK * SLOTS * WORKERS <= PinnedPool::BYTES, "slots of all workers");
    // a few chunks per segment, in whole pages: enough to overlap, few enough
    // that the 10 us each takes the host to enqueue do not count
    static size_t chunk_of(size_t bytes)
    {
        return std::min(CHUNK, (std::max(bytes / 4, UNIT / 4) + 4095) & ~(size_t)4095);
    }
    // fn(worker, first byte, end) over segments of [0, bytes), side by side
    template <class Fn> hipError_t segments(size_t bytes, Fn&& fn)
    {
        const size_t n = std::min<size_t>(bytes / (4 * UNIT) + 1, WORKERS);
        const size_t len = (bytes / n + 4095) & ~(size_t)4095;
        hipError_t res[WORKERS] = {};
        int dev = 0;
        res[0] = hipGetDevice(&dev);
        if (res[0] != hipSuccess) return res[0];
        std::thread th[WORKERS];
        for (size_t w = 1; w < n; ++w) {
            auto part = [&, w] { res[w] = fn((int)w, w * len, w + 1 < n ? (w + 1) * len : bytes); };
            try {
                th[w] = std::thread([&, w, part] {
                    res[w] = hipSetDevice(dev);
                    if (res[w] == hipSuccess) part();
                });
            } catch (...) { // no thread to be had
                part();
            }
        }
        res[0] = fn(0, 0, n > 1 ? len : bytes);
        for (size_t w = 1; w < n; ++w)
            if (th[w].joinable()) th[w].join();
        for (const hipError_t e : res)
            if (e != hipSuccess) return e;
        return hipSuccess;
    }
    bool serves(const void* host, size_t bytes, hipStream_t s)
    {
        if (bytes < LEAST || off_) return false;
        // events have to be of the stream's device
        hipDevice_t of = 0;
        int dev = 0;
        if (hipStreamGetDevice(s, &of) != hipSuccess || hipGetDevice(&dev) != hipSuccess || of != dev) {
            (void)hipGetLastError();
            return false;
        }
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, host) == hipSuccess) {
            if (a.type != hipMemoryTypeUnregistered) return false;
        } else {
            (void)hipGetLastError(); // memory that the runtime does not know
        }
        if (ready_) return true;
        bool ok = true;
        for (auto& w : ev_)
            for (hipEvent_t& e : w) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
        if (ok) {
            PinnedPool::get().join();
            ready_ = true;
        } else {
            (void)hipGetLastError();
            release();
            off_ = true;
        }
        return ok;
    }
    hipEvent_t ev_[WORKERS][SLOTS] = {};
    bool ready_ = false;
    bool off_ = false; // no events: the runtime's copies
};

} // namespace lbm

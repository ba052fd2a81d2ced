// lbm_host.hpp -- host-side helpers shared by the simulation context and the
// serving engine.
#pragma once

#include <algorithm>
#include <cstring>
#include <string>
#include <thread>

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
    return hipStreamIsCapturing(s, &st) == hipSuccess && st == hipStreamCaptureStatusActive;
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

// Copies from the device to pageable host memory through pinned chunks, the
// host's copy of one beside the transfer of the next, in two segments by two
// threads.  The runtime's own pageable copy takes 1200 us for 21.6 MB (18 GB/s)
// where the transfer to pinned memory takes 385; here 680 (one thread 825: it
// reads what the transfer left in memory; three and more the same as two), and
// into memory not touched before 1100 instead of 2200 (one thread).  The
// runtime's copies to the device (580 us) did not gain this way.  One ring per
// simulation, 8 MiB from its first large copy on.  Pinned and device memory,
// and copies too small to gain, go straight to the runtime.
class HostRing {
public:
    // src (device) -> dst; on return the data is in dst, or the copy is
    // enqueued on s
    hipError_t to_host(void* dst, const void* src, size_t bytes, hipStream_t s)
    {
        if (!serves(dst, bytes)) return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
        return segments(bytes, [=](int w, size_t lo, size_t hi) {
            const size_t chunk = chunk_of(hi - lo), n = (hi - lo + chunk - 1) / chunk;
            for (size_t i = 0; i < n + SLOTS; ++i) {
                if (i >= SLOTS && i - SLOTS < n) { // the chunk sent for before in this slot
                    const size_t at = lo + (i - SLOTS) * chunk;
                    const hipError_t e = hipEventSynchronize(ev_[w][i % SLOTS]);
                    if (e != hipSuccess) return e;
                    std::memcpy((char*)dst + at, slot(w, i), std::min(chunk, hi - at));
                }
                if (i < n) {
                    const size_t at = lo + i * chunk;
                    hipError_t e = hipMemcpyAsync(slot(w, i), (const char*)src + at, std::min(chunk, hi - at),
                                                  hipMemcpyDeviceToHost, s);
                    if (e == hipSuccess) e = hipEventRecord(ev_[w][i % SLOTS], s);
                    if (e != hipSuccess) return e;
                }
            }
            return hipSuccess;
        });
    }
    void release()
    {
        for (auto& w : ev_)
            for (hipEvent_t& e : w) {
                if (e) (void)hipEventDestroy(e);
                e = nullptr;
            }
        if (buf_) (void)hipHostFree(buf_);
        buf_ = nullptr;
    }

private:
    static constexpr size_t CHUNK = (size_t)2 << 20, SLOTS = 2, LEAST = (size_t)1 << 20, WORKERS = 2;
    char* slot(int w, size_t i) const { return buf_ + (w * SLOTS + i % SLOTS) * CHUNK; }
    // a few chunks per segment, in whole pages: enough to overlap, few enough
    // that the 10 us each takes the host to enqueue do not count
    static size_t chunk_of(size_t bytes)
    {
        return std::min(CHUNK, (std::max(bytes / 4, LEAST / 4) + 4095) & ~(size_t)4095);
    }
    // fn(worker, first byte, end) over segments of [0, bytes), side by side
    template <class Fn> hipError_t segments(size_t bytes, Fn&& fn)
    {
        const size_t n = std::min<size_t>(bytes / (4 * LEAST) + 1, WORKERS);
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
    bool serves(const void* host, size_t bytes)
    {
        if (bytes < LEAST || off_) return false;
        hipPointerAttribute_t a{};
        if (hipPointerGetAttributes(&a, host) == hipSuccess) {
            if (a.type != hipMemoryTypeUnregistered) return false;
        } else {
            (void)hipGetLastError(); // memory that the runtime does not know
        }
        if (buf_) return true;
        bool ok = hipHostMalloc((void**)&buf_, WORKERS * SLOTS * CHUNK, hipHostMallocDefault) == hipSuccess;
        if (!ok) buf_ = nullptr;
        for (auto& w : ev_)
            for (hipEvent_t& e : w) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            release();
            off_ = true;
        }
        return ok;
    }
    char* buf_ = nullptr;
    hipEvent_t ev_[WORKERS][SLOTS] = {};
    bool off_ = false; // no pinned memory: the runtime's copies
};

} // namespace lbm

// lbm_fused.hpp -- several updates on one read of the lattice: the strip of
// columns that k_fused.hip and the serving kernel walk upwards, and the pieces
// it shares with the tile kernel.
#pragma once

#include "lbm_device.hpp"

namespace lbm {

// Pointers read from memory (request descriptors) are generic; these views let
// loads be global-memory instructions instead of flat ones.
template <class T> using gptr = T __attribute__((address_space(1)))*;
template <class T> __device__ __forceinline__ gptr<const T> as_global(const T* q) { return (gptr<const T>)q; }
template <class T> __device__ __forceinline__ gptr<T> as_global(T* q) { return (gptr<T>)q; }

// Lane l takes the value of lane l - 1 / l + 1 (0 past the wavefront's ends,
// where no valid value is expected).
__device__ __forceinline__ float from_left(float v)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A masked store without a branch: lanes that must not store pass OFF_NONE,
// which lies past the range of the buffer descriptor, and the hardware drops
// it.  (A branch around the stores would make the compiler wait for them
// before it uses the rows loaded ahead.)
constexpr uint32_t OFF_NONE = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(void* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00027000);
}

// The nine stored values of a lane's node, one register each (16-bit values
// undecoded in the low half).  They form 9 / D runs of D consecutive values.
template <int L, class T> struct Stored {
    static constexpr int D = L == L_STREAM ? 1 : (L == L_BUNDLE ? 3 : 9);
    uint32_t v[9];

    __device__ __forceinline__ float get(int i) const
    {
        if constexpr (sizeof(T) == 4)
            return __builtin_bit_cast(float, v[i]);
        else
            return ld(__builtin_bit_cast(T, (uint16_t)v[i]));
    }
    __device__ __forceinline__ void put(int i, T e)
    {
        if constexpr (sizeof(T) == 4)
            v[i] = __builtin_bit_cast(uint32_t, e);
        else
            v[i] = __builtin_bit_cast(uint16_t, e);
    }
    // row: the row's first value of direction 0; off: byte offset of the
    // lane's node in the row; plane: bytes from run to run
    __device__ __forceinline__ void load(gptr<const char> row, int64_t plane, uint32_t off)
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const gptr<const char> a = row + i / D * plane + i % D * (int)sizeof(T) + off;
            if constexpr (sizeof(T) == 4)
                v[i] = *(gptr<const uint32_t>)a;
            else
                v[i] = *(gptr<const uint16_t>)a;
        }
    }
    __device__ __forceinline__ void store(char* row, int64_t plane, uint32_t off) const
    {
#pragma unroll
        for (int r = 0; r < 9 / D; ++r) {
            const __amdgpu_buffer_rsrc_t b = buffer_at(row + r * plane);
            const uint32_t* o = v + r * D;
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int k = 0; k < D; ++k)
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)o[k], b, off + 2 * k, 0, 0);
            } else if constexpr (D == 1) {
                __builtin_amdgcn_raw_buffer_store_b32(o[0], b, off, 0, 0);
            } else if constexpr (D == 3) {
                __builtin_amdgcn_raw_buffer_store_b96(u32x3{o[0], o[1], o[2]}, b, off, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, b, off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[4], o[5], o[6], o[7]}, b, off + 16, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(o[8], b, off + 32, 0, 0);
            }
        }
    }
};

// f rounded to storage with the increments draw(i) decides, as ld(enc(f)) does;
// encoding the result again with st<T> is exact.  FP16C's code is the FP32
// pattern of the scaled magnitude with 12 bits dropped, so a value that stays
// in registers needs no packing and unpacking: 7 instructions per value instead
// of 12.  Values that round to the top code (NaN) are rare; one test per node.
template <class T, int Q = 9, class Rng> __device__ __forceinline__ void round_stored(float* f, const Rng& rng)
{
    if constexpr (std::is_same_v<T, int16_t> || std::is_same_v<T, char16_t>) {
        constexpr uint32_t TOP = 0x07fff000u; // bits of C16_TOP
        uint32_t a[Q], top = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const uint32_t m = c16_scaled(f[i]);
            a[i] = (m + (std::is_same_v<T, int16_t> ? 0x7ff + ((m >> 12) & 1) : rng.draw(i) >> 20)) & 0xfffff000u;
            top = max(top, a[i]);
        }
#pragma unroll
        for (int i = 0; i < Q; ++i)
            f[i] = __builtin_copysignf(__builtin_bit_cast(float, a[i]) * 0x1p112f, f[i]);
        if (__any(top == TOP)) {
            asm volatile("");
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = a[i] == TOP ? __builtin_nanf("") : f[i];
        }
    } else if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < Q; ++i) f[i] = ld(enc<T>(f[i], rng.draw(i)));
    }
}

// a where bit `bit` of the link word is set, else b.
__device__ __forceinline__ float pick(uint32_t lk, int bit, float a, float b)
{
    const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)lk, bit, 1);
    return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, a) & m) | (__builtin_bit_cast(uint32_t, b) & ~m));
}
// Bounce-back: the own value where bit 0 of direction I's kind is set.
template <int I> __device__ __forceinline__ void by_solid(uint32_t lk, float& f, float own) { f = pick(lk, 2 * I, own, f); }
// Clamped source (c_x = -1) or inlet (c_x = +1) where bit 1 is set, after
// by_solid (a clamped source has both bits set).
template <int I> __device__ __forceinline__ void by_side(uint32_t lk, float& f, float v) { f = pick(lk, 2 * I + 1, v, f); }

// Keeps a boundary block behind its (wavefront-uniform) branch: without it the
// compiler runs the selects on every row.
__device__ __forceinline__ void keep_branch() { asm volatile(""); }

// The slot that holds direction i in state kind S.
template <int S> __device__ constexpr int slot(int i) { return S == ST_SWAP ? dir_opp(i) : i; }

// What an update keeps between rows: the started inflow (directions 3..8) of
// the last row it was given and that row's c_y = +1 results.
struct Carry {
    float in[6];
    float north[3];
};

// Stream the results p of row r: f receives the complete inflow of row r - 1
// (link word la), s moves on to row r (link word lb).  fa, fb: some lane's
// word of that row is not 0.  ein: the inlet equilibrium of directions 2, 5,
// 8; inout: the x axis has an inlet and an outlet.
__device__ __forceinline__ void stream_row(const float* ein, bool inout, const float* p, Carry& s, uint32_t la, bool fa,
                                           uint32_t lb, bool fb, float* f)
{
    f[0] = from_right(p[0]);
    f[1] = p[1];
    f[2] = from_left(p[2]);
    if (fa) {
        keep_branch();
        by_solid<0>(la, f[0], s.north[2]);
        by_solid<1>(la, f[1], s.north[1]);
        by_solid<2>(la, f[2], s.north[0]);
        if (inout) {
            keep_branch();
            by_side<0>(la, f[0], p[0]);
            by_side<2>(la, f[2], ein[0]);
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) f[3 + k] = s.in[k];
    s.in[0] = from_right(p[3]);
    s.in[1] = p[4];
    s.in[2] = from_left(p[5]);
    s.in[3] = from_right(s.north[0]);
    s.in[4] = s.north[1];
    s.in[5] = from_left(s.north[2]);
    if (fb) {
        keep_branch();
        by_solid<3>(lb, s.in[0], p[5]);
        by_solid<5>(lb, s.in[2], p[3]);
        by_solid<6>(lb, s.in[3], p[2]);
        by_solid<7>(lb, s.in[4], p[1]);
        by_solid<8>(lb, s.in[5], p[0]);
        if (inout) {
            keep_branch();
            by_side<3>(lb, s.in[0], p[3]);
            by_side<5>(lb, s.in[2], ein[1]);
            by_side<6>(lb, s.in[3], s.north[0]);
            by_side<8>(lb, s.in[5], ein[2]);
        }
    }
    s.north[0] = p[6];
    s.north[1] = p[7];
    s.north[2] = p[8];
}

// kk updates of the nodes in columns x0 .. x0 + 63 - 2 halo of rows y0 .. y1 - 1
// by the calling wavefront, src -> dst.  S: ST_PULL (stored values are
// post-collision results), ST_SWAP (the same, each in the opposite direction's
// slot) or ST_PUSH (streamed values).  1 <= kk <= K, kk <=
// halo and, on a periodic y axis, kk <= ny.  STEP: a block barrier after every
// row (every wavefront of the block walks the same rows).
template <int L, class T, int S, int K, bool STEP>
__device__ __forceinline__ void fused_strip(const KParams& p, const T* src, T* dst, int kk, int halo, int x0, int y0,
                                            int y1)
{
    using R = Stored<L, T>;
    constexpr int E = (int)sizeof(T) * lat_stride<L>();
    const Geometry& g = p.g;
    const int nx = (int)g.nx, ny = (int)g.ny;
    const int lane = (int)threadIdx.x;
    // the lane's column, wrapped on a periodic axis; past any other side the
    // last column stands in (nothing valid is taken from it)
    int x = x0 - halo + lane;
    const bool keep = lane >= halo && lane < 64 - halo && x < nx;
    if (g.xa == AX_PERIODIC) {
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;
    } else {
        x = min(max(x, 0), nx - 1);
    }
    const uint32_t off = (uint32_t)x * (uint32_t)E;
    const bool yper = g.ya == AX_PERIODIC, inout = g.xa == AX_INOUT;
    const bool outlet = g.zh && x == nx - 1;
    const bool fix = __any(outlet); // the pressure outlet lies in this strip
    float omc = p.ph.omc;
    asm volatile("" : "+v"(omc)); // a vector register: the force terms take the scalar operand
    const float ein[3] = {inlet_value(p, 2), inlet_value(p, 5), inlet_value(p, 8)};
    const int64_t pitch = g.px * E;                                // bytes from row to row
    const int64_t plane = (int64_t)R::D * g.P * (int)sizeof(T);    // and from run to run

    // rows y0 - kk .. y1 + kk - 1 enter; a chunk at a closed side starts at it
    const int lo = yper ? y0 - kk : 0; // no row before it is used
    const int ys = max(y0 - kk, lo), ye = y1 + kk;
    auto next_row = [&](int r) { return r + 1 < ny ? r + 1 : (yper ? 0 : ny - 1); };
    int r1 = ys < 0 ? ys + ny : ys; // the row sent for, on the grid (kk <= ny on a periodic axis)
    // link words where a node type is marked irregular (other lanes load
    // nothing and get 0)
    auto links_of = [&](int r, uint32_t type) -> uint32_t {
        return __builtin_amdgcn_raw_buffer_load_b32(buffer_at(const_cast<uint32_t*>(p.links) + (int64_t)r * g.px),
                                                    (type & IRREGULAR) ? (uint32_t)x * 4u : OFF_NONE, 0, 0);
    };
    auto type_of = [&](int r) -> uint32_t { return as_global(p.types + (int64_t)r * g.px)[(uint32_t)x]; };
    Carry s[K] = {};
    uint32_t lk[K + 1] = {}; // link words of rows y, y - 1, ..., y - K
    uint32_t any = 0;        // bit j: some lane's lk[j] is not 0
    R nv;                    // the row sent for, its link words, and the types of the row after it
    nv.load(as_global((const char*)src + r1 * pitch), plane, off);
    uint32_t nlk = links_of(r1, type_of(r1));
    r1 = next_row(r1);
    uint32_t nty = type_of(r1);
    // the row sent for is waited for at the end of a turn, where the stores
    // behind it are counted; at the loop's head, reached also from before the
    // first turn, the compiler would wait for those stores too
    auto take = [&]() {
#pragma unroll
        for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(nv.v[i]));
        asm volatile("" : "+v"(nlk), "+v"(nty));
    };
    take();

#pragma unroll 1
    for (int y = ys; y < ye; ++y) {
        // row y is here; row y + 1 is sent for
        float f[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = nv.get(slot<S>(i));
#pragma unroll
        for (int l = K; l > 0; --l) lk[l] = lk[l - 1];
        lk[0] = nlk;
        any = (any << 1) | (__any(nlk != 0) ? 1u : 0u);
        nv.load(as_global((const char*)src + r1 * pitch), plane, off);
        nlk = links_of(r1, nty);
        r1 = next_row(r1);
        nty = type_of(r1);

        auto fix_outlet = [&]() {
            if (fix) {
                keep_branch();
                if (outlet) outlet_fix(g, nx - 1, f);
            }
        };
        auto collide_row = [&](int j) { // results of row y - j, rounded to storage
            int r = y - j;
            r = r < 0 ? r + ny : (r >= ny ? r - ny : r);
            collide(f, omc, p.ph.F);
            const NodeRng<T> rng((uint32_t)r * (uint32_t)g.px + (uint32_t)x, f);
            round_stored<T>(f, rng);
        };
        if constexpr (S == ST_PUSH) {
            if (any & 1u) {
                keep_branch();
                by_side<2>(lk[0], f[2], ein[0]);
                by_side<5>(lk[0], f[5], ein[1]);
                by_side<8>(lk[0], f[8], ein[2]);
            }
            fix_outlet();
        }
        // Update l + 1 streams then collides (pull form), or collides then
        // streams (push form).  In the first rows of a chunk it has no
        // complete inflow yet: results of update l exist from row
        // max(y0 - kk + l, lo) on.
#pragma unroll
        for (int l = 0; l < K; ++l) {
            if (l >= kk || y - l < max(y0 - kk + l, lo)) break;
            if constexpr (S == ST_PUSH) collide_row(l);
            float q[9];
            stream_row(ein, inout, f, s[l], lk[l + 1], (any >> (l + 1)) & 1u, lk[l], (any >> l) & 1u, q);
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = q[i];
            if (y - l - 1 < max(y0 - kk + l + 1, lo)) break;
            if constexpr (S == ST_PUSH) {
                if (l + 1 < kk) fix_outlet();
            } else {
                fix_outlet();
                collide_row(l + 1);
            }
        }
        R e;
#pragma unroll
        for (int i = 0; i < 9; ++i) e.put(slot<S>(i), st<T>(f[i]));
        const int yo = y - kk;
        if ((any >> kk) & 1u) { // nodes that are not updated hold 0
            keep_branch();
            uint32_t w = lk[1];
#pragma unroll
            for (int l = 2; l <= K; ++l) w = kk == l ? lk[l] : w;
#pragma unroll
            for (int i = 0; i < 9; ++i) e.v[i] = (w & LINK_NONE) ? 0u : e.v[i];
        }
        const bool ok = keep && yo >= y0 && yo < y1;
        e.store((char*)dst + max(yo, 0) * pitch, plane, ok ? off : OFF_NONE);
        take();
        if constexpr (STEP) __builtin_amdgcn_s_barrier();
    }
}

} // namespace lbm

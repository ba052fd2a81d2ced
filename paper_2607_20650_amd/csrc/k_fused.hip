// k_fused.hip -- several lattice updates per launch for the two-lattice
// schemes (LPTL, NPTL, PUSH), every layout and storage precision.
//
// One update per launch is bound by memory: 18 stored values move per node and
// update, about 75 FP32 instructions run on them.  Here a wavefront takes a
// strip of 64 columns and walks it upwards row by row, keeping the rows its
// updates still need in registers, so that kk updates cost one read and one
// write of the lattice:
//
//   row y enters (9 loads), the strip's update 1 completes row y - 1, update 2
//   row y - 2, ..., update kk completes row y - kk, which leaves (9 stores).
//
// An update's result on row r is streamed as soon as it exists: its c_y = -1
// values complete the inflow of row r - 1 (which then collides as the next
// update), its c_y = 0 values and row r - 1's c_y = +1 values start the inflow
// of row r.  Between rows an update therefore keeps nine values: six of a
// started inflow and the three c_y = +1 results still to be streamed.  The +-1
// column shifts are wavefront shifts between lanes (DPP), so no value passes
// through LDS.  The outermost lanes lose one column of validity per update: kk
// columns on each side are recomputed by the neighbouring strip, kk rows above
// and below by the neighbouring chunk.  Every value is computed by the same
// collide() and rounded to the storage precision after every update, so the
// result is bitwise that of kk single updates.
//
// Boundary rules come from the per-node link words: a row with a link word
// that is not 0 in the wavefront takes the selects of stream_row, other rows
// none of them.
#include <algorithm>

#include "lbm_device.hpp"
#include "lbm_edges.hpp"
#include "lbm_kernels.hpp"

namespace lbm {

namespace {

// Most updates per launch of k_fused.  FP32 is bound by memory up to about six
// (8192 x 4096: 502 us per update for single updates, 132 us for 4 per launch,
// 107 for 6, 95 - 102 for 8, where the instructions bound it); the carries
// take 9 registers per update (121 in all for 8, four wavefronts per SIMD).
// 16-bit storage moves half the bytes and spends more instructions on its
// codec, so it is bound by instructions from 4 on and loses to the recomputed
// columns beyond (4096 x 1024 FP16S-SR: 20 us per update for 4, 28 for 8).
template <class T> constexpr int fused_most() { return sizeof(T) == 4 ? 8 : 4; }
// Wavefronts (adjacent strips) per block, kept in step by a barrier per row:
// neighbouring strips share the cache lines at their seams, which without the
// barrier are read from memory again by most of them (a 64-column row starts
// and ends inside a 128-byte line).  8192 x 4096, 4 updates per launch: 176 us
// per update for single wavefronts, 172 for four without, 134 with the barrier.
constexpr int FUSED_WAVES = 4;

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
    __device__ __forceinline__ void load(const char* row, int64_t plane, uint32_t off)
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const char* a = row + i / D * plane + i % D * (int)sizeof(T) + off;
            if constexpr (sizeof(T) == 4)
                v[i] = *reinterpret_cast<const uint32_t*>(a);
            else
                v[i] = *reinterpret_cast<const uint16_t*>(a);
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
template <class T, class Rng> __device__ __forceinline__ void round_stored(float* f, const Rng& rng)
{
    if constexpr (std::is_same_v<T, int16_t> || std::is_same_v<T, char16_t>) {
        constexpr uint32_t TOP = 0x07fff000u; // bits of C16_TOP
        uint32_t a[9], top = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const uint32_t m = c16_scaled(f[i]);
            a[i] = (m + (std::is_same_v<T, int16_t> ? 0x7ff + ((m >> 12) & 1) : rng.draw(i) >> 20)) & 0xfffff000u;
            top = max(top, a[i]);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i)
            f[i] = __builtin_copysignf(__builtin_bit_cast(float, a[i]) * 0x1p112f, f[i]);
        if (__any(top == TOP)) {
            asm volatile("");
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = a[i] == TOP ? __builtin_nanf("") : f[i];
        }
    } else if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = ld(enc<T>(f[i], rng.draw(i)));
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

} // namespace

// S: ST_PULL (stored values are post-collision results) or ST_PUSH (streamed
// values).  kk updates, 1 <= kk <= fused_most<T>() and, on a periodic y axis,
// kk <= ny.
template <int L, class T, int S>
__global__ void __launch_bounds__(64 * FUSED_WAVES, S == ST_PULL || sizeof(T) == 2 ? 4 : 3) k_fused(KParams p, const T* __restrict__ src, T* __restrict__ dst,
                                                            int kk, int rows, int strip_blocks)
{
    using R = Stored<L, T>;
    constexpr int K = fused_most<T>();
    constexpr int E = (int)sizeof(T) * lat_stride<L>();
    const Geometry& g = p.g;
    const int nx = (int)g.nx, ny = (int)g.ny;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(t / (uint32_t)strip_blocks);
    const int strip = (int)(t - (uint32_t)chunk * (uint32_t)strip_blocks) * FUSED_WAVES +
                      (int)__builtin_amdgcn_readfirstlane(threadIdx.y);
    const int x0 = strip * (64 - 2 * kk), y0 = chunk * rows, y1 = min(y0 + rows, ny);
    const int lane = (int)threadIdx.x;
    // the lane's column, wrapped on a periodic axis; past any other side the
    // last column stands in (nothing valid is taken from it)
    int x = x0 - kk + lane;
    const bool keep = lane >= kk && lane < 64 - kk && x < nx;
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
    int r1 = ys < 0 ? ys + ny : ys; // the row sent for, on the grid
    // link words where a node type is marked irregular (other lanes load
    // nothing and get 0)
    auto links_of = [&](int r, uint32_t type) -> uint32_t {
        return __builtin_amdgcn_raw_buffer_load_b32(buffer_at(const_cast<uint32_t*>(p.links) + (int64_t)r * g.px),
                                                    (type & IRREGULAR) ? (uint32_t)x * 4u : OFF_NONE, 0, 0);
    };
    auto type_of = [&](int r) -> uint32_t { return p.types[(int64_t)r * g.px + (uint32_t)x]; };
    Carry s[K] = {};
    uint32_t lk[K + 1] = {}; // link words of rows y, y - 1, ..., y - K
    uint32_t any = 0;        // bit j: some lane's lk[j] is not 0
    R nv;                    // the row sent for, its link words, and the types of the row after it
    nv.load((const char*)src + r1 * pitch, plane, off);
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
        for (int i = 0; i < 9; ++i) f[i] = nv.get(i);
#pragma unroll
        for (int l = K; l > 0; --l) lk[l] = lk[l - 1];
        lk[0] = nlk;
        any = (any << 1) | (__any(nlk != 0) ? 1u : 0u);
        nv.load((const char*)src + r1 * pitch, plane, off);
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
        for (int i = 0; i < 9; ++i) e.put(i, st<T>(f[i]));
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
        __builtin_amdgcn_s_barrier(); // in step with the neighbouring strips (see FUSED_WAVES)
    }
}

// ------------------------------------------------------------------ tiles
// The same updates for small grids: a block holds a tile of 64 columns and
// TILE_ROWS rows, one node per thread, and does kk updates on it; the c_y != 0
// values pass between the rows through LDS (one barrier per update, two
// buffers), the others between lanes.  A launch waits for memory once and for
// one chain of kk collisions, where k_fused waits for rows one after another.
// The tile loses a ring of one node per update, recomputed by its neighbours.
constexpr int TILE_ROWS = 16; // 1024 threads

template <int L, class T, int S>
__global__ void __launch_bounds__(1024) k_fused_tile(KParams p, const T* __restrict__ src, T* __restrict__ dst, int kk,
                                                     int strips)
{
    using R = Stored<L, T>;
    constexpr int E = (int)sizeof(T) * lat_stride<L>();
    __shared__ float smem_tile[2 * 6 * 64 * TILE_ROWS]; // [2][6][rows][64]: directions 0..2 and 6..8
    const Geometry& g = p.g;
    const int nx = (int)g.nx, ny = (int)g.ny;
    constexpr int H = TILE_ROWS;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.y), lane = (int)threadIdx.x;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(t / (uint32_t)strips), strip = (int)(t - (uint32_t)chunk * (uint32_t)strips);
    const int x0 = strip * (64 - 2 * kk), y0 = chunk * (H - 2 * kk), y = y0 - kk + w;
    // column and row wrapped on a periodic axis; past any other side the last
    // ones stand in (nothing valid is taken from them)
    int x = x0 - kk + lane;
    const bool keep = lane >= kk && lane < 64 - kk && x < nx && w >= kk && w < H - kk && y < ny;
    if (g.xa == AX_PERIODIC) {
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;
    } else {
        x = min(max(x, 0), nx - 1);
    }
    int r = y;
    if (g.ya == AX_PERIODIC) {
        if (r < 0 || r >= ny) r = ((r % ny) + ny) % ny;
    } else {
        r = min(max(r, 0), ny - 1);
    }
    const int64_t pitch = g.px * E;
    const int64_t plane = (int64_t)R::D * g.P * (int)sizeof(T);
    const uint32_t off = (uint32_t)x * (uint32_t)E;
    R e;
    e.load((const char*)src + r * pitch, plane, off);
    const uint32_t node = (uint32_t)r * (uint32_t)g.px + (uint32_t)x;
    const uint32_t type = p.types[node];
    const uint32_t lk =
        __builtin_amdgcn_raw_buffer_load_b32(buffer_at(const_cast<uint32_t*>(p.links) + (int64_t)r * g.px),
                                             (type & IRREGULAR) ? (uint32_t)x * 4u : OFF_NONE, 0, 0);
    const bool inout = g.xa == AX_INOUT, outlet = g.zh && x == nx - 1;
    const bool some = __any(lk != 0), fix = __any(outlet);
    const float ein[3] = {inlet_value(p, 2), inlet_value(p, 5), inlet_value(p, 8)};
    float f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = e.get(i);
    auto fix_outlet = [&]() {
        if (fix) {
            keep_branch();
            if (outlet) outlet_fix(g, nx - 1, f);
        }
    };
    auto collide_node = [&]() {
        collide(f, p.ph.omc, p.ph.F);
        const NodeRng<T> rng(node, f);
        round_stored<T>(f, rng);
    };
    if constexpr (S == ST_PUSH) {
        if (some) {
            keep_branch();
            by_side<2>(lk, f[2], ein[0]);
            by_side<5>(lk, f[5], ein[1]);
            by_side<8>(lk, f[8], ein[2]);
        }
        fix_outlet();
    }
    constexpr int row = 64 * H; // values per direction
#pragma unroll 1
    for (int l = 0; l < kk; ++l) {
        if constexpr (S == ST_PUSH) {
            if (w >= l && w <= H - 1 - l) collide_node();
        }
        float* b = smem_tile + (l & 1) * 6 * row + 64 * w + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k) b[k * row] = f[k], b[(3 + k) * row] = f[6 + k];
        __syncthreads();
        // rows up to l past the tile's edge hold no valid inflow any more
        const bool live = w > l && w < H - 1 - l;
        if (!live) continue;
        const float w3 = from_right(f[3]), w5 = from_left(f[5]);
        // a row's neighbours: below (w - 1) for c_y = +1, above for c_y = -1;
        // a column past the tile's edge reads another row's value, unused
        const float n0 = b[64 + 1], n1 = b[row + 64], n2 = b[2 * row + 64 - 1];
        const float n6 = b[3 * row - 64 + 1], n7 = b[4 * row - 64], n8 = b[5 * row - 64 - 1];
        float q[9] = {n0, n1, n2, w3, f[4], w5, n6, n7, n8};
        if (some) {
            keep_branch();
            by_solid<0>(lk, q[0], f[8]);
            by_solid<1>(lk, q[1], f[7]);
            by_solid<2>(lk, q[2], f[6]);
            by_solid<3>(lk, q[3], f[5]);
            by_solid<5>(lk, q[5], f[3]);
            by_solid<6>(lk, q[6], f[2]);
            by_solid<7>(lk, q[7], f[1]);
            by_solid<8>(lk, q[8], f[0]);
            if (inout) {
                keep_branch();
                by_side<0>(lk, q[0], b[64]);
                by_side<2>(lk, q[2], ein[0]);
                by_side<3>(lk, q[3], f[3]);
                by_side<5>(lk, q[5], ein[1]);
                by_side<6>(lk, q[6], b[3 * row - 64]);
                by_side<8>(lk, q[8], ein[2]);
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = q[i];
        if constexpr (S == ST_PUSH) {
            if (l + 1 < kk) fix_outlet();
        } else {
            fix_outlet();
            collide_node();
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) e.put(i, st<T>(f[i]));
    if (lk & LINK_NONE) { // nodes that are not updated hold 0
#pragma unroll
        for (int i = 0; i < 9; ++i) e.v[i] = 0u;
    }
    e.store((char*)dst + r * pitch, plane, keep ? off : OFF_NONE);
}

FusedPlan fused_plan(const KParams& p, int scheme, int layout, int prec)
{
    FusedPlan q;
    const Geometry& g = p.g;
    const int elem = prec == P_FP32 ? 4 : 2;
    const int64_t stride = layout == L_STREAM ? 1 : (layout == L_BUNDLE ? 3 : 9);
    // the Neumann inlet and full-way bounce-back keep the single-update
    // kernels; byte offsets within a row stay below OFF_NONE
    if ((scheme != S_LPTL && scheme != S_NPTL && scheme != S_PUSH) || g.fw || p.rin != nullptr ||
        g.px * stride * elem >= ((int64_t)1 << 30))
        return q;
    auto tiles = [&](int kk) {
        const int w = 64 - 2 * kk, h = TILE_ROWS - 2 * kk;
        return ((g.nx + w - 1) / w) * ((g.ny + h - 1) / h);
    };
    // Small grids: tiles, with as many updates per launch as leave at most one
    // block per CU (128 x 64: 6.1 us per update for single updates, 1.14 us for
    // 7 per launch; 513 x 257: 4.4 and 2.2 us for 3 per launch).  Larger grids
    // stay with 3 up to about 700,000 nodes, beyond which the columns and rows
    // the tiles recompute cost more than the strips' serial rows (1000 x 601:
    // 6.1 against 7.2 us; 1600 x 700: 9.2 against 9.8 us, and 8.1 against 5.3
    // with other simulations beside it).
    if (g.nx * g.ny <= 700000) {
        q.tile = 1;
        q.kk = 3;
        for (int kk : {7, 5, 4})
            if (q.kk == 3 && tiles(kk) <= 256) q.kk = kk;
        return q;
    }
    // FP16C on lattices that fit the 256 MB cache is bound by its codec either
    // way and loses to the recomputed nodes (4096 x 1024: 31 against 28 us per
    // update, FP16C-SR 36 against 31).
    if ((prec == P_FP16C || prec == P_FP16CSR) && 18 * g.P * elem <= ((int64_t)256 << 20)) return q;
    // Strips: chunks of rows that make at most 1024 blocks, four per CU, all
    // resident at once: one round, few recomputed rows at the chunks' ends
    // (4096 x 1024 FP32: 21.4 us per update; 768 blocks 23.0, 512 27.2, 1280
    // 24.1); at most 128 rows.
    q.kk = (int)std::min<int64_t>(prec == P_FP32 ? fused_most<float>() : fused_most<uint16_t>(), g.ny);
    const int64_t w = (int64_t)(64 - 2 * q.kk) * FUSED_WAVES, cols = (g.nx + w - 1) / w;
    const int64_t chunks = std::max<int64_t>(1024 / cols, 1);
    const int64_t rows = (g.ny + chunks - 1) / chunks;
    q.rows = (int)std::min<int64_t>(std::max<int64_t>(rows, 12), 128);
    return q;
}

hipError_t launch_fused(int scheme, int layout, int prec, const KParams& p, const FusedPlan& q, int kk, const void* src,
                        void* dst, hipStream_t s)
{
    if (kk < 1 || kk > q.kk) return hipErrorInvalidValue;
    const int w = 64 - 2 * kk;
    const int64_t cols = q.tile ? (p.g.nx + w - 1) / w : (p.g.nx + w * FUSED_WAVES - 1) / (w * FUSED_WAVES);
    const int rows = q.tile ? TILE_ROWS - 2 * kk : q.rows;
    const int64_t blocks = cols * ((p.g.ny + rows - 1) / rows);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    return with_layout_storage(layout, prec, [&](auto L, auto TT) {
        using T = typename decltype(TT)::type;
        constexpr int LV = decltype(L)::value;
        auto go = [&](auto S) {
            constexpr int SV = decltype(S)::value;
            if (q.tile)
                hipLaunchKernelGGL((k_fused_tile<LV, T, SV>), dim3((uint32_t)blocks), dim3(64, TILE_ROWS),
                                   0, s, p, (const T*)src, (T*)dst, kk, (int)cols);
            else
                hipLaunchKernelGGL((k_fused<LV, T, SV>), dim3((uint32_t)blocks), dim3(64, FUSED_WAVES), 0, s, p,
                                   (const T*)src, (T*)dst, kk, rows, (int)cols);
            return hipGetLastError();
        };
        return scheme == S_PUSH ? go(IC<ST_PUSH>{}) : go(IC<ST_PULL>{});
    });
}

} // namespace lbm

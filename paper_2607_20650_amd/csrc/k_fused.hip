// k_fused.hip -- several lattice updates per launch, every scheme, layout and
// storage precision: from one lattice to another, in the state kind the scheme
// keeps (the one-lattice schemes have a second lattice on grids up to 1.5 GiB;
// AA comes here at even update counts, in its push state).
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

#include "lbm_edges.hpp"
#include "lbm_fused.hpp"
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

} // namespace

template <int L, class T, int S>
__global__ void __launch_bounds__(64 * FUSED_WAVES, S != ST_PUSH || sizeof(T) == 2 ? 4 : 3)
    k_fused(KParams p, const T* __restrict__ src, T* __restrict__ dst, int kk, int rows, int strip_blocks)
{
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(t / (uint32_t)strip_blocks);
    const int strip = (int)(t - (uint32_t)chunk * (uint32_t)strip_blocks) * FUSED_WAVES +
                      (int)__builtin_amdgcn_readfirstlane(threadIdx.y);
    const int y0 = chunk * rows;
    fused_strip<L, T, S, fused_most<T>(), true>(p, src, dst, kk, kk, strip * (64 - 2 * kk), y0,
                                                min(y0 + rows, (int)p.g.ny));
}

// ------------------------------------------------------------------ tiles
// The same updates for small grids: a block holds a tile of 32 x 32 nodes, one
// per thread (two rows per wavefront), and does kk updates on it; the c_y != 0
// values pass between the rows through LDS (one barrier per update, two
// buffers), the others between lanes.  A launch waits for memory once and for
// one chain of kk collisions, where k_fused waits for rows one after another.
// The tile loses a ring of one node per update, recomputed by its neighbours;
// 32 x 32 loses less than 64 x 16 (513 x 257: 1.85 us per update for 4 per
// launch, 2.13 for 3 of 64 x 16).  An update of a tile takes about 0.6 us, the
// VALU issue of 16 wavefronts; a launch 3 - 4 us besides.
constexpr int TILE_X = 32, TILE_ROWS = 32; // 1024 threads

template <int L, class T, int S>
__global__ void __launch_bounds__(1024) k_fused_tile(KParams p, const T* __restrict__ src, T* __restrict__ dst, int kk,
                                                     int strips)
{
    using R = Stored<L, T>;
    constexpr int E = (int)sizeof(T) * lat_stride<L>();
    __shared__ float smem_tile[2 * 6 * TILE_X * TILE_ROWS]; // [2][6][rows][columns]: directions 0..2 and 6..8
    const Geometry& g = p.g;
    const int nx = (int)g.nx, ny = (int)g.ny;
    constexpr int H = TILE_ROWS;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.y), lane = (int)threadIdx.x;
    const int col = lane % TILE_X, line = 2 * w + lane / TILE_X; // of the tile
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(t / (uint32_t)strips), strip = (int)(t - (uint32_t)chunk * (uint32_t)strips);
    const int x0 = strip * (TILE_X - 2 * kk), y0 = chunk * (H - 2 * kk), y = y0 - kk + line;
    // column and row wrapped on a periodic axis; past any other side the last
    // ones stand in (nothing valid is taken from them)
    int x = x0 - kk + col;
    const bool keep = col >= kk && col < TILE_X - kk && x < nx && line >= kk && line < H - kk && y < ny;
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
    const uint32_t off = (uint32_t)r * (uint32_t)pitch + (uint32_t)x * (uint32_t)E;
    R e;
    e.load(as_global((const char*)src), plane, off);
    const uint32_t node = (uint32_t)r * (uint32_t)g.px + (uint32_t)x;
    const uint32_t type = p.types[node];
    const uint32_t lk = __builtin_amdgcn_raw_buffer_load_b32(buffer_at(const_cast<uint32_t*>(p.links)),
                                                             (type & IRREGULAR) ? node * 4u : OFF_NONE, 0, 0);
    const bool inout = g.xa == AX_INOUT, outlet = g.zh && x == nx - 1;
    const bool some = __any(lk != 0), fix = __any(outlet);
    const float ein[3] = {inlet_value(p, 2), inlet_value(p, 5), inlet_value(p, 8)};
    float f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = e.get(slot<S>(i));
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
    constexpr int row = TILE_X * H; // values per direction
#pragma unroll 1
    for (int l = 0; l < kk; ++l) {
        if constexpr (S == ST_PUSH) {
            if (2 * w + 1 >= l && 2 * w <= H - 1 - l) collide_node();
        }
        float* b = smem_tile + (l & 1) * 6 * row + 64 * w + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k) b[k * row] = f[k], b[(3 + k) * row] = f[6 + k];
        __syncthreads();
        // rows up to l from the tile's edge hold no valid inflow any more
        const bool live = 2 * w + 1 > l && 2 * w < H - 1 - l;
        if (!live) continue;
        const float w3 = from_right(f[3]), w5 = from_left(f[5]);
        // a row's neighbours: below for c_y = +1, above for c_y = -1; past the
        // tile's edge another row's or direction's value is read, unused
        constexpr int X = TILE_X;
        const float n0 = b[X + 1], n1 = b[row + X], n2 = b[2 * row + X - 1];
        const float n6 = b[3 * row - X + 1], n7 = b[4 * row - X], n8 = b[5 * row - X - 1];
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
                by_side<0>(lk, q[0], b[X]);
                by_side<2>(lk, q[2], ein[0]);
                by_side<3>(lk, q[3], f[3]);
                by_side<5>(lk, q[5], ein[1]);
                by_side<6>(lk, q[6], b[3 * row - X]);
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
    for (int i = 0; i < 9; ++i) e.put(slot<S>(i), st<T>(f[i]));
    if (lk & LINK_NONE) { // nodes that are not updated hold 0
#pragma unroll
        for (int i = 0; i < 9; ++i) e.v[i] = 0u;
    }
    e.store((char*)dst, plane, keep ? off : OFF_NONE);
}

FusedPlan fused_plan(const KParams& p, int scheme, int layout, int prec)
{
    FusedPlan q;
    const Geometry& g = p.g;
    const int elem = prec == P_FP32 ? 4 : 2;
    const int64_t stride = layout == L_STREAM ? 1 : (layout == L_BUNDLE ? 3 : 9);
    // the Neumann inlet and full-way bounce-back keep the single-update
    // kernels; byte offsets within a row stay below OFF_NONE
    if (g.fw || p.rin != nullptr || g.px * stride * elem >= ((int64_t)1 << 30))
        return q;
    // A call of one update of NPOL or NSOL passes from lattice to lattice here
    // and in place in the scheme's own kernel.  That is the faster one where two
    // lattices no longer stay in the cache: FP32 beyond 3 million nodes (1800 x
    // 1400 NPOL stream 35 us here, 34 there, NSOL 35, 36; 2000 x 1800 65, 45 and
    // 65, 48; 6000 x 3000 330, 299), 16-bit NSOL beyond 256 MB (4096 x 1024 FP16S
    // 37, 40; 5000 x 1200 49, 53; 4096 x 2048 91, 73).  16-bit NPOL has a lean
    // kernel that wins beyond 1.4 million (1600 x 1000 FP16S 19, 16; 4096 x 1024
    // 36, 32; 1000 x 601 10, 11), and in the collision layout 2-byte stores apart
    // from each other cost more than the exchange (700 x 500 FP16S 9.6, 8.0; 4096
    // x 1024 67, 38; 513 x 257 6.6, 7.0).
    if (scheme == S_NPOL || scheme == S_NSOL)
        q.own = elem == 4                 ? g.nx * g.ny > 3000000
                : layout == L_COLLISION   ? g.nx * g.ny > 250000
                : scheme == S_NPOL        ? g.nx * g.ny > 1400000
                                          : 18 * g.P * elem > ((int64_t)256 << 20);
    auto tiles = [&](int kk) {
        const int w = TILE_X - 2 * kk, h = TILE_ROWS - 2 * kk;
        return ((g.nx + w - 1) / w) * ((g.ny + h - 1) / h);
    };
    // Small grids: tiles, with as many updates per launch, up to 12, as leave at
    // most one block per CU (per update, alone: 128 x 64 6.1 us for single
    // updates, 1.14 for 12 per launch; 513 x 257 4.4, 1.85 for 4 per launch).
    // Larger grids stay with 4 up to 1.6 million nodes, beyond which the nodes
    // the tiles recompute cost more than the strips' serial rows (FP32, alone
    // and with two simulations beside: 1000 x 900 5.9, 4.4 against 10.1, 4.5 us
    // in strips; 1600 x 1000 8.5, 8.0 against 12.5, 7.7; 2048 x 2048 in strips
    // 24, 19).
    // Not where most of every tile lies outside: long grids of few rows, by how
    // well the scheme's own kernel takes them (600000 x 1 NPTL FP32 62 us per
    // update in tiles, 19 by single updates; 100000 x 8 NPTL FP32 13, 11, FP16S 14,
    // 10; 100000 x 6 PUSH FP32 13.5, 11.5, AA FP16C-SR 21, 15; 100000 x 4 AA FP16S
    // 14, 14, NPOL FP32 12, 20, FP16S 14, 13; 300000 x 2 NSOL FP16S 38, 29), and
    // columns of one or two nodes with the costly codecs (1 x 100000 FP16C-SR 23,
    // 13).
    const bool codec = elem == 2 && prec != P_FP16S;
    const int few = codec || scheme == S_NPTL || scheme == S_LPTL ? 8
                    : scheme == S_NPOL                            ? (elem == 4 ? 0 : 4)
                    : scheme == S_NSOL                            ? (elem == 4 ? 1 : 2)
                    : elem == 2                                   ? 2
                                                                  : 6;
    if (g.nx * g.ny <= 1600000 && tiles(4) > 1024 && (g.ny <= few || (codec && g.nx <= 2))) return FusedPlan{};
    if (g.nx * g.ny <= 1600000) {
        q.tile = 1;
        const int unit = scheme == S_AA ? 2 : 1; // AA's updates come in pairs
        q.kk = 12;
        while (q.kk > 4 && tiles(q.kk) > 256) q.kk -= unit;
        return q;
    }
    // FP16C on lattices that fit the 256 MB cache is bound by its codec either
    // way and loses to the recomputed nodes where the scheme's own kernel is one
    // of the fast ones (4096 x 1024, FP16C / FP16C-SR: 32 / 36 us per update here;
    // NPTL 28 - 34 / 30 - 34, AA and PUSH stream 33 / 35 us; the others 39 - 62).
    const bool fast = scheme == S_NPTL || ((scheme == S_AA || scheme == S_PUSH) && layout == L_STREAM);
    if ((prec == P_FP16C || prec == P_FP16CSR) && fast && 18 * g.P * elem <= ((int64_t)256 << 20)) return q;
    // Strips: chunks of rows that make at most 1024 blocks, four per CU, all
    // resident at once: one round, few recomputed rows at the chunks' ends
    // (4096 x 1024 FP32: 21.4 us per update; 768 blocks 23.0, 512 27.2, 1280
    // 24.1); whole rounds more where that leaves more than 128 rows (8192 x 4096
    // alone: two rounds 135 us, 1.3 146).  Of the FP32 push form three per CU
    // are resident (4096 x 1024: 768 blocks 24.8, 1024 26.5).
    // FP32 up to 3 million nodes: six updates per launch, where the chunks are
    // so short that the rows recomputed for eight cost more than two launches
    // less (6000 x 400 bundle: 10.6 against 11.2 us per update, alone 14.4
    // against 17.6; 1000 x 2600: 12.8, 13.5; 4096 x 1024: 17.3, 16.7).
    // The FP16S-SR pull spends most on its codec: three, on 1280 blocks.  Beside
    // the fast single updates of NPTL (stream, bundle) that is no gain for a
    // simulation alone, whose lattices stay in the cache, and a large one for
    // several on streams of their own, whose lattices do not (per update alone,
    // and of each of three side by side, strips against single updates: 1300 x
    // 1300 17.6 : 13.8, 13.1 : 13.1; 2048 x 1024 17.2 : 16.0, 13.8 : 13.4; 2500 x
    // 1100 21.8 : 21.8, 17.5 : 29.4; 4096 x 1024 29.8 : 29.5, 22.2 : 37.6).  So
    // from the size on where three no longer fit it together.
    const bool push = scheme == S_PUSH || scheme == S_AA, sr = prec == P_FP16SR && !push;
    if (sr && scheme == S_NPTL && layout != L_COLLISION && g.nx * g.ny <= 2400000) return FusedPlan{};
    const int most = sr                ? 3
                     : prec != P_FP32  ? fused_most<uint16_t>()
                     : g.nx * g.ny <= 3000000 ? 6
                                              : fused_most<float>();
    q.kk = (int)std::min<int64_t>(most, g.ny);
    if (scheme == S_AA) q.kk &= ~1;
    if (q.kk < 2) return FusedPlan{};
    const int64_t resident = sr ? 1280 : (push && prec == P_FP32 ? 768 : 1024);
    const int64_t w = (int64_t)(64 - 2 * q.kk) * FUSED_WAVES, cols = (g.nx + w - 1) / w;
    int64_t rows = INT64_MAX;
    for (int64_t rounds = 1; rows > 128; ++rounds) {
        const int64_t chunks = std::max<int64_t>(resident * rounds / cols, 1);
        rows = (g.ny + chunks - 1) / chunks;
    }
    q.rows = (int)std::max<int64_t>(rows, 12);
    return q;
}

hipError_t launch_fused(int scheme, int layout, int prec, const KParams& p, const FusedPlan& q, int kk, const void* src,
                        void* dst, hipStream_t s)
{
    if (kk < 1 || kk > q.kk) return hipErrorInvalidValue;
    const int w = (q.tile ? TILE_X : 64) - 2 * kk;
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
                hipLaunchKernelGGL((k_fused_tile<LV, T, SV>), dim3((uint32_t)blocks), dim3(64, TILE_X * TILE_ROWS / 64),
                                   0, s, p, (const T*)src, (T*)dst, kk, (int)cols);
            else
                hipLaunchKernelGGL((k_fused<LV, T, SV>), dim3((uint32_t)blocks), dim3(64, FUSED_WAVES), 0, s, p,
                                   (const T*)src, (T*)dst, kk, rows, (int)cols);
            return hipGetLastError();
        };
        if (scheme == S_NSOL) return go(IC<ST_SWAP>{});
        return scheme == S_PUSH || scheme == S_AA ? go(IC<ST_PUSH>{}) : go(IC<ST_PULL>{});
    });
}

} // namespace lbm

// k_d3q19_fused.hip -- two D3Q19 updates per launch, from one lattice to
// another: the pull, and AA in its push state (one even and one odd update),
// in the stream and blocked layouts.
//
// One update per launch is bound by memory: 38 stored values move per node and
// update.  Here a block takes a tile of 64 columns and TILE3_Y rows, two rows
// per wavefront, and walks it through the planes: plane z enters (19 loads per
// node), the first update completes plane z - 1, the second plane z - 2, which
// leaves (19 stores).  Between planes an update keeps 19 values per node in
// registers: 14 of a started inflow (c_z >= 0) and its five c_z = +1 results,
// streamed with the next plane.  Values that move between columns are wavefront
// shifts; those that move between rows pass through LDS (one barrier per
// update, a buffer for each) unless both rows are the thread's own.  The tile
// loses a ring of one node per update, recomputed by its neighbours: 60 x 12
// of 64 x 16 nodes are kept.
//
// Two nodes per thread and 8 wavefronts per CU (226 registers): one node per
// thread and 16 wavefronts need more than the 128 registers they may have.
// Per update, three simulations in turn: 201 x 97 x 85 AA FP32 stream 66 us
// in place one by one, 54 us here; 230 x 140 x 200 FP32 stream pull 257 and
// 184 us; 256^3 FP32 blocked pull 520 and 445 us (alone 512 and 402), where a
// block's plane takes 6 us: 4 us of VALU work (a fifth of it on columns past
// the grid, 256 being 4.3 times 60), the rest exposed loads and stores.  Stores
// of four columns gathered through LDS (10 instead of 38 per plane) lost 20 %.
#include <algorithm>

#include "lbm3_device.hpp"
#include "lbm3_kernels.hpp"
#include "lbm_edges.hpp"
#include "lbm_fused.hpp"

namespace lbm {

namespace {
constexpr int TILE3_X = 64, TILE3_Y = 16;
constexpr int KEPT3_X = TILE3_X - 2 * FUSED3, KEPT3_Y = TILE3_Y - 2 * FUSED3;
} // namespace

// Link words: bit i where direction i's pull source is solid (bounce-back),
// LINK_NONE where the node is not updated.
__global__ void k3_links(Geometry3 g, const uint8_t* __restrict__ types, uint32_t* __restrict__ links)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= g.plane * g.nz) return;
    const uint8_t t = types[n];
    uint32_t w = 0;
    if (!updated(t)) {
        w = LINK_NONE;
    } else if (t & IRREGULAR) {
        const int64_t z = n / g.plane, r = n - z * g.plane, y = r / g.px, x = r - y * g.px;
        for (int i = 0; i < Q3; ++i) {
            int64_t sn;
            if (pull_source3(g, types, x, y, z, i, sn) == K_SOLID) w |= 1u << i;
        }
    }
    links[n] = w;
}

// What an update keeps between planes: the started inflow (directions 5..18)
// of the last plane it was given and that plane's c_z = +1 results.
struct Carry3 {
    float in[14];
    float north[5];
};

// Waits for this wavefront's LDS accesses and meets the block; loads and
// stores of global memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int L, class T, int S>
__global__ void __launch_bounds__(TILE3_X* TILE3_Y / 2) k3_fused(KParams3 p, const T* __restrict__ src,
                                                                 T* __restrict__ dst, int planes, int strips, int tiles)
{
    constexpr int K = FUSED3, R = 2; // updates, rows per thread
    constexpr int E = (int)sizeof(T);
    constexpr int W = TILE3_Y / R, DIR = TILE3_X * W;
    __shared__ float smem_tile3[K * 10 * DIR]; // [update][10][wavefront][64]
    const Geometry3& g = p.g;
    const int nx = (int)g.nx, ny = (int)g.ny, nz = (int)g.nz;
    const int w = (int)__builtin_amdgcn_readfirstlane(threadIdx.y), lane = (int)threadIdx.x;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(t / (uint32_t)tiles), in_plane = (int)(t - (uint32_t)chunk * (uint32_t)tiles);
    const int tile = in_plane / strips, strip = in_plane - tile * strips;
    const int y = tile * KEPT3_Y - K + R * w; // the first row
    const int z0 = chunk * planes, z1 = min(z0 + planes, nz);
    // columns and rows wrapped on a periodic axis; past any other side the last
    // ones stand in (nothing valid is taken from them)
    int x = strip * KEPT3_X - K + lane;
    const bool keep_x = lane >= K && lane < TILE3_X - K && x < nx;
    auto inside = [](int a, int n, bool periodic) {
        if (!periodic) return min(max(a, 0), n - 1);
        return a < 0 || a >= n ? ((a % n) + n) % n : a;
    };
    x = inside(x, nx, g.xa == AX_PERIODIC);
    const bool inout = g.xa == AX_INOUT;
    const bool west = inout && x == 1, east = inout && x == nx - 1;
    const bool side = __any(west || east);
    const int64_t rowp = (L == L_BLOCKED ? g.rstep : g.px) * E;      // bytes from row to row,
    const int64_t planep = (L == L_BLOCKED ? g.pstep : g.plane) * E; // plane to plane
    const int64_t dirp = (L == L_BLOCKED ? 64 : g.P) * E;            // and direction to direction
    const uint32_t xoff = (L == L_BLOCKED ? (uint32_t)(x >> 6) * (Q3 * 64) + (uint32_t)(x & 63) : (uint32_t)x) * E;
    int r[R];
    bool keep[R];
    uint32_t off[R], node[R]; // in the plane: byte offset of the first direction, and node
#pragma unroll
    for (int j = 0; j < R; ++j) {
        r[j] = inside(y + j, ny, g.ya == AX_PERIODIC);
        keep[j] = keep_x && R * w + j >= K && R * w + j < TILE3_Y - K && y + j < ny;
        off[j] = (uint32_t)r[j] * (uint32_t)rowp + xoff;
        node[j] = (uint32_t)r[j] * (uint32_t)g.px + (uint32_t)x;
    }
    float omc = p.ph.omc;
    asm volatile("" : "+v"(omc)); // a vector register: the force terms take the scalar operand
    const bool zper = g.za == AX_PERIODIC;
    const int lo = zper ? z0 - K : 0; // no plane before it is used
    const int zs = max(z0 - K, lo), ze = z1 + K;
    auto wrap_z = [&](int z) { return z < 0 ? z + nz : (z >= nz ? z - nz : z); }; // K <= nz on a periodic axis
    auto next_plane = [&](int z) { return z + 1 < nz ? z + 1 : (zper ? 0 : nz - 1); };

    uint32_t nv[R][Q3], nlk[R], nty[R]; // the plane sent for, its link words, and the types of the plane after it
    auto send = [&](int z, int j) {
        const gptr<const char> a = as_global((const char*)src + z * planep);
#pragma unroll
        for (int i = 0; i < Q3; ++i) {
            if constexpr (E == 4)
                nv[j][i] = *(gptr<const uint32_t>)(a + i * dirp + off[j]);
            else
                nv[j][i] = *(gptr<const uint16_t>)(a + i * dirp + off[j]);
        }
    };
    auto send_links = [&](int z) { // where the type marks the node irregular; other lanes get 0
        const __amdgpu_buffer_rsrc_t b = buffer_at(const_cast<uint32_t*>(p.links) + (int64_t)z * g.plane);
#pragma unroll
        for (int j = 0; j < R; ++j)
            nlk[j] = __builtin_amdgcn_raw_buffer_load_b32(b, (nty[j] & IRREGULAR) ? node[j] * 4u : OFF_NONE, 0, 0);
    };
    auto send_types = [&](int z) {
        const gptr<const uint8_t> a = as_global(p.types + (int64_t)z * g.plane);
#pragma unroll
        for (int j = 0; j < R; ++j) nty[j] = a[node[j]];
    };
    // the plane sent for is waited for at the end of a turn, where the stores
    // behind it are counted
    auto take = [&]() {
#pragma unroll
        for (int j = 0; j < R; ++j) {
#pragma unroll
            for (int i = 0; i < Q3; ++i) asm volatile("" : "+v"(nv[j][i]));
            asm volatile("" : "+v"(nlk[j]), "+v"(nty[j]));
        }
    };
    int zn = wrap_z(zs);
    send_types(zn);
    send(zn, 0);
    send(zn, 1);
    send_links(zn);
    zn = next_plane(zn);
    send_types(zn);
    // rows that no kept row needs: meet the block only
    if (y >= ny + K) {
        for (int z = zs; z < ze; ++z) {
#pragma unroll
            for (int l = 0; l < K; ++l) lds_barrier();
        }
        return;
    }
    Carry3 s[K][R] = {};
    uint32_t lk[R][K + 1] = {}; // link words of planes z, z - 1, ..., z - K
    uint32_t any = 0;           // bit l: some lane's lk[.][l] is not 0
    take();

    // In the first planes of a chunk the updates work on incomplete inflows,
    // whose results no kept node takes.
#pragma unroll 1
    for (int z = zs; z < ze; ++z) {
        float f[R][Q3];
#pragma unroll
        for (int j = 0; j < R; ++j) {
#pragma unroll
            for (int i = 0; i < Q3; ++i) {
                if constexpr (E == 4)
                    f[j][i] = __builtin_bit_cast(float, nv[j][i]);
                else
                    f[j][i] = ld(__builtin_bit_cast(T, (uint16_t)nv[j][i]));
            }
#pragma unroll
            for (int l = K; l > 0; --l) lk[j][l] = lk[j][l - 1];
            lk[j][0] = nlk[j];
        }
        any = (any << 1) | (__any((nlk[0] | nlk[1]) != 0) ? 1u : 0u);
        auto send_rest = [&]() {
            send(zn, 1);
            send_links(zn);
            zn = next_plane(zn);
            send_types(zn);
        };
        auto collide_plane = [&](int l) { // results of plane z - l, rounded to storage
            const uint32_t zr = (uint32_t)wrap_z(z - l) * (uint32_t)ny;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                collide3(f[j], omc, p.ph.F);
                const NodeRng<T, Q3> rng((zr + (uint32_t)r[j]) * (uint32_t)nx + (uint32_t)x, f[j]);
                round_stored<T, Q3>(f[j], rng);
            }
        };
        // The first row of the next plane is sent for at once.  The pull streams
        // plane z first and sends for the second row then: 38 stores are still
        // on their way, and 63 accesses may be (both rows at once 451 us per
        // update on the 256^3 pull, both after streaming 420, this 402).
        send(zn, 0);
        if constexpr (S == ST_PUSH) {
            send_rest();
            if (side) { // values fed by the inlet
                keep_branch();
#pragma unroll
                for (int j = 0; j < R; ++j) {
#pragma unroll
                    for (int i = 0; i < Q3; ++i)
                        if (q3_cx(i) == 1) f[j][i] = west && !((lk[j][0] >> i) & 1u) ? inlet3(p, i) : f[j][i];
                }
            }
        }
#pragma unroll
        for (int l = 0; l < K; ++l) {
            if constexpr (S == ST_PUSH) collide_plane(l);
            // stream the results f of plane z - l: between the thread's two
            // rows in registers, to the rows beyond them through LDS
            float* const b = smem_tile3 + l * 10 * DIR + w * TILE3_X + lane;
            Carry3* const c = s[l];
            const float* const fa = f[0];
            const float* const fb = f[1];
            b[0 * DIR] = fa[0];
            b[1 * DIR] = fa[5];
            b[2 * DIR] = fa[6];
            b[3 * DIR] = fa[7];
            b[4 * DIR] = c[0].north[0];
            b[5 * DIR] = fb[4];
            b[6 * DIR] = fb[11];
            b[7 * DIR] = fb[12];
            b[8 * DIR] = fb[13];
            b[9 * DIR] = c[1].north[4];
            lds_barrier();
            // a row past the tile's edge reads another direction's values, unused
            const float* const up = b + TILE3_X;
            const float* const down = b + 5 * DIR - TILE3_X;
            float q[R][Q3], in[R][14];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const float* const o = f[j ^ 1]; // the thread's other row
                q[j][0] = j ? up[0] : o[0];
                q[j][1] = from_right(f[j][1]);
                q[j][2] = f[j][2];
                q[j][3] = from_left(f[j][3]);
                q[j][4] = j ? o[4] : down[0];
#pragma unroll
                for (int k = 0; k < 14; ++k) q[j][5 + k] = c[j].in[k];
                in[j][0] = j ? up[DIR + 1] : from_right(o[5]);
                in[j][1] = j ? up[2 * DIR] : o[6];
                in[j][2] = j ? up[3 * DIR - 1] : from_left(o[7]);
                in[j][3] = from_right(f[j][8]);
                in[j][4] = f[j][9];
                in[j][5] = from_left(f[j][10]);
                in[j][6] = j ? from_right(o[11]) : down[DIR + 1];
                in[j][7] = j ? o[12] : down[2 * DIR];
                in[j][8] = j ? from_left(o[13]) : down[3 * DIR - 1];
                in[j][9] = j ? up[4 * DIR] : c[1].north[0];
                in[j][10] = from_right(c[j].north[1]);
                in[j][11] = c[j].north[2];
                in[j][12] = from_left(c[j].north[3]);
                in[j][13] = j ? c[0].north[4] : down[4 * DIR];
            }
            if (side) { // zero-gradient outlet and inlet; solid sources below
                keep_branch();
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    q[j][1] = east ? f[j][1] : q[j][1];
                    in[j][0] = east ? (j ? up[DIR] : fb[5]) : in[j][0];
                    in[j][3] = east ? f[j][8] : in[j][3];
                    in[j][6] = east ? (j ? fa[11] : down[DIR]) : in[j][6];
                    in[j][10] = east ? c[j].north[1] : in[j][10];
                    q[j][3] = west ? inlet3(p, 3) : q[j][3];
                    in[j][2] = west ? inlet3(p, 7) : in[j][2];
                    in[j][5] = west ? inlet3(p, 10) : in[j][5];
                    in[j][8] = west ? inlet3(p, 13) : in[j][8];
                    in[j][12] = west ? inlet3(p, 17) : in[j][12];
                }
            }
            if ((any >> (l + 1)) & 1u) {
                keep_branch();
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int i = 0; i < 5; ++i) q[j][i] = pick(lk[j][l + 1], i, c[j].north[4 - i], q[j][i]);
            }
            if ((any >> l) & 1u) {
                keep_branch();
#pragma unroll
                for (int j = 0; j < R; ++j)
#pragma unroll
                    for (int i = 5; i < Q3; ++i)
                        if (i != 9) in[j][i - 5] = pick(lk[j][l], i, f[j][18 - i], in[j][i - 5]);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
#pragma unroll
                for (int k = 0; k < 5; ++k) c[j].north[k] = f[j][14 + k];
#pragma unroll
                for (int k = 0; k < 14; ++k) c[j].in[k] = in[j][k];
#pragma unroll
                for (int i = 0; i < Q3; ++i) f[j][i] = q[j][i];
            }
            if constexpr (S != ST_PUSH) {
                if (l == 0) send_rest();
                collide_plane(l + 1);
            }
        }
        const int zo = z - K;
        const bool here = zo >= z0 && zo < z1;
        char* const o = (char*)dst + max(zo, 0) * planep;
        uint32_t at[R];
#pragma unroll
        for (int j = 0; j < R; ++j) at[j] = here && keep[j] && !(lk[j][K] & LINK_NONE) ? off[j] : OFF_NONE;
#pragma unroll
        for (int i = 0; i < Q3; ++i) {
            const __amdgpu_buffer_rsrc_t b = buffer_at(o + i * dirp);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const T e = st<T>(f[j][i]);
                if constexpr (E == 4)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, e), b, at[j], 0, 0);
                else
                    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, e), b, at[j], 0, 0);
            }
        }
        take();
    }
}

hipError_t launch3_links(const Geometry3& g, const uint8_t* types, uint32_t* links, hipStream_t s)
{
    hipLaunchKernelGGL(k3_links, dim3((uint32_t)((g.plane * g.nz + 255) / 256)), dim3(256), 0, s, g, types, links);
    return hipGetLastError();
}

bool fused3_serves(const Geometry3& g, int scheme, int layout, int prec)
{
    // While the lattices stay in the cache, single updates hold out: a block's
    // planes come one after another, and small grids leave CUs without a block.
    // FP32 from 1.5 million nodes on, where duct and periodic box, pull and AA
    // gain (us per update here : single updates, alone, and of each of three side
    // by side; pull in the stream layout, then AA: 201 x 97 x 85 duct 49 : 63, 46
    // : 64 and 54 : 55, 52 : 66, box 44 : 60, 48 : 59 and 46 : 51, 50 : 58).
    // Below, some lose what others gain: 128 x 112 x 100 duct 45 : 47, 41 : 50 and
    // 48 : 42, 46 : 49, box 43 : 44, 42 : 42 and 46 : 35, 45 : 38; 128 x 96 x 96
    // duct 38 : 41, 35 : 41 and 40 : 36, 38 : 44, box 36 : 39, 37 : 36 and 39 : 30,
    // 39 : 34.
    // Grids that leave most of every tile, or of a chunk's planes with the four
    // around it, outside stay with single updates: fewer than 6 rows (as above:
    // 1250 x 1 x 1250 box 136 : 49, 133 : 47 and 139 : 41, 136 : 46; 700 x 4 x 600
    // duct 63 : 53, 59 : 53 and 69 : 45, 62 : 52; 500 x 8 x 420 46 : 53, 45 : 54
    // and 48 : 45, 49 : 53), fewer than 3 planes (900 x 900 x 2 box 66 : 56, 66 :
    // 55 and 68 : 46, 68 : 51; 900 x 600 x 3 51 : 56, 53 : 56 and 53 : 45, 56 : 50)
    // and, in the stream layout, rows of fewer than 24 nodes (16 x 320 x 320 box
    // 101 : 48, 108 : 46 and 108 : 40, 119 : 48; 24 x 300 x 250 93 : 94, 92 : 126
    // and 100 : 91, 98 : 100); the blocked layout pads such rows for both.
    // Periodic rows of 32 or 64 nodes stay with single updates at any size, and
    // those of 128 but for the stream pull: they fill whole wavefronts there, and
    // 60 columns kept of 64 make two strips of 64, three of 128 (box; pull in the
    // stream layout, in the blocked one, then AA: 32 x 256 x 256 70 : 63, 68 : 62
    // and 69 : 60, 69 : 60 and 75 : 50, 74 : 65; 64 x 160 x 160 54 : 48, 49 : 46
    // and 51 : 44, 49 : 44 and 56 : 39, 53 : 45; 64 x 256 x 256 135 : 120, 118 :
    // 123 and 123 : 111, 112 : 112 and 145 : 110, 127 : 123; 128^3 68 : 68, 61 : 69
    // and 63 : 55, 57 : 57 and 72 : 51, 65 : 65).  With an inlet and an outlet two
    // wavefronts of such a row take the boundary path, and beside others most gain
    // (128^3 duct 66 : 68, 62 : 82 and 64 : 60, 59 : 71 and 72 : 60, 64 : 77).
    // 16-bit storage makes two updates per launch bound by its codec: it gains
    // where the x axis is not periodic, so that two of a row's few wavefronts hold
    // boundary nodes in single updates, from 2 million nodes on (FP16S, AA: 160 x
    // 130 x 128 86 / 73 against 61 / 70), the costlier formats from 4 (FP16S-SR
    // pull: 160 x 130 x 128 70 / 64 against 74 / 82, 230 x 140 x 200 181 / 181
    // against 143 / 156); 256^3 all periodic FP16S 258 against 322 alone.
    // The kernel's byte offsets within a plane stay below OFF_NONE.  The
    // collision layout keeps its staged kernels: a wavefront's load of one
    // direction is not one run there.
    static_assert(FUSED3 <= 3, "a block's planes wrap around a periodic z axis once");
    if (g.ny < 6 || g.nz < 3 || (layout == L_STREAM && g.nx < 24)) return false;
    if (g.xa == AX_PERIODIC) {
        const bool stream_pull = scheme != S_AA && layout == L_STREAM;
        if (prec != P_FP32 || g.nx == 32 || g.nx == 64 || (g.nx == 128 && !stream_pull)) return false;
    }
    const int64_t least = prec == P_FP32 ? 1500000 : prec == P_FP16S ? 2000000 : 4000000;
    const int64_t plane = (layout == L_BLOCKED ? g.pstep : g.plane) * (prec == P_FP32 ? 4 : 2);
    return layout != L_COLLISION && g.nx * g.ny * g.nz >= least && plane < ((int64_t)1 << 30) && g.plane < ((int64_t)1 << 28);
}

hipError_t launch3_fused(int scheme, int layout, int prec, const KParams3& p, const void* src, void* dst, hipStream_t s)
{
    if (!p.links || !fused3_serves(p.g, scheme, layout, prec)) return hipErrorInvalidValue;
    const Geometry3& g = p.g;
    const int64_t strips = (g.nx + KEPT3_X - 1) / KEPT3_X, tiles = strips * ((g.ny + KEPT3_Y - 1) / KEPT3_Y);
    // Chunks of planes: rounds of 256 blocks, one per CU, times the planes a
    // block walks.
    int64_t planes = g.nz, best = INT64_MAX;
    for (int64_t chunks = 1; chunks <= 64; ++chunks) {
        const int64_t n = (g.nz + chunks - 1) / chunks;
        if (n < 4 && chunks > 1) break;
        const int64_t cost = (tiles * ((g.nz + n - 1) / n) + 255) / 256 * (n + 2 * FUSED3);
        if (cost < best) best = cost, planes = n;
    }
    const int64_t blocks = tiles * ((g.nz + planes - 1) / planes);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    return with_storage(prec, [&](auto TT) {
        using T = typename decltype(TT)::type;
        auto go = [&](auto L, auto S) {
            hipLaunchKernelGGL((k3_fused<decltype(L)::value, T, decltype(S)::value>), dim3((uint32_t)blocks),
                               dim3(TILE3_X, TILE3_Y / 2), 0, s, p, (const T*)src, (T*)dst, (int)planes, (int)strips,
                               (int)tiles);
            return hipGetLastError();
        };
        if (layout == L_BLOCKED)
            return scheme == S_AA ? go(IC<L_BLOCKED>{}, IC<ST_PUSH>{}) : go(IC<L_BLOCKED>{}, IC<ST_PULL>{});
        return scheme == S_AA ? go(IC<L_STREAM>{}, IC<ST_PUSH>{}) : go(IC<L_STREAM>{}, IC<ST_PULL>{});
    });
}

} // namespace lbm

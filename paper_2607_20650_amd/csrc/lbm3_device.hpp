// lbm3_device.hpp -- device code shared by the D3Q19 kernels: slot indices of
// the layouts, the collision and the pull sources.
#pragma once

#include <type_traits>

#include "lbm3.hpp"
#include "lbm_device.hpp"

namespace lbm {

// ------------------------------------------------------------------ layouts
// stream (SoA): i * P + n      collision (AoS): 19 n + i
// blocked (AoSoA): rows are cut into blocks of 64 nodes (the row pitch is a
// multiple of 64) and a block stores its 19 directions one after the other,
// 64 nodes each: ((n / 64) 19 + i) 64 + n mod 64.  A wavefront's load of one
// direction stays one contiguous run as in SoA, but all 19 directions of a
// block share a few DRAM pages, so an update touches 9 source rows and 1
// destination region instead of 19 + 19 separate planes.
template <int L> __device__ __forceinline__ int64_t lat3(int i, int64_t n, int64_t P)
{
    if constexpr (L == L_STREAM)
        return (int64_t)i * P + n;
    else if constexpr (L == L_BLOCKED)
        return (((n >> 6) * Q3 + i) << 6) + (n & 63);
    else
        return (int64_t)Q3 * n + i;
}

// ------------------------------------------------------------------ collision
// Weights 1/3, 1/18, 1/36; first-moment constants t_i = 3 w_i with t_edge
// the float nearest 1/12 and t_axis = (1 - 8 t_edge) / 2 (both exact), so
// that 2 t_axis + 8 t_edge == 1 exactly along every axis; 9/2 w_i is exact.
constexpr float W3_REST = 1.0f / 3.0f;
constexpr float W3_AXIS = 1.0f / 18.0f;
constexpr float W3_EDGE = 1.0f / 36.0f;
constexpr float T3_EDGE = 1.0f / 12.0f;
constexpr float T3_AXIS = (1.0f - 8.0f * T3_EDGE) / 2.0f;
constexpr float H3_AXIS = 0.25f;
constexpr float H3_EDGE = 0.125f;

template <int I> __device__ __forceinline__ float c_dot3(float jx, float jy, float jz)
{
    constexpr int X = q3_cx(I), Y = q3_cy(I), Z = q3_cz(I);
    float s = 0.0f;
    bool first = true;
    if constexpr (X != 0) {
        s = X > 0 ? jx : -jx;
        first = false;
    }
    if constexpr (Y != 0) {
        s = first ? (Y > 0 ? jy : -jy) : (Y > 0 ? s + jy : s - jy);
        first = false;
    }
    if constexpr (Z != 0) s = first ? (Z > 0 ? jz : -jz) : (Z > 0 ? s + jz : s - jz);
    return s;
}

template <int I> __device__ __forceinline__ float feq3_shifted(float base, float jx, float jy, float jz)
{
    constexpr int C2 = q3_c2(I);
    if constexpr (C2 == 0) {
        return W3_REST * base;
    } else {
        const float cu = c_dot3<I>(jx, jy, jz);
        if constexpr (C2 == 1)
            return __builtin_fmaf(W3_AXIS, base, cu * __builtin_fmaf(H3_AXIS, cu, T3_AXIS));
        else
            return __builtin_fmaf(W3_EDGE, base, cu * __builtin_fmaf(H3_EDGE, cu, T3_EDGE));
    }
}

template <int I>
__device__ __forceinline__ void relax3(float* f, float base, float jx, float jy, float jz, float omc, const float* F)
{
    const float e = feq3_shifted<I>(base, jx, jy, jz);
    f[I] = e + __builtin_fmaf(omc, f[I] - e, F[I]);
}

template <int... Is>
__device__ __forceinline__ void relax3_all(float* f, float base, float jx, float jy, float jz, float omc,
                                           const float* F, std::integer_sequence<int, Is...>)
{
    (relax3<Is>(f, base, jx, jy, jz, omc, F), ...);
}

// Moments of shifted populations in a fixed order (collide3 and readouts).
__device__ __forceinline__ void moments3(const float* f, float& rho, float& jx, float& jy, float& jz)
{
    rho = ((((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]))) +
           (((f[8] + f[9]) + (f[10] + f[11])) + ((f[12] + f[13]) + (f[14] + f[15])))) +
          ((f[16] + f[17]) + f[18]);
    jx = (((f[3] + f[7]) + (f[10] + f[13])) + f[17]) - (((f[1] + f[5]) + (f[8] + f[11])) + f[15]);
    jy = (((f[4] + f[11]) + (f[12] + f[13])) + f[18]) - (((f[0] + f[5]) + (f[6] + f[7])) + f[14]);
    jz = (((f[14] + f[15]) + (f[16] + f[17])) + f[18]) - (((f[0] + f[1]) + (f[2] + f[3])) + f[4]);
}

// In: shifted incoming populations.  Out: shifted post-collision values.
__device__ __forceinline__ void collide3(float* f, float omc, const float* F)
{
    float rho, jx, jy, jz;
    moments3(f, rho, jx, jy, jz);
    const float jj = __builtin_fmaf(jx, jx, __builtin_fmaf(jy, jy, jz * jz));
    const float base = __builtin_fmaf(-1.5f, jj, rho);
    relax3_all(f, base, jx, jy, jz, omc, F, std::make_integer_sequence<int, Q3>{});
}

// ------------------------------------------------------------------ sources
// Pull source of direction i for node (x, y, z): (x, y, z) - c_i after the
// axis rules (periodic wraps, outside a closed side is solid, past the
// outlet the last plane is used).  Returns K_NODE with its index in sn,
// K_SOLID or K_INLET.
__device__ __forceinline__ int pull_source3(const Geometry3& g, const uint8_t* __restrict__ types, int64_t x,
                                            int64_t y, int64_t z, int i, int64_t& sn, int64_t& row)
{
    int64_t sx = x - q3_cx(i), sy = y - q3_cy(i), sz = z - q3_cz(i);
    if (sy < 0 || sy >= g.ny) {
        if (g.ya != AX_PERIODIC) return K_SOLID;
        sy = sy < 0 ? sy + g.ny : sy - g.ny;
    }
    if (sz < 0 || sz >= g.nz) {
        if (g.za != AX_PERIODIC) return K_SOLID;
        sz = sz < 0 ? sz + g.nz : sz - g.nz;
    }
    if (sx < 0 || sx >= g.nx) {
        if (g.xa == AX_PERIODIC)
            sx = sx < 0 ? sx + g.nx : sx - g.nx;
        else if (g.xa == AX_INOUT && sx >= g.nx)
            sx = g.nx - 1;
        else
            return K_SOLID;
    }
    row = sz * g.ny + sy;
    sn = row * g.px + sx;
    const uint8_t t = node_type(types[sn]);
    return t == T_SOLID ? K_SOLID : (t == T_INLET ? K_INLET : K_NODE);
}
__device__ __forceinline__ int pull_source3(const Geometry3& g, const uint8_t* __restrict__ types, int64_t x,
                                            int64_t y, int64_t z, int i, int64_t& sn)
{
    int64_t row;
    return pull_source3(g, types, x, y, z, i, sn, row);
}

__device__ __forceinline__ float inlet3(const KParams3& p, int i)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, p.ph.ein[i])));
}

} // namespace lbm

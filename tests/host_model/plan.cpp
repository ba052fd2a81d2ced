// The plans of grids (fused_plan, fused3_serves of the built library), for
// test_plans_cpu.py.
#include <string>

#include "lbm3_kernels.hpp"
#include "lbm_host.hpp"
#include "lbm_kernels.hpp"

extern "C" int plan_of(const lbm_grid* grid, const lbm_bc* bc, const uint8_t* flags, int32_t out[4])
{
    lbm::KParams p{};
    std::string why;
    if (lbm::setup_params(grid, flags, 0.8, bc, p, why) != LBM_OK) return 1;
    const lbm::FusedPlan q = lbm::fused_plan(p, grid->scheme, grid->layout, grid->precision);
    out[0] = q.kk;
    out[1] = q.tile;
    out[2] = q.rows;
    out[3] = q.own;
    return 0;
}

extern "C" int serves3_of(int64_t nx, int64_t ny, int64_t nz, int xa, int scheme, int layout)
{
    lbm::Geometry3 g{};
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.px = (nx + 15) / 16 * 16;
    g.plane = g.px * ny;
    g.xa = xa;
    g.ya = g.za = lbm::AX_CLOSED;
    return lbm::fused3_serves(g, scheme, layout, lbm::P_FP32);
}

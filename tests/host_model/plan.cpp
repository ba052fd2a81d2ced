// The plan of a grid (fused_plan of the built library), for test_plans_cpu.py.
#include <string>

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

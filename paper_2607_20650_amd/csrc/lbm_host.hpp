// lbm_host.hpp -- host-side helpers shared by the simulation context and the
// serving engine.
#pragma once

#include <string>

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

} // namespace lbm

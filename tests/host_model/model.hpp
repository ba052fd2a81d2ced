// The modelled device: its memory and what has been launched.
#pragma once

#include <algorithm>
#include <cstdint>

#include "lbm_kernels.hpp"

struct Device {
    size_t total = (size_t)288 << 30, free_bytes = (size_t)288 << 30;
    size_t largest = SIZE_MAX; // larger allocations fail
    int faults = 0;            // accesses to memory that is not allocated
    int singles = 0, fused = 0, graph_launches = 0, captures = 0;
};
extern Device dev;
extern lbm::FusedPlan plan; // what fused_plan returns
extern bool serves3;        // what fused3_serves returns

constexpr long BAD = -1000000;
long count_at(const void* p);           // the update count held at a device address
void set_count(const void* p, long t);

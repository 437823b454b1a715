// Grids of more workgroups than one grid dimension holds (plain C++, no HIP).
#pragma once

#include <cstdint>

namespace rs {

// x by y workgroups, y > 1 only where n workgroups of `threads` threads are 2^32 threads or more: a dimension's
// threads are counted in 32 bits, and a launch beyond that is cut short without an error.  Kernels number their
// workgroups y * gridDim.x + x; rows are whole multiples of 8, so that the numbers meet the dies in turn, and up
// to 8 y - 1 workgroups past n find no work.
struct GroupGrid {
    uint32_t x, y;
};

inline GroupGrid group_grid(int64_t n, int threads)
{
    if (n * threads < int64_t(1) << 32) return {(uint32_t)n, 1};
    const int64_t most = ((int64_t(1) << 32) - 1) / threads & ~int64_t(7);
    const int64_t rows = (n + most - 1) / most;
    return {(uint32_t)(((n + rows - 1) / rows + 7) & ~int64_t(7)), (uint32_t)rows};
}

}  // namespace rs

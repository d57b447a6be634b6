// lpv_grid.h -- workgroups of a large launch as a two-dimensional grid (plain
// C++, host side).
#pragma once

#include <stdint.h>

namespace lpv {

// The runtime holds the threads of a grid dimension in 32 bits: 2^32 (2^22 workgroups of
// 1024, 2^24 of 256) are refused, and of more only the remainder runs, without an
// error.  The largest accepted calls have more, so from 2^20 workgroups on the grid has
// several rows: workgroup L = blockIdx.y gridDim.x + blockIdx.x does piece L.  The last
// row may reach past the last piece, so kernels check L.  A row is a multiple of 8:
// workgroup L runs on XCD L % 8 whatever its row.
constexpr int64_t GRID_ROW = (int64_t)1 << 20;

struct Grid2 {
    uint32_t x, y;
};

inline Grid2 grid_of(int64_t workgroups)
{
    if (workgroups <= GRID_ROW)
        return {(uint32_t)workgroups, 1u};
    return {(uint32_t)GRID_ROW, (uint32_t)((workgroups + GRID_ROW - 1) / GRID_ROW)};
}

}  // namespace lpv

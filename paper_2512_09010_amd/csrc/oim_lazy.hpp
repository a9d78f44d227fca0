// Grids of row ids (paper Section 3.2, Algorithm 1, with few tokens leaving a line per pass): shared by the kernels
// that run a pass without moving the tokens (oim_wide_lazy.hip, oim_adjacent.hip).
#pragma once
#include "common.hpp"

namespace luvc {

namespace {

struct LazyGeom {
    int n0;         // tokens per image of the call's input grid: ids below it are rows of x
    int h, w;       // grid before this pass
    int D, axis, m, radius;
    int cap;        // overlay rows per image over the whole call
    int ov_base;    // first overlay row of this pass
    int per_line;   // overlay rows a line of this pass may write: min(m, destinations of the line)
};

template <typename T>
__device__ __forceinline__ const T* row_of(const T* x, const T* ov, int64_t b, int id, const LazyGeom& g, int D)
{
    return id < g.n0 ? x + (b * g.n0 + id) * D : ov + (b * g.cap + (id - g.n0)) * D;
}

}  // namespace

}  // namespace luvc

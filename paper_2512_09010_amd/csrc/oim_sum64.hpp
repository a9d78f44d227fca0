// fp64 sums over a wavefront, eight at a time (paper Section 3.2: the similarity decisions of OIM are taken on fp64 sums).
#pragma once
#include "common.hpp"

namespace luvc {

namespace {

// the value of another lane, by DPP: lane ^ 1, lane ^ 2, lane ^ 7, lane ^ 3, lane ^ 8
__device__ __forceinline__ float dpp_get(float v, const int sel)
{
    const int x = __float_as_int(v);
    switch (sel) {
        case 0: return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true));    // quad_perm [1,0,3,2]: lane ^ 1
        case 1: return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true));    // quad_perm [2,3,0,1]: lane ^ 2
        case 2: return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true));   // row_half_mirror: lane ^ 7
        case 3: return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x1B, 0xf, 0xf, true));    // quad_perm [3,2,1,0]: lane ^ 3
        default: return __int_as_float(__builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true));  // row_ror:8: lane ^ 8
    }
}

__device__ __forceinline__ double dpp_get64(double v, const int sel)
{
    const float lo = dpp_get(__int_as_float(__double2loint(v)), sel), hi = dpp_get(__int_as_float(__double2hiint(v)), sel);
    return __hiloint2double(__float_as_int(hi), __float_as_int(lo));
}

// v + (v of the lane 32 away), then 16 away: lane-swap instructions on both halves of the value
__device__ __forceinline__ double add_far_lanes64(double r)
{
    const uint32_t lo = (uint32_t)__double2loint(r), hi = (uint32_t)__double2hiint(r);
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    r = __hiloint2double((int)h32[0], (int)l32[0]) + __hiloint2double((int)h32[1], (int)l32[1]);
    const uint32_t lo2 = (uint32_t)__double2loint(r), hi2 = (uint32_t)__double2hiint(r);
    const auto l16 = __builtin_amdgcn_permlane16_swap(lo2, lo2, false, false), h16 = __builtin_amdgcn_permlane16_swap(hi2, hi2, false, false);
    return __hiloint2double((int)h16[0], (int)l16[0]) + __hiloint2double((int)h16[1], (int)l16[1]);
}

// Eight or nine wave64 sums at once, that of v[i] in lane i: three exchange steps (lanes 1, 2, 4 apart) after which a
// lane keeps only the partial sum of value (lane & 7), one between the half rows that keeps the ninth in the upper ones, then lanes
// 32 and 16 apart.  Every step adds the partial sums of two lane groups, so all values are summed over the same tree: a sum has
// the same bits in whichever of these places it is formed, which two workgroups that look at one source rely on.
template <int M>
__device__ __forceinline__ double wave_totals64(const double (&v)[M], int lane)
{
    static_assert(M == 8 || M == 9, "");
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    double p[4], q[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double keep = b0 ? v[2 * i + 1] : v[2 * i], send = b0 ? v[2 * i] : v[2 * i + 1];
        p[i] = keep + dpp_get64(send, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double keep = b1 ? p[2 * i + 1] : p[2 * i], send = b1 ? p[2 * i] : p[2 * i + 1];
        q[i] = keep + dpp_get64(send, 1);
    }
    const double keep = b2 ? q[1] : q[0], send = b2 ? q[0] : q[1];
    double r = keep + dpp_get64(dpp_get64(send, 2), 3);             // (lane ^ 7) ^ 3 = lane ^ 4
    if constexpr (M == 9) {
        double t = v[8] + dpp_get64(v[8], 0);
        t += dpp_get64(t, 1);
        t += dpp_get64(dpp_get64(t, 2), 3);
        const double keep = b3 ? t : r, send = b3 ? r : t;
        r = keep + dpp_get64(send, 4);
    } else {
        r += dpp_get64(r, 4);
    }
    return add_far_lanes64(r);
}
// all eight in every lane
__device__ __forceinline__ void wave_total64x8(double (&v)[8], int lane)
{
    const double r = wave_totals64(v, lane);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        v[i] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(r), i), __builtin_amdgcn_readlane(__double2loint(r), i));
}

// the largest value of the wavefront, in every lane (all 64 lanes take part, no NaN)
__device__ __forceinline__ double wave_max64(double v)
{
    v = fmax(v, dpp_get64(v, 0));
    v = fmax(v, dpp_get64(v, 1));
    v = fmax(v, dpp_get64(v, 2));                // lane ^ 7: every quad holds its largest by now
    v = fmax(v, dpp_get64(v, 4));
    const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    v = fmax(__hiloint2double((int)h32[0], (int)l32[0]), __hiloint2double((int)h32[1], (int)l32[1]));
    const uint32_t lo2 = (uint32_t)__double2loint(v), hi2 = (uint32_t)__double2hiint(v);
    const auto l16 = __builtin_amdgcn_permlane16_swap(lo2, lo2, false, false), h16 = __builtin_amdgcn_permlane16_swap(hi2, hi2, false, false);
    return fmax(__hiloint2double((int)h16[0], (int)l16[0]), __hiloint2double((int)h16[1], (int)l16[1]));
}

}  // namespace

}  // namespace luvc

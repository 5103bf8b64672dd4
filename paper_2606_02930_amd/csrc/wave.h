// Wavefront-wide reductions of doubles by DPP lane permutations (sums within
// quads, half rows and rows, then the row broadcasts across the four rows),
// which stay in the vector register file instead of passing through LDS as
// cross-lane shuffles do.
#pragma once

#include <hip/hip_runtime.h>

namespace ite {

// One DPP data movement on both halves of a double; lanes of rows outside
// ROWS receive 0.  (With all rows in ROWS and a control that has a source for
// every lane nothing is left to fill, and no register is zeroed for it.)
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double v) {
    const long long bits = __double_as_longlong(v);
    if constexpr (ROWS == 0xf) {
        const int lo = __builtin_amdgcn_mov_dpp((int)bits, CTRL, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(bits >> 32), CTRL, 0xf, 0xf, true);
        return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    }
    const int lo = __builtin_amdgcn_update_dpp(0, (int)bits, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Value of v in lane `lane` (uniform), returned to every lane.
__device__ inline double lane_value(double v, int lane) {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)bits, lane);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over the 64 lanes, returned to every lane (lane 63 ends with the total).
__device__ inline double wave_sum(double v) {
    v += dpp_move<0xB1, 0xf>(v);     // quad_perm [1, 0, 3, 2]
    v += dpp_move<0x4E, 0xf>(v);     // quad_perm [2, 3, 0, 1]
    v += dpp_move<0x141, 0xf>(v);    // row_half_mirror
    v += dpp_move<0x140, 0xf>(v);    // row_mirror
    v += dpp_move<0x142, 0xa>(v);    // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);    // row_bcast:31 into rows 2 and 3
    return lane_value(v, 63);
}

// Largest value over the 64 lanes of non-negative v, returned to every lane
// (the zeros moved into the rows outside a broadcast's mask leave it as is).
__device__ inline double wave_max_nonneg(double v) {
    v = fmax(v, dpp_move<0xB1, 0xf>(v));
    v = fmax(v, dpp_move<0x4E, 0xf>(v));
    v = fmax(v, dpp_move<0x141, 0xf>(v));
    v = fmax(v, dpp_move<0x140, 0xf>(v));
    v = fmax(v, dpp_move<0x142, 0xa>(v));
    v = fmax(v, dpp_move<0x143, 0xc>(v));
    return lane_value(v, 63);
}

// Exchange of the upper 32 (16 of each half) lanes of a with the lower ones of
// b, both halves of the doubles.
__device__ inline void swap32(double& a, double& b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
    b = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ inline void swap16(double& a, double& b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
    b = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// Sums over the wavefront of eight values at once: lane l returns the sum of
// value sum8_index(l).  Halving the values with every exchange takes 34
// instructions where eight separate sums take 160.
__device__ inline int sum8_index(int lane) { return (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1); }
__device__ inline double sum8(double (&v)[8], int lane) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        swap32(v[j], v[j + 4]);
        v[j] += v[j + 4];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        swap16(v[j], v[j + 2]);
        v[j] += v[j + 2];
    }
    const bool up = lane & 8;
    const double keep = up ? v[1] : v[0], give = up ? v[0] : v[1];
    double s = keep + dpp_move<0x128, 0xf>(give);   // row_ror:8
    s += dpp_move<0x141, 0xf>(s);                   // row_half_mirror
    s += dpp_move<0x4E, 0xf>(s);                    // quad_perm [2, 3, 0, 1]
    s += dpp_move<0xB1, 0xf>(s);                    // quad_perm [1, 0, 3, 2]
    return s;
}

// ---------------------------------------------------------------------------
// One workgroup
// ---------------------------------------------------------------------------

// Exchange and add: lanes 0..31 (of each half 0..15) end with the sum of a over
// the halves, the others with that of b.
__device__ inline double swap_add32(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ inline double swap_add16(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) + __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// 1 / x and 1 / sqrt(x) to rounding for normal x away from the ends of the
// range: the hardware estimate (relative error below 1e-7) and two Newton
// steps.
__device__ inline double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ inline double recip_sqrt(double x) {
    double r = __builtin_amdgcn_rsq(x);
    r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
    return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// The sequence number of a HostPost, after everything this wavefront wrote.
template <typename Post> __device__ inline void post_flag(const Post& p) {
    __hip_atomic_store(p.flag, p.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace ite

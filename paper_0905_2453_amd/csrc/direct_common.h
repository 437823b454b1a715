// Device functions shared by the direct-sum kernels (direct.hip, split.hip): ray coordinates, the lens
// record as the loop reads it, source pixels and the origin of the LDS map window.
#pragma once

#include <limits.h>

#include "rs_internal.h"

namespace rs {

// Coordinate i of a grid axis at offset u in [0, 1) of its cell, FP64 then rounded to float32.
__device__ __forceinline__ float ray_coord(double lo, double t, int64_t i, double u = 0.5)
{
    double v = ((double)i + u) * t;
    double w = lo + v;
    return (float)w;
}

// (The launch's constants `a` below are DirectArgs in any address space.)
// Half-open source pixel of y; returns p2 * n1 + p1, or -1 when the ray is lost.
template <class Args>
__device__ __forceinline__ int pixel_of(double y1, double y2, const Args &a, int &p1, int &p2)
{
    double f1 = floor((y1 - a.mlo1) * a.ms1);
    double f2 = floor((y2 - a.mlo2) * a.ms2);
    if (!(f1 >= 0.0 && f1 < (double)a.mn1 && f2 >= 0.0 && f2 < (double)a.mn2)) return -1;
    p1 = (int)f1;
    p2 = (int)f2;
    return p2 * a.mn1 + p1;
}

// 1 / (1 + mean relative error of v_rcp_f32), the error measured over every float32 mantissa
// in [1, 2) with weight 1/x.
constexpr double kRcpBiasComp = 1.0 + 6.41e-9;

// Ray and lens coordinates enter the lens loop scaled by 2^-4.  The scaling is exact, so every
// rounding is that of the unscaled arithmetic; it keeps the product of four squared distances (four
// rows sharing one reciprocal) in the float32 range for lenses up to about 1e6 from the rays.  The
// sums come out 2^4 times the deflection and are scaled back with the bias compensation.
constexpr float kLoopScale = 0.0625f;
constexpr double kLoopBack = kRcpBiasComp * 0.0625;

// One-column blocks add kQuadRuns consecutive float32 runs in float32 before the FP64 addition:
// one float32 add per run instead of a conversion and an FP64 add, at an error between that of
// single runs and of one run kQuadRuns times as long.
constexpr int kQuadRuns = 4;

// Lens i as the loop reads it: moved to the launch's time, coordinates scaled.
template <class Args>
__device__ __forceinline__ float4 loop_lens(const Args &a, int64_t i)
{
    float4 l = moved_lens(a.lenses[i], a.vel, i, a.time);
    l.x *= kLoopScale;
    l.y *= kLoopScale;
    return l;
}

// Zero-mass padding of the last lens tile: at lens 0's position, so that its squared distances are
// ordinary numbers (products stay finite and its terms are exactly zero); a ray exactly there takes
// the per-ray recomputation below, as a ray on lens 0 does anyway.
template <class Args>
__device__ __forceinline__ float4 pad_lens(const Args &a)
{
    float4 l = loop_lens(a, 0);
    l.z = 0.0f;
    l.w = 0.0f;
    return l;
}

// Window origin from the pixels of 8 sample rays (INT_MIN: lost): the per-axis median, robust to rays
// scattered far by a close lens.  Each lane ranks one sample; the whole wave must call it.
__device__ __forceinline__ void window_origin(const int *c1, const int *c2, int lane, int W, int &o1, int &o2)
{
    const int c = lane & 7, a1 = c1[c], a2 = c2[c];
    int n = 0, k1 = 0, k2 = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int b1 = c1[j], b2 = c2[j];
        const bool in = b1 != INT_MIN;
        n += in;
        k1 += in && (b1 < a1 || (b1 == a1 && j < c));
        k2 += in && (b2 < a2 || (b2 == a2 && j < c));
    }
    const unsigned long long w1 = __ballot(a1 != INT_MIN && k1 == n / 2), w2 = __ballot(a1 != INT_MIN && k2 == n / 2);
    if (n > 0) {
        o1 = __builtin_amdgcn_readlane(a1, __builtin_ctzll(w1)) - W / 2;
        o2 = __builtin_amdgcn_readlane(a2, __builtin_ctzll(w2)) - W / 2;
    }
}

// Counter of lost rays for the i-th workgroup: one of lost_mask + 1, a cache line apart (additions to one
// address complete one after the other, about 12 ns each).
template <class Args>
__device__ __forceinline__ unsigned long long *lost_slot(const Args &a, uint32_t i)
{
    return a.lost + (size_t)(i & a.lost_mask) * kLostStride;
}

// Runs of equal keys among consecutive lanes: true on a run's first lane, with the run's length.
__device__ __forceinline__ bool run_head(int key, int lane, uint32_t &cnt)
{
    const int prev = __shfl_up(key, 1);
    const bool head = (lane == 0) || (key != prev);
    const unsigned long long H = __ballot(head);
    const unsigned long long above = lane == 63 ? 0ull : (H >> (lane + 1));
    const int next = above ? lane + 1 + __builtin_ctzll(above) : 64;
    cnt = (uint32_t)(next - lane);
    return head;
}

}  // namespace rs

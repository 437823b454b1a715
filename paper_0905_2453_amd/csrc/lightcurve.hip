// Light curves from a magnification map: a source profile moved along straight tracks across
// the map, giving at each point the profile-weighted magnification (eq. 4 per pixel) and the
// magnitude change (section 1, the light-curve use of the maps).
#include <algorithm>
#include <cmath>

#include "rs_internal.h"

namespace rs {

namespace {

constexpr int kLcWaves = 4;
constexpr int kLcAxis = 128;   // support bounding-box side staged in LDS per wave of a point
constexpr int kLcAhead = 4;    // pixels requested at once when there are few points

__device__ inline double wave_sum(double v)
{
    for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
    return v;
}

// One wave per track point (SPLIT 1), or one workgroup (SPLIT kLcWaves).  The point's lane l takes the
// bounding-box pixels e = l, l + 64 SPLIT, ... (row-major); each wave reduces in a fixed butterfly order and
// a workgroup adds its waves' sums in order, so a result depends only on its inputs.
// A Gaussian weight is separable, exp(-(d1^2 + d2^2) / 2 s^2) = g(d1) g(d2): the squared offsets and the
// one-axis factors of the box's columns and rows are staged in LDS, leaving one
// product per pixel.  The inclusion test d1^2 + d2^2 <= R^2 uses the same FP64 expressions as the
// plain definition.  Boxes wider than the staging area take the per-pixel path.
//
// Many points: issue; a pixel outside the support is not read (AHEAD 1).  Few points leave a wave or two per
// SIMD and nothing to cover the latency of a pixel's load: AHEAD pixels are requested at once, those outside the
// support with weight zero (2107 points, box 1764: 10.2 us, 8.8 with four ahead), and where there are
// not even waves enough, a workgroup shares a point (300 points, box 1764: 8.5 us, 4.4; box 14884: 47.1, 10.1).
// A point of a workgroup also has four times the staging area: 2107 points, box 58564: 391 us, 90.2 staged.
template <int SPLIT, int AHEAD>
__global__ void __launch_bounds__(64 * kLcWaves) k_light_curve(const LightArgs a)
{
    constexpr int kPoints = kLcWaves / SPLIT, kLanes = 64 * SPLIT;   // points of a workgroup, lanes of a point
    static_assert(SPLIT == 1 || SPLIT == kLcWaves, "a point belongs to a wave or to the workgroup");
    __shared__ double2 s_col[kPoints][kLcAxis * SPLIT];   // (d1^2, g(d1)) per box column
    __shared__ double2 s_row[kPoints][kLcAxis * SPLIT];   // (d2^2, g(d2)) per box row
    __shared__ double s_sum[kLcWaves][2];
    const int lane = threadIdx.x % kLanes, wv = threadIdx.x / kLanes;
    const int64_t gp = group_number() * kPoints + wv;
    const bool active = gp < (int64_t)a.n_tracks * a.n_points;
    int64_t tr = 0;
    int k = 0;
    if (active) {
        if (gp < 0x7fffffff) {
            tr = (uint32_t)gp / (uint32_t)a.n_points;
            k = (int)((uint32_t)gp - (uint32_t)tr * (uint32_t)a.n_points);
        } else {
            tr = gp / a.n_points;
            k = (int)(gp - tr * a.n_points);
        }
    }
    const double *t = a.tracks + 4 * tr;
    const double f = a.n_points > 1 ? (double)k / (double)(a.n_points - 1) : 0.0;
    const double ys1 = t[0] + f * (t[2] - t[0]);
    const double ys2 = t[1] + f * (t[3] - t[1]);
    const double rs = a.support, rs2 = a.support * a.support;
    const double inv2s2 = a.inv2s2;
    const bool gauss = a.kind == 0;
    // Bounding box of the support in pixel indices, clamped to the map.  A pixel inside the
    // support has (p + 1/2) w >= y - R - lo, so p >= floor((y - R - lo) / w) with half a pixel to
    // spare: multiplying by a rounded 1/w cannot push the floor past a pixel that is inside
    // (and symmetrically at the upper end); the inclusion test below decides exactly.
    const double q1lo = floor((ys1 - rs - a.lo[0]) * a.inv_w[0]), q1hi = floor((ys1 + rs - a.lo[0]) * a.inv_w[0]);
    const double q2lo = floor((ys2 - rs - a.lo[1]) * a.inv_w[1]), q2hi = floor((ys2 + rs - a.lo[1]) * a.inv_w[1]);
    const int p1lo = (int)fmax(0.0, fmin(q1lo, (double)a.n[0]));
    const int p1hi = (int)fmax(-1.0, fmin(q1hi, (double)a.n[0] - 1));
    const int p2lo = (int)fmax(0.0, fmin(q2lo, (double)a.n[1]));
    const int p2hi = (int)fmax(-1.0, fmin(q2hi, (double)a.n[1] - 1));
    const int nx = active ? p1hi - p1lo + 1 : 0, ny = active ? p2hi - p2lo + 1 : 0;
    const bool staged = nx <= kLcAxis * SPLIT && ny <= kLcAxis * SPLIT;
    if (staged) {
        for (int c = lane; c < nx; c += kLanes) {
            const double d = (a.lo[0] + ((double)(p1lo + c) + 0.5) * a.w[0]) - ys1;
            const double d2 = d * d;
            s_col[wv][c] = make_double2(d2, gauss ? exp(-d2 * inv2s2) : 1.0);
        }
        for (int r = lane; r < ny; r += kLanes) {
            const double d = (a.lo[1] + ((double)(p2lo + r) + 0.5) * a.w[1]) - ys2;
            const double d2 = d * d;
            s_row[wv][r] = make_double2(d2, gauss ? exp(-d2 * inv2s2) : 1.0);
        }
    }
    __syncthreads();
    double num = 0.0, den = 0.0;
    if (nx > 0 && ny > 0) {
        if (staged) {
            const int total = nx * ny;
            // e = dr * nx + dc, advanced by kLanes without a division per pixel
            int dr = lane / nx, dc = lane - (lane / nx) * nx;
            const int sr = kLanes / nx, sc = kLanes - (kLanes / nx) * nx;
            const int64_t n0 = a.n[0];
            const uint32_t *base = a.counts + (int64_t)k * a.frame_stride + (int64_t)p2lo * n0 + p1lo;
            auto advance = [&]() {
                dc += sc;
                dr += sr;
                if (dc >= nx) {
                    dc -= nx;
                    ++dr;
                }
            };
            if constexpr (AHEAD == 1) {
                for (int e = lane; e < total; e += kLanes) {
                    const double2 cx = s_col[wv][dc], ry = s_row[wv][dr];
                    if (cx.x + ry.x <= rs2) {
                        const double n = (double)base[(int64_t)dr * n0 + dc];
                        if (gauss) {
                            const double wgt = cx.y * ry.y;
                            num += wgt * n;
                            den += wgt;
                        } else {
                            num += n;
                            den += 1.0;
                        }
                    }
                    advance();
                }
            } else {
                for (int e = lane; e < total; e += kLanes * AHEAD) {
                    double wgt[AHEAD];
                    uint32_t n[AHEAD];
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        const bool box = e + kLanes * u < total;
                        const int c = box ? dc : 0, r = box ? dr : 0;
                        const double2 cx = s_col[wv][c], ry = s_row[wv][r];
                        n[u] = base[(int64_t)r * n0 + c];
                        wgt[u] = box && cx.x + ry.x <= rs2 ? (gauss ? cx.y * ry.y : 1.0) : 0.0;
                        advance();
                    }
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        num += wgt[u] * (double)n[u];
                        den += wgt[u];
                    }
                }
            }
        } else {
            const int64_t total = (int64_t)nx * ny;
            for (int64_t e = lane; e < total; e += kLanes) {
                const int r = (int)(e / nx);
                const int p1 = p1lo + (int)(e - (int64_t)r * nx), p2 = p2lo + r;
                const double d1 = (a.lo[0] + ((double)p1 + 0.5) * a.w[0]) - ys1;
                const double d2 = (a.lo[1] + ((double)p2 + 0.5) * a.w[1]) - ys2;
                const double d2s = d1 * d1 + d2 * d2;
                if (d2s <= rs2) {
                    const double wgt = gauss ? exp(-d2s * inv2s2) : 1.0;
                    num += wgt * (double)a.counts[(int64_t)k * a.frame_stride + (int64_t)p2 * a.n[0] + p1];
                    den += wgt;
                }
            }
        }
    }
    num = wave_sum(num);
    den = wave_sum(den);
    if constexpr (SPLIT > 1) {
        if ((threadIdx.x & 63) == 0) {
            s_sum[threadIdx.x >> 6][0] = num;
            s_sum[threadIdx.x >> 6][1] = den;
        }
        __syncthreads();
        num = den = 0.0;
        for (int w = 0; w < kLcWaves; ++w) {
            num += s_sum[w][0];
            den += s_sum[w][1];
        }
    }
    if (active && lane == 0) {
        const double mu = den > 0.0 ? num / (den * a.n_av) : __builtin_nan("");
        if (a.mu) a.mu[gp] = mu;
        if (a.mag) a.mag[gp] = -2.5 * log10(mu);
    }
}

// Four consecutive counts; the address is only 4-byte aligned (global loads of any width take that).
__device__ __forceinline__ uint4 load4(const uint32_t *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

// One lane per track point (used when there are many points): the lane
// walks its support box row by row, so no cross-lane reduction or staging is needed and
// consecutive lanes (consecutive points of a track) read neighbouring pixels.  The Gaussian
// factors along a row and down a column follow the exact recurrences
//   g(d + w) = g(d) r(d),  r(d + w) = r(d) exp(-w^2 / s^2),  r(d) = exp(-(2 d w + w^2) / 2 s^2),
// FP64 multiplies instead of an exp per pixel.
// The pixels of a row inside the support are one run of columns: |c - y| grows with the distance of the column,
// rounded or not.  Its ends are estimated with a square root and settled by the plain definition's own FP64
// inclusion test, so the included set is that of testing every pixel; the pixels between them take no test (14
// FP64 instructions a pixel of the box before, 6 a pixel inside and about 45 a row now), and their counts come four
// to a load.  Row sums take the row's Gaussian factor once.  The settling loops end at their first test as a rule: four
// tests unrolled were half of a row's instructions (266 us).
// Bound: FP64 issue and the L1 lines that the lanes of a load touch.  1e6 points, 1024^2 map, 21 x 21-pixel box: 192 us
// (testing every pixel of the box 480); error against 80-bit sums 2.6e-16 (7.9e-16) rms.
__global__ void __launch_bounds__(256) k_light_curve_lanes(const LightArgs a)
{
    const int64_t gp = group_number() * 256 + threadIdx.x;
    if (gp >= (int64_t)a.n_tracks * a.n_points) return;
    const int64_t tr = gp / a.n_points;
    const int k = (int)(gp - tr * a.n_points);
    const double *t = a.tracks + 4 * tr;
    const double f = a.n_points > 1 ? (double)k / (double)(a.n_points - 1) : 0.0;
    const double ys1 = t[0] + f * (t[2] - t[0]);
    const double ys2 = t[1] + f * (t[3] - t[1]);
    const double rs = a.support, rs2 = a.support * a.support;
    const bool gauss = a.kind == 0;
    const double q1lo = floor((ys1 - rs - a.lo[0]) * a.inv_w[0]), q1hi = floor((ys1 + rs - a.lo[0]) * a.inv_w[0]);
    const double q2lo = floor((ys2 - rs - a.lo[1]) * a.inv_w[1]), q2hi = floor((ys2 + rs - a.lo[1]) * a.inv_w[1]);
    const int p1lo = (int)fmax(0.0, fmin(q1lo, (double)a.n[0]));
    const int p1hi = (int)fmax(-1.0, fmin(q1hi, (double)a.n[0] - 1));
    const int p2lo = (int)fmax(0.0, fmin(q2lo, (double)a.n[1]));
    const int p2hi = (int)fmax(-1.0, fmin(q2hi, (double)a.n[1] - 1));
    double num = 0.0, den = 0.0;
    if (p1hi >= p1lo && p2hi >= p2lo) {
        const double w1 = a.w[0], w2 = a.w[1], h = a.inv2s2;
        // the recurrences stay finite while every exponent is moderate; otherwise (a source much
        // narrower than a pixel) each weight takes its own exp
        const double ext = rs + 2.0 * fmax(w1, w2);
        const bool rec = gauss && ext * ext * h < 600.0 && 2.0 * ext * fmax(w1, w2) * h < 600.0;
        const double dx0 = (a.lo[0] + ((double)p1lo + 0.5) * w1) - ys1;
        const double gx0 = rec ? exp(-dx0 * dx0 * h) : 1.0;
        const double rx0 = rec ? exp(-(2.0 * dx0 * w1 + w1 * w1) * h) : 1.0;
        const double kx = rec ? exp(-2.0 * w1 * w1 * h) : 1.0;
        const double dy0 = (a.lo[1] + ((double)p2lo + 0.5) * w2) - ys2;
        double gy = rec ? exp(-dy0 * dy0 * h) : 1.0;
        double ry = rec ? exp(-(2.0 * dy0 * w2 + w2 * w2) * h) : 1.0;
        const double ky = rec ? exp(-2.0 * w2 * w2 * h) : 1.0;
        // the source's place in columns, and what rounding may move a column's place or the end of a run by (in
        // columns; a rounding of R^2 moves the end by up to 3e-8 R)
        const double mid = (ys1 - a.lo[0]) * a.inv_w[0] - 0.5;
        const double slack =
            1e-3 + (1e-7 * rs + 0x1p-46 * (fabs(a.lo[0]) + (double)a.n[0] * w1 + fabs(ys1))) * a.inv_w[0];
        for (int p2 = p2lo; p2 <= p2hi; ++p2) {
            const double dy = (a.lo[1] + ((double)p2 + 0.5) * w2) - ys2;
            const double dy2 = dy * dy;
            auto offset = [&](int p1) { return (a.lo[0] + ((double)p1 + 0.5) * w1) - ys1; };
            auto inside = [&](int p1) {
                const double dx = offset(p1);
                return dx * dx + dy2 <= rs2;
            };
            if (dy2 <= rs2) {
                // estimated ends, widened by more than the estimate's error, then moved in to where the test
                // holds (mostly at once, so the loops are not unrolled); first ends past last when no pixel of the
                // row is inside
                const double half = __builtin_amdgcn_sqrt(rs2 - dy2) * a.inv_w[0];
                const double reach = half + (half * 1e-6 + slack);
                int first = (int)fmin(fmax(ceil(mid - reach), (double)p1lo), (double)p1hi);
                int last = (int)fmin(fmax(floor(mid + reach), (double)p1lo), (double)p1hi);
#pragma clang loop unroll(disable) vectorize(disable)
                while (first <= last && !inside(first)) ++first;
#pragma clang loop unroll(disable) vectorize(disable)
                while (last > first && !inside(last)) --last;
                const uint32_t *row = a.counts + (int64_t)k * a.frame_stride + (int64_t)p2 * a.n[0];
                double sn = 0.0, sw = 0.0;
                // the run's counts in order, four to a load; the last one to three come with the four that end the run
                // (four requested ahead, too: 100 VGPRs instead of 78, and slower, 208 us against 192)
                auto walk = [&](auto add4, auto add) __attribute__((always_inline)) {
                    int p1 = first;
                    if (p1 + 3 <= last) {
                        const uint4 tail = load4(row + last - 3);
                        for (; p1 + 3 <= last; p1 += 4) add4(load4(row + p1));
                        const int rest = last - p1 + 1;
                        if (rest > 2) add(tail.y);
                        if (rest > 1) add(tail.z);
                        if (rest > 0) add(tail.w);
                    } else {
#pragma clang loop unroll(disable) vectorize(disable)
                        for (; p1 <= last; ++p1) add(row[p1]);
                    }
                };
                if (rec) {
                    double gx = gx0, rx = rx0;
                    for (int p1 = p1lo; p1 < first; ++p1) {
                        gx *= rx;
                        rx *= kx;
                    }
                    auto add = [&](uint32_t n) {
                        sn = fma(gx, (double)n, sn);
                        sw += gx;
                        gx *= rx;
                        rx *= kx;
                    };
                    walk([&](const uint4 &n) {
                        add(n.x);
                        add(n.y);
                        add(n.z);
                        add(n.w);
                    }, add);
                    num = fma(gy, sn, num);
                    den = fma(gy, sw, den);
                } else if (gauss) {
                    for (int p1 = first; p1 <= last; ++p1) {
                        const double dx = offset(p1);
                        const double wgt = exp(-(dx * dx + dy2) * h);
                        num += wgt * (double)row[p1];
                        den += wgt;
                    }
                } else {
                    walk([&](const uint4 &n) { sn += ((double)n.x + (double)n.y) + ((double)n.z + (double)n.w); },
                         [&](uint32_t n) { sn += (double)n; });
                    num += sn;
                    den += (double)(last - first + 1);
                }
            }
            if (rec) {
                gy *= ry;
                ry *= ky;
            }
        }
    }
    const double mu = den > 0.0 ? num / (den * a.n_av) : __builtin_nan("");
    if (a.mu) a.mu[gp] = mu;
    if (a.mag) a.mag[gp] = -2.5 * log10(mu);
}

}  // namespace

hipError_t launch_light_curve(const LightArgs &a, hipStream_t s)
{
    const int64_t pts = (int64_t)a.n_tracks * a.n_points;
    if (pts <= 0) return hipSuccess;
    // the support box spans at most this many pixels per axis
    const double bx = std::min(std::ceil(2.0 * a.support * a.inv_w[0]) + 2.0, (double)a.n[0]);
    const double by = std::min(std::ceil(2.0 * a.support * a.inv_w[1]) + 2.0, (double)a.n[1]);
    // Which layout is faster, from what each measured over 50 to 1e6 points and boxes of 15 to 6e4 pixels: the
    // time of one point on an idle GPU and the time that a point of very many adds, combined as a root of
    // squares.  Waves take 0.75 ns a point and 0.58 ps a pixel of its box, but 3.2 us and 2.9 ns a pixel one by
    // one; with pixels requested ahead 0.85, 0.63, 3.5 and 1.1; workgroups 1.9, 0.6, 3.3 and 0.27 (1.6 ps and
    // 1.3 ns where the box is not staged).  Lanes take 0.2 ps a pixel, but never less than 7.5 us and 39 ns a
    // pixel, one lane's walk.  Box 1764, us of the three wave layouts: 300 points 8.5, 5.7, 4.4; 6020 15.2, 14.4,
    // 20.9; 15050 29.6, 30.0, 45.1.  38400 points, lanes and waves: box 234 15, 32; 1279 52, 56; 27836 866, 668.
    // 1e6 points: box 1279 238, 1250; 27836 4340, 17100.
    const double box = bx * by, np = (double)pts, inf = HUGE_VAL;
    const double side = std::max(bx, by);
    const double t1 = side <= kLcAxis ? std::hypot(3.2e3 + 2.9 * box, np * (0.75 + 0.58e-3 * box)) : inf;
    const double t4 = side <= kLcAxis ? std::hypot(3.5e3 + 1.1 * box, np * (0.85 + 0.63e-3 * box)) : inf;
    const bool wide = side > kLcAxis * kLcWaves;
    const double tg = std::hypot(3.3e3 + (wide ? 1.3 : 0.27) * box, np * (1.9 + (wide ? 1.6e-3 : 0.6e-3) * box));
    const double t_lane = std::max(np * (0.04 + 0.2e-3 * box), 7.5e3 + 39.0 * box);
    const bool lanes = a.path == 1 || (a.path == 0 && t_lane < std::min(tg, std::min(t1, t4)));
    if (lanes) {
        const int64_t blocks = (pts + 255) / 256;
        if (blocks > 0x7fffffff) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_light_curve_lanes, group_dim3(blocks, 256), dim3(256), 0, s, a);
    } else {
        const int64_t blocks = (pts + kLcWaves - 1) / kLcWaves;
        if (blocks > 0x7fffffff) return hipErrorInvalidValue;
        const dim3 blk(64 * kLcWaves);
        const dim3 g = group_dim3(blocks, 64 * kLcWaves);
        if (tg < t1 && tg < t4)
            hipLaunchKernelGGL((k_light_curve<kLcWaves, kLcAhead>), group_dim3(pts, 64 * kLcWaves), blk, 0, s, a);
        else if (t4 < t1) hipLaunchKernelGGL((k_light_curve<1, kLcAhead>), g, blk, 0, s, a);
        else hipLaunchKernelGGL((k_light_curve<1, 1>), g, blk, 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace rs

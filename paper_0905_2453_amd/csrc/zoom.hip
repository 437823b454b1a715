// Interactive zoom (section 4: a selected area of a map recomputed at higher ray density).
//
// The zoom map is, by definition, the map that shooting EVERY ray of the fine grid would give on
// the selected source-plane window.  Only rays that can land in the window matter, so the fine
// grid is split into culling cells and each cell's whole image under the lens equation (eq. 6
// with the deflection of eq. 2) is bounded from one evaluation at the cell centre c:
//
//   y(x) = y(c) + J(c)(x - c) + R(x)     for the lenses at distance >= 3 rho from c
//                                         (rho = half-diagonal of the cell), with
//   J = diag(l1, l2) - grad alpha,  grad alpha_i = m_i / r^4 [[f2^2 - f1^2, -2 f1 f2], [-2 f1 f2, f1^2 - f2^2]]
//   |R| <= rho^2 sum m_i / (r_i - rho)^3 <= rho^2 (3/2)^3 sum m_i / r_i^3    (|d^2 alpha_i| = 2 m / r^3)
//
// while a lens closer than 3 rho moves the image by at most |alpha_i(x) - alpha_i(c)| <= 2 m_i / delta_i
// (delta_i = its distance to the cell rectangle); a lens inside the rectangle leaves the image
// unbounded.  A cell whose bounding box, widened by a rounding allowance, misses the window cannot
// contribute and is skipped; the rays of the kept cells are shot exactly as the plain path shoots
// them, so the zoom map equals the full fine-grid map on the window.
#include <algorithm>

#include "rs_internal.h"

namespace rs {

namespace {

constexpr int kZoomRun = 16;     // float32 run length before the FP64 combine
constexpr int kZoomSums = 8;

__device__ __forceinline__ float4 zoom_pad_lens()
{
    return make_float4(kPadCoord, kPadCoord, 0.0f, 0.0f);
}

// A wave's LDS accesses are performed in order; this keeps the compiler to the order as well.
__device__ __forceinline__ void zoom_wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The Taylor terms of a run: Jacobian and remainder sums over its lenses (SELECT: only those at distance >=
// 3 rho), and the smallest squared distance.  The operations of a lens are the same either way.
template <bool SELECT>
__device__ __forceinline__ void zoom_run(const float4 *L, float cf1, float cf2, float near2, float &s1, float &s2,
                                         float &sd, float &so, float &sc, float &sp, float &sq, float &rmin)
{
    s1 = s2 = sd = so = sc = sp = sq = 0.f;
    rmin = INFINITY;
#pragma unroll SELECT ? 1 : kZoomRun
    for (int j = 0; j < kZoomRun; ++j) {
        const float4 l = L[j];
        const float f1 = cf1 - l.x, f2 = cf2 - l.y;
        const float f1s = f1 * f1, f2s = f2 * f2;
        const float r2 = f1s + f2s;
        const float s = __builtin_amdgcn_rsqf(r2);
        const float q = s * s;
        const float d = l.z * q;
        if (!SELECT) {
            s1 = fmaf(d, f1, s1);
            s2 = fmaf(d, f2, s2);
            // the rounding-allowance sums take every lens (an over-estimate is safe)
            sp = fmaf(l.z, s, sp);
            sq += d;
            rmin = fminf(rmin, r2);
        }
        const float dt = SELECT && r2 < near2 ? 0.0f : d;
        const float dq = dt * q;
        sd = fmaf(dq, f2s - f1s, sd);
        so = fmaf(dq, f1 * f2, so);
        sc = fmaf(dt, s, sc);
    }
}

// One work item per cell of one culling level; kept cells are appended to that level's list.
//   level 0: every cell of the coarsest level;
//   level l > 0: the cells inside the cells kept at level l - 1: item t takes child t % P^2 of
//                kept cell lists[l - 1][t / P^2].
// With z.flags the last level sets a flag per kept cell instead (k_zoom_rows lists them by row).
// A child's rectangle lies inside its parent's, so a cell whose image can meet the map is kept
// at every level above it.
//
// Persistent: a workgroup takes 64 / ks cells at a time from the level's counter.  Its WV waves split the lenses
// (wave w sums the chunks of 64 lenses w, w + WV, ..., staged privately), and ks (1, 2 or 4) consecutive
// lanes share a cell, each summing every ks-th run of the chunks; the partial sums meet in a fixed butterfly
// and then in LDS in wave order.  A level has few cells (15 000 to 140 000 on the benchmark's zoom), so a lane
// that sums a cell alone, or a sixteenth of it, leaves most wave slots empty (1.8 waves per SIMD on average).  The
// Taylor terms are summed without a look at the distance and redone for the rare run that holds a near lens.
// The five levels of that zoom (1e5 lenses): 16.1 ms, 31.0 before both changes.  Lanes that share a cell read
// different runs at once: with a place skipped after each run these lie on different banks, and with eight waves two
// workgroups fit a compute unit, one's merge under the other's sums: 14.3 ms (runs on the same banks 16.1, the skip
// alone 15.1; 30 000 lenses: 2.45, 2.17, both 2.02).
// Fields of fewer chunks than eight take as many waves; their items are cheap, so workgroups step through them without
// the counter (a take costs about 12 ns, with 4096 workgroups 50 us a level), and ks follows the level's real number of
// cells (`lanes` of them or more: 1; 64 lenses, 0.02 of 4096^2 rays' span: 76 us from the host's estimate, 69).
template <int WV>
__global__ void __launch_bounds__(64 * WV, 4) k_zoom_mark(const ZoomArgs z, int level, int ks, int lanes)
{
    __shared__ union {
        float4 lens[WV][64 + 64 / kZoomRun];   // a place is skipped after each run
        double sum[WV][kZoomSums][64];
    } sm;
    __shared__ uint32_t s_inside[64];
    __shared__ uint32_t s_item;
    constexpr bool QUEUE = WV == 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t P = z.P, PP = z.P * z.P;
    const int64_t cw1 = z.lcw1[level], cw2 = z.lcw2[level];
    const int64_t n_items = level == 0 ? z.lnx[0] * z.lny[0] : (int64_t)z.stats[4 + level - 1] * PP;
    if (!QUEUE)
        for (ks = 1; ks < 4 && n_items * ks < lanes;) ks <<= 1;
    const int part = lane & (ks - 1);
    const int64_t n_chunks = (z.n_lens + 63) / 64;
    auto fetch = [&](int64_t c) -> float4 {
        const int64_t i = c * 64 + lane;
        return i < z.n_lens ? moved_lens(z.lenses[i], z.vel, i, z.time) : zoom_pad_lens();
    };
    for (int64_t item = blockIdx.x;; item += gridDim.x) {
        __syncthreads();   // the last item's sums are read
        if (QUEUE && tid == 0) s_item = atomicAdd(&z.stats[kZoomQueue + level], 1u);
        if (tid < 64) s_inside[tid] = 0u;
        __syncthreads();
        const int64_t first = (QUEUE ? (int64_t)s_item : item) * (64 / ks);
        if (first >= n_items) break;
        const int64_t t_id = first + lane / ks;
        int64_t cx = 0, cy = 0, idx = 0;
        if (t_id < n_items) {
            if (level == 0) {
                cx = t_id % z.lnx[0];
                cy = t_id / z.lnx[0];
                idx = t_id;
            } else {
                const int64_t par = z.lists[level - 1][t_id / PP], k = t_id % PP;
                cx = (par % z.lnx[level - 1]) * P + k % P;
                cy = (par / z.lnx[level - 1]) * P + k / P;
                idx = cy * z.lnx[level] + cx;
            }
        }
        const bool active = t_id < n_items && cx * cw1 < z.wn1 && cy * cw2 < z.wn2;
        // the cell's float32 centre and the half-widths of the rectangle around it that holds every fine ray's
        // float32 coordinates (evaluated again after the lens loop, not kept across it)
        auto geometry = [&](float &cf1, float &cf2, double &h1, double &h2) {
            const int64_t g10 = z.wlo1 + min(cx * cw1, z.wn1), g11 = z.wlo1 + min((cx + 1) * cw1, z.wn1);
            const int64_t g20 = z.wlo2 + min(cy * cw2, z.wn2), g21 = z.wlo2 + min((cy + 1) * cw2, z.wn2);
            const double e1lo = z.glo1 + (double)g10 * z.gt1, e1hi = z.glo1 + (double)g11 * z.gt1;
            const double e2lo = z.glo2 + (double)g20 * z.gt2, e2hi = z.glo2 + (double)g21 * z.gt2;
            cf1 = (float)(0.5 * (e1lo + e1hi));
            cf2 = (float)(0.5 * (e2lo + e2hi));
            h1 = fmax(fabs(e1lo - (double)cf1), fabs(e1hi - (double)cf1)) + z.pad;
            h2 = fmax(fabs(e2lo - (double)cf2), fabs(e2hi - (double)cf2)) + z.pad;
        };
        float cf1, cf2, fh1, fh2, near2;
        {
            double h1, h2;
            geometry(cf1, cf2, h1, h2);
            near2 = (float)(9.0 * (h1 * h1 + h2 * h2));
            fh1 = (float)h1;
            fh2 = (float)h2;
        }

        double A1 = 0.0, A2 = 0.0, Jd = 0.0, Jo = 0.0, C3 = 0.0, P1 = 0.0, D2 = 0.0, nearsum = 0.0;
        bool inside = false;
        float4 nxt = zoom_pad_lens();
        if (wave < n_chunks) nxt = fetch(wave);
        for (int64_t c = wave; c < n_chunks; c += WV) {
            sm.lens[wave][lane + lane / kZoomRun] = nxt;
            zoom_wave_fence();
            if (c + WV < n_chunks) nxt = fetch(c + WV);
            for (int r = part * kZoomRun; r < 64; r += ks * kZoomRun) {
                const float4 *L = &sm.lens[wave][r + r / kZoomRun];
                float s1, s2, sd, so, sc, sp, sq, rmin;
                zoom_run<false>(L, cf1, cf2, near2, s1, s2, sd, so, sc, sp, sq, rmin);
                // (keeps the Taylor sums in the loop above: moved behind the branch, their terms would all
                // have to be held until it)
                asm volatile("" : "+v"(sd), "+v"(so), "+v"(sc));
                if (__any(rmin < near2)) {
                    // near lenses (rare): the Taylor terms again without them, and each one's whole
                    // variation over the cell bounded by 2 m / delta
                    float x1, x2, xp, xq, xr;
                    zoom_run<true>(L, cf1, cf2, near2, x1, x2, sd, so, sc, xp, xq, xr);
                    float ns = 0.0f;
#pragma unroll 1
                    for (int j = 0; j < kZoomRun; ++j) {
                        const float4 l = L[j];
                        const float f1 = cf1 - l.x, f2 = cf2 - l.y;
                        const bool nr = f1 * f1 + f2 * f2 < near2 && l.z != 0.0f;
                        const float ex = fmaxf(fabsf(f1) - fh1, 0.0f), ey = fmaxf(fabsf(f2) - fh2, 0.0f);
                        const float dl2 = ex * ex + ey * ey;
                        inside = inside || (nr && !(dl2 > 0.0f));
                        ns += nr && dl2 > 0.0f ? l.z * __builtin_amdgcn_rsqf(dl2) : 0.0f;
                    }
                    nearsum += (double)ns;
                }
                A1 += (double)s1;
                A2 += (double)s2;
                Jd += (double)sd;
                Jo += (double)so;
                C3 += (double)sc;
                P1 += (double)sp;
                D2 += (double)sq;
            }
            zoom_wave_fence();
        }
        // the lanes' partial sums of a cell in a fixed order, then the waves'
        for (int o = 1; o < ks; o <<= 1) {
            A1 += __shfl_xor(A1, o, 64);
            A2 += __shfl_xor(A2, o, 64);
            Jd += __shfl_xor(Jd, o, 64);
            Jo += __shfl_xor(Jo, o, 64);
            C3 += __shfl_xor(C3, o, 64);
            P1 += __shfl_xor(P1, o, 64);
            D2 += __shfl_xor(D2, o, 64);
            nearsum += __shfl_xor(nearsum, o, 64);
        }
        if constexpr (WV > 1) {
            __syncthreads();   // every wave is done with its staged lenses
            const double v[kZoomSums] = {A1, A2, Jd, Jo, C3, P1, D2, nearsum};
#pragma unroll
            for (int k = 0; k < kZoomSums; ++k) sm.sum[wave][k][lane] = v[k];
        }
        if (inside) s_inside[lane - part] = 1u;
        __syncthreads();
        if (wave == 0) {
            if constexpr (WV > 1) {
                double v[kZoomSums] = {};
                for (int w = 0; w < WV; ++w)
#pragma unroll
                    for (int k = 0; k < kZoomSums; ++k) v[k] += sm.sum[w][k][lane];
                A1 = v[0];
                A2 = v[1];
                Jd = v[2];
                Jo = v[3];
                C3 = v[4];
                P1 = v[5];
                D2 = v[6];
                nearsum = v[7];
            }
            inside = s_inside[lane - part] != 0u;
            double h1, h2;
            geometry(cf1, cf2, h1, h2);
            const double rho2 = h1 * h1 + h2 * h2;

            // centre image and the bounds, FP64
            const double y1 = z.lam1 * (double)cf1 - A1, y2 = z.lam2 * (double)cf2 - A2;
            const double J11 = fabs(z.lam1 - Jd), J22 = fabs(z.lam2 + Jd), J12 = 2.0 * fabs(Jo);
            const double tay = rho2 * 3.375 * C3;
            const double nv = 2.0 * nearsum;
            // rounding allowance: float32 arithmetic of the fine rays and of this centre evaluation
            const double scale = 1.5 * P1 + nearsum + fabs(z.lam1 * (double)cf1) + fabs(z.lam2 * (double)cf2) +
                                 fabs(y1) + fabs(y2) + z.xmax * 2.25 * D2;
            const double slack = 1e-5 * scale + z.margin;
            const double E1 = (J11 * h1 + J12 * h2 + tay + nv + slack) * (1.0 + 1e-6);
            const double E2 = (J12 * h1 + J22 * h2 + tay + nv + slack) * (1.0 + 1e-6);
            bool keep = inside || !(fabs(y1) < 1e300 && fabs(y2) < 1e300 && E1 < 1e300 && E2 < 1e300);
            if (!keep)
                keep = (y1 + E1 >= z.zlo1) && (y1 - E1 <= z.zhi1) && (y2 + E2 >= z.zlo2) && (y2 - E2 <= z.zhi2);
            if (keep && active && part == 0) {
                if (level == z.levels - 1 && z.flags) {
                    atomicAdd(&z.stats[0], 1u);
                    z.list[idx] = 1u;
                } else {
                    uint32_t *cnt = level == z.levels - 1 ? &z.stats[0] : &z.stats[4 + level];
                    z.lists[level][atomicAdd(cnt, 1u)] = (uint32_t)idx;
                }
            }
        }
    }
}

// Everything a zoom clears or sets before its kernels, in one launch: the statistics, the cells' flags, the partial maps.
__global__ void __launch_bounds__(256) k_zoom_init(const ZoomInit z)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (first < kZoomQueue + kZoomLevels)
        z.stats[first] = first == 1 ? z.cells : first == 2 ? z.blocks : first == 3 ? z.rays : 0u;
    for (int64_t i = first; i < z.n_flags; i += stride) z.flags[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = first; i < z.n_part; i += stride) z.part[i] = make_uint4(0u, 0u, 0u, 0u);
}

// A row of cells per workgroup at a time: its kept cells' columns, in order, to the front of the row's part of the
// list (in place: a place is written after the flags up to it are read), and the items they make (CellBlocks).
__global__ void __launch_bounds__(1024) k_zoom_rows(const CellBlocks cb, uint32_t *list)
{
    __shared__ uint32_t s_wave[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int64_t my = blockIdx.x; my < cb.ncy; my += gridDim.x) {
        uint32_t *row = list + my * cb.ncx;
        uint32_t kept = 0;
        for (int64_t i0 = 0; i0 < cb.ncx; i0 += 1024) {
            const bool k = i0 + tid < cb.ncx && row[i0 + tid] != 0u;
            const unsigned long long b = __ballot(k);
            if (lane == 0) s_wave[wave] = (uint32_t)__popcll(b);
            __syncthreads();
            uint32_t before = kept;
            for (int w = 0; w < 16; ++w) {
                if (w == wave) before = kept;
                kept += s_wave[w];
            }
            if (k) row[before + __popcll(b & ((1ull << lane) - 1))] = (uint32_t)(i0 + tid);
            __syncthreads();
        }
        if (tid == 0) {
            cb.cells[my] = kept;
            const uint64_t cols = kept ? max((uint64_t)kept * (uint64_t)cb.c1, (uint64_t)kMinColumns) : 0;
            cb.start[my] = (cols * (uint64_t)cb.groups + 63) / 64;
        }
    }
}

// Exclusive scan of start[0 .. ncy) in place, the sum to start[ncy], with one workgroup.
__global__ void __launch_bounds__(1024) k_zoom_row_scan(const CellBlocks cb)
{
    __shared__ uint64_t part[1024];
    const int tid = threadIdx.x;
    const int64_t per = (cb.ncy + 1023) / 1024, b = min(cb.ncy, tid * per), e = min(cb.ncy, b + per);
    uint64_t s = 0;
    for (int64_t i = b; i < e; ++i) s += cb.start[i];
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    uint64_t run = part[tid] - s;
    for (int64_t i = b; i < e; ++i) {
        const uint64_t v = cb.start[i];
        cb.start[i] = run;
        run += v;
    }
    if (tid == 1023) cb.start[cb.ncy] = part[1023];
}

}  // namespace

hipError_t launch_zoom_init(const ZoomInit &z, hipStream_t s)
{
    const int64_t blocks = std::min<int64_t>(8192, std::max<int64_t>(1, (std::max(z.n_flags, z.n_part) + 255) / 256));
    hipLaunchKernelGGL(k_zoom_init, dim3((unsigned)blocks), dim3(256), 0, s, z);
    return hipGetLastError();
}

hipError_t launch_zoom_rows(const CellBlocks &cb, uint32_t *list, hipStream_t s)
{
    if (cb.ncx <= 0 || cb.ncy <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zoom_rows, dim3((unsigned)std::min<int64_t>(cb.ncy, 4096)), dim3(1024), 0, s, cb, list);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zoom_row_scan, dim3(1), dim3(1024), 0, s, cb);
    return hipGetLastError();
}

template <int WV>
hipError_t launch_mark(const ZoomArgs &z, hipStream_t s)
{
    int64_t items = z.lnx[0] * z.lny[0];
    if (items <= 0) return hipSuccess;
    int occ = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_zoom_mark<WV>, 64 * WV, 0) != hipSuccess) occ = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    const int lanes = 64 * 4 / WV * cus;
    for (int l = 0; l < z.levels; ++l) {
        // level l > 0 runs over at most every child of every cell of level l - 1.  Lanes per cell: enough
        // to give two workgroups per compute unit for the expected work (every cell at level 0, the children
        // of about a third of the cells above further down); the choice only affects speed.
        if (l > 0) items = z.lnx[l - 1] * z.lny[l - 1] * z.P * z.P;
        const int64_t expect = l == 0 ? items : std::max<int64_t>(1, items / 3);
        int ks = 1;
        while (ks < 4 && expect * ks < int64_t(64) * 2 * cus) ks <<= 1;
        const int64_t per_block = WV < 8 ? 16 : 64 / ks;
        const int64_t grid = std::min<int64_t>((items + per_block - 1) / per_block, (int64_t)std::max(1, occ) * cus);
        hipLaunchKernelGGL(k_zoom_mark<WV>, dim3((unsigned)grid), dim3(64 * WV), 0, s, z, l, ks, lanes);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_zoom_mark(const ZoomArgs &z, hipStream_t s)
{
    // As many waves as there are chunks of 64 lenses, up to eight: waves without a chunk only wait and merge, and one
    // wave with two chunks takes longer (128 lenses, 4096^2 rays: 107 us a zoom with one wave, 81 with two, 127 with
    // eight).
    if (z.n_lens <= 64) return launch_mark<1>(z, s);
    if (z.n_lens <= 128) return launch_mark<2>(z, s);
    if (z.n_lens <= 256) return launch_mark<4>(z, s);
    return launch_mark<8>(z, s);
}

}  // namespace rs

// Direct inverse ray-shooting with the lenses split over the waves of a workgroup: the one-column ray
// blocks of rs_shoot, rs_shoot_batched and rs_shoot_zoom.
//
// Method: Thompson, Fluke, Barnes & Barsdell (2009), section 1 eqs. 1, 2, 4; section 2 eq. 5 (the sum
// over the lenses as partial sums over subsets); section 3.2 eq. 6.
//
// Work decomposition.  The WV waves of a workgroup share 64 blocks of four rays: lane l holds column
// c0 + l, rows r0 .. r0 + 3 (or its own block of the kept culling cells).  Wave w sums the groups of
// T kQuadRuns lenses w, w + WV, w + 2 WV, ... of the field; every group is summed operation by operation as
// k_direct sums it, and the waves' FP64 sums meet in LDS in wave order.  FP64 addition of the groups'
// float32 sums is exact while they stay within 2^29 of each other (24-bit numbers in a 53-bit sum), so
// the order does not show in a ray's position, and the maps are those of k_direct.
#include <algorithm>

#include "direct_common.h"

namespace rs {

namespace {

// Where the four rays of a lane lie: on rows that all lanes share, on one of up to kRowGroups consecutive
// groups of four rows, or each at a random point of its cell.
enum RayMode { kSharedRows = 0, kGroupRows = 1, kJitter = 2 };
constexpr int kRowGroups = 3;
static_assert((kMinColumns - 1 + 63) / kMinColumns + 1 <= kRowGroups, "64 blocks in a row meet kRowGroups groups");

// kGroupRows: window row of the first group, groups of the workgroup's blocks, the lane's one.
struct RowGroups {
    uint32_t first;
    int n, mine;
};

// B lenses are staged by a wave at a time (private to it: the lens loop has no barrier).
template <int B, int WV, int G = 1>
struct SplitSmem {
    union {
        struct {
            float4 dy[WV][B * G];   // kJitter: the lens record; else x2 - x2_i of the four rows, of each row group
            float2 xm[WV][B];       // x1_i and the mass
        } st;
        double2 sum[WV][4][64];  // the waves' sums, after the lens loop
    };
    float4 rows[G];   // kGroupRows: x2 of the groups' rows
    uint32_t bad[64];
    int2 only[4];     // a row's only pixel and its rays there
    uint32_t lost;
};

// A wave's LDS accesses are performed in order; this keeps the compiler to the order as well.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// N staged lenses of a float32 run for the lane's four rays: the arithmetic of shoot_rays with four rows per
// reciprocal.  FIRST: they begin the run.
template <int N, bool FIRST, RayMode MODE, int B, int WV, int G>
__device__ __forceinline__ void quad_lenses(const SplitSmem<B, WV, G> &sm, int wave, int at, int mine, const float *x1,
                                            const float *x2, float *s1, float *s2)
{
#pragma unroll
    for (int j = 0; j < N; ++j) {
        float dx[4], dx2[4], dy[4], q[4], m;
        const float4 l = sm.st.dy[wave][(at + j) * G + mine];
        if constexpr (MODE != kJitter) {
            const float2 xm = sm.st.xm[wave][at + j];
            m = xm.y;
            dx[0] = x1[0] - xm.x;
            dy[0] = l.x;
            dy[1] = l.y;
            dy[2] = l.z;
            dy[3] = l.w;
        } else {
            m = l.z;
#pragma unroll
            for (int e = 0; e < 4; ++e) dy[e] = x2[e] - l.y;
#pragma unroll
            for (int e = 0; e < 4; ++e) dx[e] = x1[e] - l.x;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (MODE != kJitter && e > 0) dx[e] = dx[0];
            dx2[e] = MODE != kJitter && e > 0 ? dx2[0] : dx[e] * dx[e];
            q[e] = fmaf(dy[e], dy[e], dx2[e]);
        }
        const float p01 = q[0] * q[1], p23 = q[2] * q[3];
        const float g = m * __builtin_amdgcn_rcpf(p01 * p23);
        const float g01 = g * p23, g23 = g * p01;
        const float d[4] = {g01 * q[1], g01 * q[0], g23 * q[3], g23 * q[2]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s1[e] = FIRST && j == 0 ? d[e] * dx[e] : fmaf(d[e], dx[e], s1[e]);
            s2[e] = FIRST && j == 0 ? d[e] * dy[e] : fmaf(d[e], dy[e], s2[e]);
        }
    }
}

// One float32 run of T staged lenses.  (32 lenses as eight at a time: all unrolled, the compiler requested so many
// at once that 88 registers were spilled, 2048^2 rays, 3000 lenses: 2154 us, so 1716; k_direct 1622.)
template <int T, RayMode MODE, int B, int WV, int G>
__device__ __forceinline__ void quad_run(const SplitSmem<B, WV, G> &sm, int wave, int at, int mine, const float *x1,
                                         const float *x2, float *s1, float *s2)
{
    constexpr int N = T > 16 ? 8 : T;
    quad_lenses<N, true, MODE>(sm, wave, at, mine, x1, x2, s1, s2);
#pragma unroll 1
    for (int j = N; j < T; j += N) quad_lenses<N, false, MODE>(sm, wave, at + j, mine, x1, x2, s1, s2);
}

// Shoot the workgroup's 64 blocks of four rays.  The lane's block starts at window column c0 and row r0
// (a multiple of 4); a ray counts when its column is below cmax and its row in [rmin, rmax).  `group` (a
// workgroup's number) selects the partial map and the lost-ray counter.  Every thread of the workgroup
// must call it, lane l of every wave with the same block.
//
// Bound: issue of the lens loop.  The rows of kSharedRows belong to all lanes alike, so the lane that stages
// a lens takes x2 - x2_i of the four rows once and the loop reads the four back as one broadcast
// ds_read_b128: 24 FP32 instructions and a reciprocal per lens and four rays, where every lane subtracting
// them itself takes 28.  1e5 lenses, 4096^2 rays: 192.4 ms (8.72e12 interactions/s), k_direct 206.3 ms on the
// same box; 512^2 rays, which fill a quarter of the chip's wave slots as blocks of 1024: 3.5 ms, k_direct 8.0.
//
// kGroupRows differs in that the lens's differences are staged for each of the workgroup's row groups, and
// a lane reads its own's (adjacent 16-byte words: no bank conflict).
template <int T, int B, int WV, RayMode MODE, bool DUMP, int G, class Args>
__device__ __forceinline__ void shoot_split(const Args &a, uint32_t c0, uint32_t r0, int64_t cmax, int64_t rmin,
                                            int64_t rmax, uint32_t group, SplitSmem<B, WV, G> &sm, RowGroups rg = {})
{
    static_assert(MODE == kGroupRows || G == 1, "row groups");
    constexpr int GS = T * kQuadRuns, NG = B / GS, PL = B / 64, NX = MODE == kJitter ? 4 : 1;
    static_assert(B % GS == 0 && B % 64 == 0 && (GS & (GS - 1)) == 0 && WV >= 4, "staging shape");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    float x1[NX], x2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t g1 = a.wlo1 + c0, g2 = a.wlo2 + r0 + e, r = g2 * a.gn1 + g1;
        if (e < NX) x1[e] = ray_coord(a.glo1, a.gt1, g1, MODE == kJitter ? jitter_u(a.jkey1, r) : 0.5) * kLoopScale;
        x2[e] = ray_coord(a.glo2, a.gt2, g2, MODE == kJitter ? jitter_u(a.jkey2, r) : 0.5) * kLoopScale;
        if (MODE == kSharedRows) x2[e] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x2[e])));
    }
    if (MODE == kGroupRows) {
        if (tid < 4 * rg.n)
            reinterpret_cast<float *>(sm.rows)[tid] =
                ray_coord(a.glo2, a.gt2, a.wlo2 + rg.first + tid, 0.5) * kLoopScale;
        __syncthreads();
    }

    // the wave's k-th group is group k WV + wave of the field; staged lens `at` belongs to its group
    // gb + at / GS
    auto lens_index = [&](int64_t gb, int at) -> int64_t {
        return ((gb + at / GS) * WV + wave) * GS + (at & (GS - 1));
    };
    const int64_t n_groups = (a.n_lens + GS - 1) / GS;
    const int64_t my_groups = n_groups > wave ? (n_groups - wave + WV - 1) / WV : 0;
    float4 reg[PL];
    auto fetch = [&](int64_t gb) {
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            const int64_t i = lens_index(gb, p * 64 + lane);
            const bool in = i < a.n_lens;
            reg[p] = moved_lens(a.lenses[in ? i : 0], a.vel, in ? i : 0, a.time);
            if (!in) reg[p].z = 0.0f;            // padding as pad_lens: lens 0's position, no mass
        }
    };
    double A1[4] = {}, A2[4] = {};
    if (my_groups > 0) fetch(0);
    for (int64_t gb = 0; gb < my_groups; gb += NG) {
#pragma unroll
        for (int p = 0; p < PL; ++p) {
            float4 l = reg[p];
            l.x *= kLoopScale;
            l.y *= kLoopScale;
            if constexpr (MODE == kSharedRows) {
                sm.st.dy[wave][p * 64 + lane] = make_float4(x2[0] - l.y, x2[1] - l.y, x2[2] - l.y, x2[3] - l.y);
                sm.st.xm[wave][p * 64 + lane] = make_float2(l.x, l.z);
            } else if constexpr (MODE == kGroupRows) {
                for (int g = 0; g < rg.n; ++g) {
                    const float4 r = sm.rows[g];
                    sm.st.dy[wave][(p * 64 + lane) * G + g] = make_float4(r.x - l.y, r.y - l.y, r.z - l.y, r.w - l.y);
                }
                sm.st.xm[wave][p * 64 + lane] = make_float2(l.x, l.z);
            } else {
                sm.st.dy[wave][p * 64 + lane] = l;
            }
        }
        wave_fence();
        if (gb + NG < my_groups) fetch(gb + NG);
        const int ng = (int)min((int64_t)NG, my_groups - gb);
        for (int k = 0; k < ng; ++k) {
            const int64_t left = a.n_lens - lens_index(gb, k * GS);
            float m1[4], m2[4];
            if (left >= GS) {
#pragma unroll
                for (int h = 0; h < kQuadRuns; ++h) {
                    float s1[4], s2[4];
                    quad_run<T, MODE>(sm, wave, k * GS + h * T, rg.mine, x1, x2, s1, s2);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        m1[e] = h == 0 ? s1[e] : m1[e] + s1[e];
                        m2[e] = h == 0 ? s2[e] : m2[e] + s2[e];
                    }
                }
            } else {
                // the field's last group: only the runs that hold a lens (padding alone adds exact zeros)
#pragma unroll
                for (int e = 0; e < 4; ++e) m1[e] = m2[e] = 0.0f;
                const int runs = (int)((left + T - 1) / T);
                for (int h = 0; h < runs; ++h) {
                    float s1[4], s2[4];
                    quad_run<T, MODE>(sm, wave, k * GS + h * T, rg.mine, x1, x2, s1, s2);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        m1[e] += s1[e];
                        m2[e] += s2[e];
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                A1[e] += (double)m1[e];
                A2[e] += (double)m2[e];
            }
        }
        wave_fence();
    }

    // From here on thread (w, l), w < 4, owns the ray of row r0 + w of block l.
    const bool owner = wave < 4;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) sm.sum[wave][e][lane] = make_double2(A1[e], A2[e]);
    if (tid < 64) sm.bad[tid] = 0u;
    if (tid < 4) sm.only[tid].y = 0;
    if (tid == 0) sm.lost = 0u;
    __syncthreads();
    double B1 = 0.0, B2 = 0.0;
    if (owner) {
#pragma unroll
        for (int w = 0; w < WV; ++w) {
            const double2 v = sm.sum[w][wave][lane];
            B1 += v.x;
            B2 += v.y;
        }
        if (!__builtin_isfinite(B1 + B2)) sm.bad[lane] = 1u;
    }
    const int64_t row = (int64_t)r0 + (owner ? wave : 0);
    const int64_t g1 = a.wlo1 + c0, g2 = a.wlo2 + row, id = g2 * a.gn1 + g1;
    const float X1 = ray_coord(a.glo1, a.gt1, g1, MODE == kJitter ? jitter_u(a.jkey1, id) : 0.5) * kLoopScale;
    const float X2 = ray_coord(a.glo2, a.gt2, g2, MODE == kJitter ? jitter_u(a.jkey2, id) : 0.5) * kLoopScale;
    __syncthreads();
    if (owner && sm.bad[lane]) {
        // see shoot_rays: a block with a non-finite sum is redone with one reciprocal per ray, in the same
        // runs and groups
        B1 = B2 = 0.0;
        float m1 = 0.0f, m2 = 0.0f;
        for (int64_t r = 0; r < a.n_lens; r += T) {
            float s1 = 0.0f, s2 = 0.0f;
            const int64_t e = min(r + (int64_t)T, a.n_lens);
            for (int64_t li = r; li < e; ++li) {
                const float4 l = loop_lens(a, li);
                const float dx = X1 - l.x, dy = X2 - l.y;
                const float d = l.z * __builtin_amdgcn_rcpf(fmaf(dy, dy, dx * dx));
                s1 = fmaf(d, dx, s1);
                s2 = fmaf(d, dy, s2);
            }
            const bool first = (r / T) % kQuadRuns == 0, last = (r / T) % kQuadRuns == kQuadRuns - 1 || e == a.n_lens;
            m1 = first ? s1 : m1 + s1;
            m2 = first ? s2 : m2 + s2;
            if (last) {
                B1 += (double)m1;
                B2 += (double)m2;
            }
        }
    }
    B1 *= kLoopBack;
    B2 *= kLoopBack;

    // Lens equation (eq. 6), source pixel and binning as in shoot_rays, one ray per thread.
    const bool ok = owner && c0 < cmax && row >= rmin && row < rmax;
    const double y1 = a.lam1 * ((double)X1 * 16.0) - B1;
    const double y2 = a.lam2 * ((double)X2 * 16.0) - B2;
    int p1 = 0, p2 = 0;
    const int kv = pixel_of(y1, y2, a, p1, p2);
    const int key = ok ? kv : -2;
    if (DUMP && ok) {
        const int64_t ri = (row - a.rskip) * a.wn1 + c0;
        a.ray_y[2 * ri] = y1;
        a.ray_y[2 * ri + 1] = y2;
        a.ray_pix[ri] = kv;
    }
    // A row whose rays in the map are one run of one pixel leaves its count to the first wave, which adds equal
    // pixels of the four rows up: where all rays meet a few pixels, additions to one cache line (10 ns each) bound
    // the launch (2048^2 rays on one pixel, 100 lenses: 103 us, so 79; a batch of four such, 512 lenses: 2777, 1092).
    // An LDS window of the map instead cost more than it saved on every map (100 lenses, 64 x 64: 105 us).
    uint32_t *part = a.partial + (size_t)(group & (kPartials - 1)) * (size_t)a.pstride;
    if (owner) {
        uint32_t cnt;
        const bool head = run_head(key, lane, cnt), hit = head && key >= 0;
        const unsigned long long hits = __ballot(hit);
        const bool one = (hits & (hits - 1)) == 0;
        if (hit) {
            if (one) sm.only[wave] = make_int2(key, (int)cnt);
            else atomicAdd(&part[key], cnt);
        } else if (head && key == -1) {
            atomicAdd(&sm.lost, cnt);
        }
    }
    __syncthreads();
    if (tid < 4 && sm.only[tid].y > 0) {
        const int k = sm.only[tid].x;
        int cnt = 0;
        bool first = true;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int2 o = sm.only[w];
            const bool same = o.x == k && o.y > 0;
            cnt += same ? o.y : 0;
            first = first && !(same && w < tid);
        }
        if (first) atomicAdd(&part[k], (uint32_t)cnt);
    }
    if (tid == 0 && sm.lost) atomicAdd(lost_slot(a, group), (unsigned long long)sm.lost);
}

// Block `tile` of the window: 64 columns x 4 rows.
template <int T, int B, int WV, bool DUMP, bool JIT, class Args>
__device__ __forceinline__ void split_tile(const Args &a, uint32_t tile, uint32_t group, SplitSmem<B, WV> &sm)
{
    const uint32_t ty = tile / (uint32_t)a.tiles_x, tx = tile - ty * (uint32_t)a.tiles_x;
    shoot_split<T, B, WV, JIT ? kJitter : kSharedRows, DUMP>(a, tx * 64 + (threadIdx.x & 63), ty * 4, a.wn1, a.rskip, a.wn2,
                                                            group, sm);
}

template <int WV>
constexpr int kSimdWaves = WV == 16 ? 4 : 6;

// Six waves per SIMD (80 VGPRs, three spilled outside the lens loop): 193.0 ms on the 1e5-lens map, five (88
// VGPRs) 196.8, eight (64, the loop spills) 201.3.  Sixteen-wave workgroups run one to a SIMD group of four.
template <int T, int B, int WV, bool DUMP, bool JIT>
__global__ void __launch_bounds__(64 * WV, kSimdWaves<WV>) k_split(const DirectArgs a)
{
    __shared__ SplitSmem<B, WV> sm;
    const uint32_t tile = (uint32_t)group_number();
    split_tile<T, B, WV, DUMP, JIT>(a, tile, tile, sm);
}

// Persistent form over the blocks of the kept culling cells.  The blocks of a row of cells are counted through
// group of four ray rows by group, the columns of the row's kept cells in order, so that 64 of them lie on at most
// kRowGroups groups and share the rows' differences as k_split's do (groups of fewer than kMinColumns columns are
// padded).  Workgroups take 64 blocks at a time from the counter cb.queue until none are left.  89 170 kept cells
// of 3 x 24 rays, 1e5 lenses: 76.2 ms, each lane subtracting rows of its own 80.0.
template <int T, int B, int WV, bool JIT>
__global__ void __launch_bounds__(64 * WV, kSimdWaves<WV>) k_split_cells(const DirectArgs a, const CellBlocks cb)
{
    __shared__ SplitSmem<B, WV, JIT ? 1 : kRowGroups> sm;
    __shared__ uint32_t s_item;
    const int lane = threadIdx.x & 63;
    const uint64_t n = cb.start[cb.ncy];
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(cb.queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= n) break;
        // the row of cells with start[my] <= item < start[my + 1], a 64th of the rows left at a time
        int64_t my = 0;
        for (int64_t left = cb.ncy; left > 1;) {
            const int64_t step = (left + 63) / 64, at = lane * step;
            const int k = __popcll(__ballot(at < left && cb.start[my + (at < left ? at : 0)] <= item)) - 1;
            my += k * step;
            left = min(step, left - k * step);
        }
        const uint32_t cols = cb.cells[my] * (uint32_t)cb.c1, padded = max(cols, (uint32_t)kMinColumns);
        const uint64_t j0 = (item - cb.start[my]) * 64;
        const uint32_t g0 = (uint32_t)(j0 / padded), rest = (uint32_t)(j0 - (uint64_t)g0 * padded);
        const uint32_t g = g0 + (rest + lane) / padded, col = (rest + lane) % padded;
        const uint32_t groups = (uint32_t)cb.groups, last = min(g0 + (rest + 63) / padded, groups - 1);
        const int64_t rmin = my * cb.c2 + a.rskip, base = rmin & ~int64_t(3);
        int64_t c0 = 0, cmax = 0;
        if (g < groups && col < cols) {
            const uint32_t k = col / (uint32_t)cb.c1;
            const int64_t mx = cb.list[my * cb.ncx + k];
            c0 = mx * cb.c1 + (col - k * (uint32_t)cb.c1);
            cmax = min((mx + 1) * cb.c1, a.wn1);
        }
        const RowGroups rg{(uint32_t)(base + 4 * (int64_t)g0), (int)(last - g0) + 1, JIT ? 0 : (int)(min(g, last) - g0)};
        shoot_split<T, B, WV, JIT ? kJitter : kGroupRows, false>(a, (uint32_t)c0, (uint32_t)(base + 4 * (int64_t)min(g, last)),
                                                                 cmax, rmin, min((my + 1) * cb.c2 + a.rskip, a.wn2), item,
                                                                 sm, rg);
        __syncthreads();
    }
}

// A table that no thread of the launch writes, read as kernel arguments are: with scalar loads.
template <class S>
using Table = const __attribute__((address_space(4))) S;

// Persistent form over a table of jobs; see k_batched.  An item is per_item consecutive blocks of its job.  The item
// and the job's record are kept scalar (with an index that might differ from lane to lane, every use of a field was
// a vector load: 33.5e6 rays, 100 lenses: 986 us, 647 with scalar ones; 500 lenses 2274, 2118).
template <int T, int B, int WV>
__global__ void __launch_bounds__(64 * WV, kSimdWaves<WV>) k_split_batched(const BatchArgs b)
{
    __shared__ SplitSmem<B, WV> sm;
    __shared__ uint32_t s_item;
    Table<DirectArgs> *jobs = (Table<DirectArgs> *)b.jobs;
    Table<uint32_t> *start = (Table<uint32_t> *)b.item_start;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(b.queue, 1u);
        __syncthreads();
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (item >= b.n_items) break;
        int lo = 0, hi = b.n_jobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (start[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        Table<DirectArgs> &a = jobs[lo];
        const uint32_t first = (item - start[lo]) * a.per_item;
        const uint32_t end = min(first + a.per_item, a.n_blocks);
        for (uint32_t t = first; t < end; ++t) {
            if (a.jitter)
                split_tile<T, B, WV, false, true>(a, t, 0u, sm);
            else
                split_tile<T, B, WV, false, false>(a, t, 0u, sm);
            __syncthreads();
        }
    }
}

template <int T, int B, int WV>
hipError_t launch(const DirectArgs &a, hipStream_t s)
{
    const dim3 g = group_dim3(a.n_blocks, 64 * WV), blk(64 * WV);
    if (a.jitter) {
        if (a.ray_y) hipLaunchKernelGGL((k_split<T, B, WV, true, true>), g, blk, 0, s, a);
        else hipLaunchKernelGGL((k_split<T, B, WV, false, true>), g, blk, 0, s, a);
    } else {
        if (a.ray_y) hipLaunchKernelGGL((k_split<T, B, WV, true, false>), g, blk, 0, s, a);
        else hipLaunchKernelGGL((k_split<T, B, WV, false, false>), g, blk, 0, s, a);
    }
    return hipGetLastError();
}

template <int T, int B, int WV>
hipError_t launch_cells(const DirectArgs &a, const CellBlocks &cb, hipStream_t s)
{
    int occ = 0, dev = 0, cus = 0;
    const hipError_t e = a.jitter
        ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_split_cells<T, B, WV, true>, 64 * WV, 0)
        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_split_cells<T, B, WV, false>, 64 * WV, 0);
    if (e != hipSuccess) occ = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    // 64 blocks at a time of every row of cells, were all of them kept
    const int64_t cols = std::max<int64_t>(cb.ncx * cb.c1, kMinColumns);
    const int64_t fit = (int64_t)std::max(1, occ) * std::max(1, cus);
    const int64_t most = cb.ncy * ((cb.groups * cols + 63) / 64);
    const dim3 g((unsigned)std::min(fit, most)), blk(64 * WV);
    if (a.jitter) hipLaunchKernelGGL((k_split_cells<T, B, WV, true>), g, blk, 0, s, a, cb);
    else hipLaunchKernelGGL((k_split_cells<T, B, WV, false>), g, blk, 0, s, a, cb);
    return hipGetLastError();
}

template <int T, int B, int WV>
hipError_t launch_batch(const BatchArgs &b, int grid, hipStream_t s)
{
    hipLaunchKernelGGL((k_split_batched<T, B, WV>), dim3(grid), dim3(64 * WV), 0, s, b);
    return hipGetLastError();
}

template <int T, int B, int WV>
int occupancy_batch()
{
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_split_batched<T, B, WV>, 64 * WV, 0);
    return e == hipSuccess ? n : 0;
}

}  // namespace

// Call F<T, B, WV>(args) for the run length and waves of a launch.  B lenses are staged at a time, 64, or for runs of 32
// the 128 of a group, then with four waves (300 x 200 rays, 3000 lenses: 66 us, k_direct 267).  Staging 128 with the shorter
// runs spilled registers and left few blocks fewer waves (the same rays, runs of 8: 72 us, with 64 39).
#define RS_SPLIT_SWITCH(T, WV, F, ...)                                         \
    do {                                                                       \
        if ((T) == 32) return F<32, 128, 4>(__VA_ARGS__);                      \
        if ((T) == 16 && (WV) == 16) return F<16, 64, 16>(__VA_ARGS__);        \
        if ((T) == 16 && (WV) == 8) return F<16, 64, 8>(__VA_ARGS__);          \
        if ((T) == 16) return F<16, 64, 4>(__VA_ARGS__);                       \
        if ((WV) == 16) return F<8, 64, 16>(__VA_ARGS__);                      \
        if ((WV) == 8) return F<8, 64, 8>(__VA_ARGS__);                        \
        return F<8, 64, 4>(__VA_ARGS__);                                       \
    } while (0)

hipError_t launch_split(const DirectArgs &a, int T, hipStream_t s)
{
    if (a.n_blocks == 0) return hipSuccess;
    // Sixteen waves while that gives a compute unit no more than one workgroup (128^2 rays, 12800 lenses:
    // 122 us, with eight waves 151, with four 256; but 512 x 640 rays 610, 560, 610); eight where lenses
    // enough for all of them meet few blocks (512 x 640 rays, 400 lenses: 28.4 us against 29.3, 200 lenses
    // 21.4 against 20.3) or the field is large (1000^2 rays, 3200 lenses: 427 us against 432, 400 lenses
    // 67.1 against 65.8; jittered rays, which share no rows, later: 4096 x 2048, 2048 lenses 2675 us, with four
    // 2653, but 1000^2, 6000 lenses 980, 991).
    const int64_t large = a.jitter ? 4096 : 2048;
    const int wv = a.n_blocks <= 256 ? 16 : (a.n_lens >= large || (a.n_lens >= 256 && a.n_blocks <= 2048)) ? 8 : 4;
    RS_SPLIT_SWITCH(T, wv, launch, a, s);
}

hipError_t launch_split_cells(const DirectArgs &a, int T, const CellBlocks &cb, hipStream_t s)
{
    if (cb.ncx <= 0 || cb.ncy <= 0) return hipSuccess;
    const int wv = a.n_lens >= 2048 ? 8 : 4;
    RS_SPLIT_SWITCH(T, wv, launch_cells, a, cb, s);
}

// Four waves a workgroup: eight leave more of them without lenses in fields of few groups (64 maps of 300^2 rays, us with
// four and eight: 512 lenses 414, 454; 1000 793, 810; 10 000 7113, 7167), but batches of few blocks end sooner with
// eight (one map of 256^2 rays: 512 lenses 24, 21; 1000 34, 27; 10 000 207, 129; one of 1000^2, 3000 lenses 405, 393).
// Between, mixed batches gain a little with eight too (24 maps of 93^2 to 372^2 rays, 90 to 9000 lenses: 258, 233).
int split_batched_waves(uint64_t blocks, int64_t most_lenses) { return blocks < 4096 && most_lenses >= 256 ? 8 : 4; }

hipError_t launch_split_batched(const BatchArgs &b, int T, int WV, int grid, hipStream_t s)
{
    RS_SPLIT_SWITCH(T, WV, launch_batch, b, grid, s);
}

int split_batched_occupancy(int T, int WV) { RS_SPLIT_SWITCH(T, WV, occupancy_batch); }

}  // namespace rs

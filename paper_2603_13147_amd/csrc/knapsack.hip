// knapsack.hip - one 0-1 knapsack (paper Section 5.8) on gfx950.
//
// A row of the DP table needs the whole row before it, so a single sweep of
// the rows (knap_rows.h) keeps one CU busy and leaves the other 255 idle.
// The maximum over item sets splits, though: with the items cut into groups,
// the best value at capacity c is the largest A[a] + B[c - a], A and B the
// last rows of the two halves' own tables.  So a knapsack of many items is
// solved as
//  - k_knap_rows: one workgroup per group of items sweeps the group's rows;
//  - k_knap_merge, once per level of a binary tree: the rows of two
//    neighbouring groups are merged, (W + 1)^2 / 2 additions and maxima spread
//    over the whole chip.
// 4000 items at W = 6400 take 195 us in 32 groups (62 in the row sweeps, 70
// in the merges' pairs, the rest in eight launches) against 2.05 ms whole;
// knap_groups has the rule and the figures behind it.
// Every value is an exact integer maximum, so the split changes no result.
// Additions saturate as in the row sweep: a value beyond int32 anywhere
// leaves G[items][W] beyond it.
#include <string.h>

#include "knap_rows.h"
#include "llp_dev.h"
#include "llp_host.h"

namespace llp {

constexpr int KM_BLOCK = 256;               // threads per workgroup of a merge
constexpr int KM_OUT = 512;                 // cells of the merged row per workgroup: 8 per lane
constexpr int KM_CHUNK = 256;               // cells of A per step of a workgroup: 64 per wave
constexpr int KM_COL = (KM_OUT + KM_CHUNK) / 8;

// Group blockIdx.x sweeps items [x * per, (x + 1) * per).  With rows set, the
// group's last row goes to rows + x * stride and its status to gstatus[x], and
// the launch clears zero[0 .. nzero) for the merge that follows; without,
// the one group's results are the knapsack's.
template <int CH>
__global__ void __launch_bounds__(ch_max_block(CH)) k_knap_rows(const int* wt, const int* val, int items, int W, int per,
                                                                int dbuf, int* rows, int stride, int* gstatus, int* zero,
                                                                int nzero, int* best, int* row) {
    extern __shared__ unsigned krow[];
    const int x = blockIdx.x, k0 = min(x * per, items);
    for (int i = x * blockDim.x + threadIdx.x; i < nzero; i += gridDim.x * blockDim.x) zero[i] = 0;
    const int st = knap_wg<CH>(wt + k0, val + k0, min(per, items - k0), W, krow, dbuf ? krow + (W + 1) : nullptr, best,
                               rows ? rows + (size_t)x * stride : row);
    // a split solve's overflow is read off its last row
    if (threadIdx.x == 0) gstatus[x] = rows && st == LLP_E_OVERFLOW ? LLP_OK : st;
}

// Merge of rows 2y and 2y + 1 of `in` into row y of `out` (cleared before), y
// = blockIdx.y: out[c] = max over a <= c of A[a] + B[c - a].
//
// What bounds it is the additions and maxima, (W + 1)^2 / 2 pairs at 1.5
// instructions each (2.3 us per merge at W = 6400 when several run at once, 9e12
// pairs a second).  A workgroup takes 512 cells c = c0 + 8 l + r (lane l, r <
// 8) and `steps` runs of 256 cells a, a quarter per wave.  A[a] is uniform in
// the wave; the 8 x 8 pairs of a lane's cells with 8 values of a need 15
// consecutive cells of B, of which a step loads 8 new ones and keeps 7.  B
// lies in LDS as 8 columns by the index modulo 8, so those loads are
// consecutive across the lanes.  The waves' maxima meet in LDS, the
// workgroups' by atomicMax.
__global__ void __launch_bounds__(KM_BLOCK) k_knap_merge(const unsigned* __restrict__ in, unsigned* __restrict__ out,
                                                         int W, int stride, int steps, int* __restrict__ zero, int nzero) {
    __shared__ unsigned bt[8][KM_COL];
    __shared__ unsigned red[KM_BLOCK / LLP_WAVE][8][LLP_WAVE];
    const int t = threadIdx.x, l = t & 63;
    const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
    const int gid = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    for (int i = gid * KM_BLOCK + t; i < nzero; i += gridDim.x * gridDim.y * gridDim.z * KM_BLOCK) zero[i] = 0;
    // the last cells have the most pairs: their workgroups start first
    const int c0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * KM_OUT;
    const int alast = min(c0 + KM_OUT - 1, W);
    int a0 = blockIdx.z * steps * KM_CHUNK;
    if (a0 > alast) return;
    const int aend = min(a0 + steps * KM_CHUNK, alast + 1);
    const unsigned* A = in + (size_t)(2 * blockIdx.y) * stride;
    const unsigned* B = A + stride;
    unsigned acc[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) acc[r] = 0u;
    for (; a0 < aend; a0 += KM_CHUNK) {
        // B[c0 - a0 - 255 + i], i in [0, 768): outside the row any cell serves,
        // the pairs that would use it are masked or past the row
        __syncthreads();
        for (int i = t; i < 8 * KM_COL; i += KM_BLOCK)
            bt[i & 7][i >> 3] = B[max(0, min(c0 - a0 - (KM_CHUNK - 1) + i, W))];
        __syncthreads();
        const int aw = a0 + 64 * wid;      // the wave's 64 cells of A
        const int kk = 31 - 8 * wid;       // column of the window's first cell, step 0
        unsigned u[15];
#pragma unroll
        for (int d = 0; d < 7; ++d) u[d] = bt[d][l + kk + 1];   // becomes the upper part
        if (aw + 63 <= c0) {
            for (int s = 0; s < 8; ++s) {
#pragma unroll
                for (int d = 14; d >= 8; --d) u[d] = u[d - 8];
#pragma unroll
                for (int d = 0; d < 8; ++d) u[d] = bt[d][l + kk - s];
                unsigned av[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) av[q] = A[aw + 8 * s + q];
#pragma unroll
                for (int q = 0; q < 8; q += 2)
#pragma unroll
                    for (int r = 0; r < 8; ++r)
                        acc[r] = max(acc[r], max(__builtin_elementwise_add_sat(u[r - q + 7], av[q]),
                                                 __builtin_elementwise_add_sat(u[r - q + 6], av[q + 1])));
            }
        } else {
            // some of these cells of A lie above some of the lane's cells
            for (int s = 0; s < 8; ++s) {
#pragma unroll
                for (int d = 14; d >= 8; --d) u[d] = u[d - 8];
#pragma unroll
                for (int d = 0; d < 8; ++d) u[d] = bt[d][l + kk - s];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int a = aw + 8 * s + q;
                    const unsigned av = A[min(a, W)];
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const unsigned x = __builtin_elementwise_add_sat(u[r - q + 7], av);
                        acc[r] = max(acc[r], a <= c0 + 8 * l + r ? x : 0u);
                    }
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r) red[wid][r][l] = acc[r];
    __syncthreads();
    for (int i = t; i < KM_OUT; i += KM_BLOCK) {
        const int r = i >> 6, c = c0 + 8 * l + r;
        unsigned x = red[0][r][l];
#pragma unroll
        for (int w = 1; w < KM_BLOCK / LLP_WAVE; ++w) x = max(x, red[w][r][l]);
        if (c <= W && x > 0u) {
            __hip_atomic_fetch_max(&out[(size_t)blockIdx.y * stride + c], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Results of a split solve: the last row, its last cell, the status.
__global__ void __launch_bounds__(256) k_knap_finish(const unsigned* last, int W, const int* gstatus, int groups,
                                                     int* best, int* row, int* status) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (row && c <= W) row[c] = (int)last[c];
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        const bool bad = threadIdx.x < groups && gstatus[threadIdx.x] != LLP_OK;
        const bool any = __any(bad);
        if (threadIdx.x == 0) {
            *best = (int)last[W];
            *status = any ? LLP_E_INPUT : (last[W] > (unsigned)LLP_INF ? LLP_E_OVERFLOW : LLP_OK);
        }
    }
}

// --------------------------------------------------------------- host
int solve_knapsack(int32_t items, int32_t W, const int32_t* wt, const int32_t* val, int32_t* best,
                   int32_t* last_row, const llp_opts* opts) {
    if (items < 0) return fail(LLP_E_ARG, "items must be >= 0 (got %d)", items);
    if (W < 0 || W > KN_MAX_W) return fail(LLP_E_ARG, "W must be in [0, %d] (got %d)", KN_MAX_W, W);
    if (!best) return fail(LLP_E_ARG, "best is required");
    if (items > 0 && (!wt || !val)) return fail(LLP_E_ARG, "wt and val are required");
    llp_opts o = opts_or_default(opts);
    hipStream_t st = (hipStream_t)o.stream;
    const int T = o.block > 0 ? o.block : 1024;
    if (T % 64 != 0 || T > 1024) return fail(LLP_E_ARG, "block must be a multiple of 64 up to 1024");
    const int ch = pick_ch(W, T);
    if (!ch) return fail(LLP_E_ARG, "W = %d needs more than 32 cells per thread at %d threads", W, T);
    const size_t row_bytes = (size_t)(W + 1) * 4;
    const int dbuf = 2 * row_bytes <= lds_per_workgroup();
    const size_t lds = dbuf ? 2 * row_bytes : row_bytes;
    if (lds > lds_per_workgroup()) return fail(LLP_E_ARG, "a row of W = %d does not fit in LDS", W);
    // Split only in a workspace of the caller's that holds the rows (the
    // library's own is shared by every call on the device), and not when the
    // caller asks for a launch shape.
    int groups = o.workspace && o.block <= 0 ? knap_groups(items, W) : 1;
    if (groups > 1 && o.workspace_bytes < knap_bytes(groups, W)) groups = 1;
    void* ws = nullptr;
    int s = get_workspace(o, KN_HEADER_BYTES, &ws);
    if (s) return s;
    int* status = (int*)ws;   // then, from word 32, the groups' statuses
    int* gstatus = groups > 1 ? status + 32 : status;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool timing = (o.flags & LLP_TIMING) && o.stats;
    if (timing) {
        LLP_HIP(hipEventCreate(&ev0));
        LLP_HIP(hipEventCreate(&ev1));
        LLP_HIP(hipEventRecord(ev0, st));
    }
    const int stride = (int)knap_stride(W);
    int* rows = (int*)((char*)ws + KN_HEADER_BYTES);
    s = dispatch_ch(ch, [&](auto c) {
        constexpr int CH = decltype(c)::value;
        if (lds > 65536) (void)hipFuncSetAttribute((const void*)k_knap_rows<CH>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        const bool split = groups > 1;
        hipLaunchKernelGGL(k_knap_rows<CH>, dim3(groups), dim3(T), lds, st, wt, val, items, W,
                           items / groups + (items % groups != 0), dbuf, split ? rows : nullptr, stride, gstatus,
                           split ? rows + (size_t)groups * stride : nullptr, split ? groups / 2 * stride : 0,
                           split ? nullptr : best, split ? nullptr : last_row);
        return hip_check(hipGetLastError(), "k_knap_rows");
    });
    if (s) return s;
    if (groups > 1) {
        const int tiles = (W + KM_OUT) / KM_OUT, chunks = (W + KM_CHUNK) / KM_CHUNK;
        for (int n = groups / 2; n >= 1; n /= 2) {
            // about four workgroups per CU in all; a pair has tiles * chunks / 2
            // runs of cells to work through
            const int want = 4 * device_info().cus;
            int steps = (int)((long long)n * tiles * chunks / 2 / want);
            steps = steps < 1 ? 1 : (steps > chunks ? chunks : steps);
            int* out = rows + (size_t)2 * n * stride;
            hipLaunchKernelGGL(k_knap_merge, dim3(tiles, n, (chunks + steps - 1) / steps), dim3(KM_BLOCK), 0, st,
                               (const unsigned*)rows, (unsigned*)out, W, stride, steps, n > 1 ? out + (size_t)n * stride : nullptr,
                               n / 2 * stride);
            rows = out;
        }
        hipLaunchKernelGGL(k_knap_finish, dim3(last_row ? (W + 256) / 256 : 1), dim3(256), 0, st, (const unsigned*)rows, W,
                           gstatus, groups, best, last_row, status);
        LLP_HIP(hipGetLastError());
    }
    if (timing) LLP_HIP(hipEventRecord(ev1, st));
    if (o.flags & LLP_ASYNC) {
        if (o.status_dev) LLP_HIP(hipMemcpyAsync(o.status_dev, status, 4, hipMemcpyDeviceToDevice, st));
        return LLP_OK;
    }
    int h = 0;
    s = readback(st, status, &h, sizeof(h));
    if (s) return s;
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = items;
        o.stats->advances = (int64_t)items * (W + 1);
        if (timing) {
            float ms = 0.f;
            LLP_HIP(hipEventElapsedTime(&ms, ev0, ev1));
            o.stats->device_ms = ms;
        }
    }
    if (timing) {
        (void)hipEventDestroy(ev0);
        (void)hipEventDestroy(ev1);
    }
    if (h == LLP_E_INPUT) return fail(h, "negative weight or value");
    if (h == LLP_E_OVERFLOW) return fail(h, "a DP value does not fit int32");
    if (h) return fail(h, "device status %d", h);
    return LLP_OK;
}

}  // namespace llp

extern "C" int llp_solve_knapsack(int32_t items, int32_t W, const int32_t* wt, const int32_t* val, int32_t* best,
                                  int32_t* last_row, const llp_opts* opts) {
    return llp::solve_knapsack(items, W, wt, val, best, last_row, opts);
}

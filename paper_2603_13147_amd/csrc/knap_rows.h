// knap_rows.h - the row sweep of one 0-1 knapsack by one workgroup (paper
// Section 5.8), shared by the single solve (knapsack.hip) and the batch
// (batch.hip).
//
// Cell (k, c) of the DP table is forbidden below max(G[k-1][c], v_k +
// G[k-1][c - w_k]); once row k-1 is final every cell of row k is forbidden
// exactly until it takes that value, so the workgroup advances a whole row
// per item.  Wave v keeps the cells [64 CH v, 64 CH (v + 1)) of the current row
// in registers, lane l those at l + 64 i; per item the row is published to
// LDS, one barrier, and every wave reads the cells w_k below its own.  With
// room for two LDS rows the buffers alternate and one barrier per item
// suffices; otherwise a second barrier protects the single buffer.  Items
// heavier than W or worth nothing leave the row unchanged and are skipped.
//
// What bounds it is the instructions per cell, then the barrier, not the LDS.
// So CH is the instance's own count of cells per thread, ceil((W + 1) / T);
// a wave whose cells all lie at or above w reads them at constant offsets
// from one address and spends one addition and one maximum on each, a wave
// whose cells all lie below w spends nothing, and only the wave (at most
// two) that straddles w or the end of the row checks its cells one by one.
// A value beyond int32 is not looked for cell by cell either: values are
// unsigned and additions saturate.  G is non-decreasing in k and in c, so
// some value exceeded 2^31 - 1 exactly if G[items][W] ends above it, and a
// saturated cell stays above it.  One knapsack of 4000 items and W = 6400
// (1024 threads): 2.02 ms, against 4.61 with every cell compared with W and w
// and its sum with 2^31 - 1; 4096 knapsacks in a batch: 0.40 against 1.23 ms.
#pragma once

#include <utility>

#include "llp_dev.h"
#include "llp_host.h"

namespace llp {

constexpr int KN_MAX_CH = 32;      // cells per thread at most

// Largest workgroup a kernel holding up to ch row cells per thread in
// registers is built for (16384 cells per workgroup keeps the register budget).
constexpr int ch_max_block(int ch) { return 16384 / ch > 1024 ? 1024 : 16384 / ch; }

// Cells per thread of a row of W + 1 cells at T threads, rounded up to a count
// the row sweep is compiled for: every count up to 16 (the average instance
// of a batch leaves no cell idle), then every fourth.
__host__ __device__ inline int knap_ch(int W, int T) {
    const int need = W / T + 1;
    return need <= 16 ? need : (need + 3) & ~3;
}

// One item: publish the row, then advance every cell from the shifted row.
// base: the wave's first cell (uniform).  Cells past W are not published.
template <int CH>
__device__ __forceinline__ void knap_item(unsigned (&g)[CH], unsigned* buf, int base, int W, int w, unsigned v) {
    int l = lane();
    asm volatile("" : "+v"(l));   // cell numbers are formed here, not kept in registers from item to item
    unsigned* p = buf + base + l;
    if (base + 64 * CH <= W + 1) {
#pragma unroll
        for (int i = 0; i < CH; ++i) p[64 * i] = g[i];
    } else {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (base + l + 64 * i <= W) p[64 * i] = g[i];
    }
    __syncthreads();
    const int d = base - w;   // the cell the wave's first one reads
    if (d >= 0 && d + 64 * CH <= W + 1) {
        const unsigned* q = buf + d + l;
        unsigned y[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) y[i] = q[64 * i];
#pragma unroll
        for (int i = 0; i < CH; ++i) g[i] = max(g[i], __builtin_elementwise_add_sat(y[i], v));
    } else if (d + 64 * CH > 0 && base <= W) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = d + l + 64 * i;
            const unsigned y = buf[max(0, min(c, W))];
            // below w: cell 0 plus nothing never exceeds the cell
            g[i] = max(g[i], __builtin_elementwise_add_sat(y, c >= 0 ? v : 0u));
        }
    }
}

// Sweep items 0 .. items-1 over the row in g (bottom 0).  buf0 / buf1: LDS rows
// of W + 1 words (buf1 == nullptr: single buffer).  Returns LLP_OK or
// LLP_E_INPUT (a negative weight or value), uniform in the workgroup.
template <int CH>
__device__ __forceinline__ int knap_sweep(const int* wt, const int* val, int items, int W, unsigned* buf0,
                                          unsigned* buf1, unsigned (&g)[CH]) {
    const int l = lane();
    const int base = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * 64 * CH;
#pragma unroll
    for (int i = 0; i < CH; ++i) g[i] = 0u;
    // words from one buffer to the other (two pointers and a choice between them
    // cost the batch kernel spilled scalar registers)
    const int flip = buf1 ? (int)(buf1 - buf0) : 0;
    int off = 0;
    // 64 items per load, one per lane; the next 64 are loaded meanwhile
    int wn = l < items ? wt[l] : 0, vn = l < items ? val[l] : 0;
    for (int k0 = 0; k0 < items; k0 += 64) {
        const int wv = wn, vv = vn;
        if (__any(wv < 0 || vv < 0)) return LLP_E_INPUT;
        const int kn = k0 + 64 + l;
        wn = kn < items ? wt[kn] : 0;
        vn = kn < items ? val[kn] : 0;
        // items heavier than W or worth nothing (padding among them) drop out
        for (uint64_t todo = ballot(wv <= W && vv != 0); todo; todo &= todo - 1) {
            const int j = __ffsll((long long)todo) - 1;
            const int w = __builtin_amdgcn_readlane(wv, j), v = __builtin_amdgcn_readlane(vv, j);
            knap_item<CH>(g, buf0 + off, base, W, w, (unsigned)v);
            if (!flip) __syncthreads();
            off = flip - off;
        }
    }
    return LLP_OK;
}

// Calls f with the compiled count of cells per thread equal to ch (a value
// of knap_ch up to MAX); nothing for any other ch.
template <int MAX, class F, int... I>
__device__ __forceinline__ void knap_dispatch(int ch, F&& f, std::integer_sequence<int, I...>) {
    auto one = [&](auto c) __attribute__((always_inline)) {
        constexpr int CH = decltype(c)::value;
        if constexpr (CH <= MAX && (CH <= 16 || CH % 4 == 0)) {
            if (ch == CH) f(c);
        }
    };
    (one(std::integral_constant<int, I + 1>()), ...);
}
template <int MAX, class F>
__device__ __forceinline__ void knap_dispatch(int ch, F&& f) {
    knap_dispatch<MAX>(ch, f, std::make_integer_sequence<int, MAX>());
}

// Solve one knapsack with the calling workgroup (knap_ch(W, T) <= MAX).  The
// best value goes to *best, the last row to row (both nullable).  Returns the status, uniform in the workgroup.
template <int MAX>
__device__ __forceinline__ int knap_wg(const int* wt, const int* val, int items, int W, unsigned* buf0, unsigned* buf1, int* best,
                       int* row) {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));   // as in knap_item: no cell numbers kept from instance to instance
    int st = LLP_OK;
    bool over = false;
    knap_dispatch<MAX>(knap_ch(W, blockDim.x), [&](auto c) __attribute__((always_inline)) {
        constexpr int CH = decltype(c)::value;
        unsigned g[CH];
        st = knap_sweep<CH>(wt, val, items, W, buf0, buf1, g);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int x = (t >> 6) * 64 * CH + (t & 63) + 64 * i;
            if (x <= W && row) row[x] = (int)g[i];
            if (x == W) {
                if (best) *best = (int)g[i];
                over = g[i] > (unsigned)LLP_INF;
            }
        }
    });
    return __syncthreads_or(over) && st == LLP_OK ? LLP_E_OVERFLOW : st;
}

// --------------------------------------------------------------- host
// Kernels are compiled for these largest counts of cells per thread: powers of
// two, and 10 for rows of 4096 to 5119 cells by 512 threads, the widest that the
// batch kernel takes with registers for 8 waves per SIMD (see k_batch).
static const int CH_OPTS[] = {4, 8, 10, 16, 32};

static int pick_ch(int W, int T) {
    for (int ch : CH_OPTS)
        if ((long long)ch * T >= (long long)W + 1 && T <= ch_max_block(ch)) return ch;
    return 0;
}

template <class F>
static int dispatch_ch(int ch, F&& f) {
    switch (ch) {
        case 4: return f(std::integral_constant<int, 4>());
        case 8: return f(std::integral_constant<int, 8>());
        case 10: return f(std::integral_constant<int, 10>());
        case 16: return f(std::integral_constant<int, 16>());
        case 32: return f(std::integral_constant<int, 32>());
        default: return fail(LLP_E_ARG, "no kernel for %d cells per thread", ch);
    }
}

static inline size_t lds_per_workgroup() {
    const size_t l = device_info().lds_per_block;
    return l ? l : 65536;
}

}  // namespace llp

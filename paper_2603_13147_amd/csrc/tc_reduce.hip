// tc_reduce.hip - transitive closure (paper Section 5.7) and parallel
// reduction (Section 5.6) as LLP sweeps on gfx950.
//
// Transitive closure.  State: boolean G[u][v]; (u, v) is forbidden while false
// if (u, v) is an arc or G[u][w] and G[w][v] for some w.  A workgroup sweeps a
// group of rows u0 .. u0 + rows - 1 together, held in LDS by column: word
// R[v] has bit s set iff G[u0 + s][v].  A vertex w whose word grew is active;
// taking it sets, for every arc (w, x), the bits of R[w] (and w's own, if it is
// one of the group's rows) in R[x], and makes x active if that set any.  Each
// such (u, x) is forbidden in the current state (G[u][w] holds and the arc
// makes G[w][x] hold), so every advance is one of the paper's, and the group
// ends when no vertex is active: the least fixpoint, reachability by paths of
// length >= 1.  One visit of an arc serves all of the group's rows.
//
// Reduction.  The tree of tiles: each workgroup sums one tile of the input
// (grid-stride, modulo 2^64) and publishes it; the root becomes forbidden once
// all its children have published, which the launch boundary tells, and the
// second launch advances it to the sum of the partials.
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "llp_dev.h"
#include "llp_host.h"

namespace llp {

// --------------------------------------------------------------- closure
constexpr int TC_MAX_N = 65536;

struct TCtrl {
    int status;
    int pad;
    int diag[8];
    long long rounds;   // summed over the groups of rows
};

__global__ void k_tc_init(TCtrl* c) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        TCtrl z;
        memset(&z, 0, sizeof(z));
        *c = z;
    }
}

// Bits s of the group's rows for vertex x, BITS of them.
template <int BITS>
__device__ __forceinline__ unsigned tc_get(const unsigned* R, int x) {
    if constexpr (BITS == 32) return R[x];
    else return (R[x >> 1] >> ((x & 1) * 16)) & 0xffffu;
}

// Sets bits in x's word and makes x active if any was clear.
template <int BITS>
__device__ __forceinline__ void tc_set(unsigned* R, unsigned* act, int x, unsigned bits) {
    const int sh = BITS == 32 ? 0 : (x & 1) * 16;
    const unsigned old = atomicOr(&R[BITS == 32 ? x : x >> 1], bits << sh) >> sh;
    if (bits & ~old) atomicOr(&act[x >> 5], 1u << (x & 31));
}

// One workgroup per group of rows (a power of two, BITS at most).  LDS: the
// active bitmap (64-bit words, one per block of 64 vertices), then the words R.
// A wave takes the vertices of a block at once, a lane each, 8 arcs in flight
// per lane, the next block's row offsets loaded meanwhile; rows of more than
// TC_LONG arcs are walked by the whole wave.  What bounds it on wide searches
// is how the arcs are read: a lane per vertex touches a line per lane and
// fetches it again for its next arcs, about 5 clocks per arc and CU (64 K arcs:
// 137 us).  On deep searches it is the round, about 0.75 us of dependent LDS and
// L2 trips and of the instructions of 16 waves.  So where no active vertex of
// a block has more than TC_SHORT arcs a wave reads those alone, and a graph of
// few vertices makes as many groups as there are CUs, of fewer rows each, which
// leaves fewer vertices active in a round: a chain of 500 vertices takes 366 us
// (508 without either, 421 with a workgroup per row), of 1000 with ids permuted
// 800 (1380 and 835), of 8192 6.0 ms (8.3 and 20.3).
// Going on with a block while it has active vertices saves rounds but costs
// more visits: 427 us at the size below, 160 if only while 8 or fewer are, and if
// only in rounds of few vertices a permuted chain 50% more.  Most arcs set
// nothing new: a plain read of R[x] spares them the atomic.  A round is one scan
// of the bitmap (wave w looks at blocks w + 16 l, lane l; a group of fewer than
// 16 blocks has a wave per block), and a wave sees what the others did meanwhile.
// n = 8192, 65536 arcs: 131 us, against 2276 with a workgroup per row
// and a bitmap search each.
constexpr int TC_BLOCK = 1024;
constexpr int TC_LONG = 64;
constexpr int TC_SHORT = 2;   // 4: a chain of 500 vertices 414 us, a band of 4 arcs a vertex 161 instead of 177

template <int BITS>
__global__ void __launch_bounds__(TC_BLOCK) k_tc_rows(int n, int m, int rows, const int* __restrict__ ptr,
                                                      const int* __restrict__ dst, unsigned* __restrict__ bits,
                                                      TCtrl* ctl) {
    extern __shared__ unsigned long long tl[];
    // by round modulo 3: a vertex was taken; bad input was met (a wave past the
    // round's barrier may set the next round's before another has read this one's)
    __shared__ int any[3], bad[3];
    const int t = threadIdx.x, l = lane();
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nb = (n + 63) >> 6, T = blockDim.x, nw = T >> 6;   // nb <= 64 nw
    unsigned* act = (unsigned*)tl;
    unsigned* R = (unsigned*)(tl + nb);
    const int u0 = blockIdx.x * rows;
    for (int i = t; i < 2 * nb; i += T) {
        // the group's rows are active: bits u0 .. u0 + rows - 1 below n
        const int lo = u0 - 32 * i;
        unsigned f = 0u;
        if (lo >= 0 && lo < 32) f = (~0u >> (32 - rows)) << lo;
        if (32 * i + 32 > n) f &= 32 * i >= n ? 0u : (1u << (n & 31)) - 1u;
        act[i] = f;
    }
    const int rw = BITS == 32 ? n : (n + 1) >> 1;
    for (int i = t; i < rw; i += T) R[i] = 0u;
    if (t < 3) any[t] = bad[t] = 0;
    __syncthreads();
    int r = 0;
    bool failed = false;
    for (;; ++r) {
        bool b2 = false, did = false;
        if (t == 0) any[(r + 1) % 3] = bad[(r + 1) % 3] = 0;   // last read in round r - 2
        const int mine = wave + nw * l;
        uint64_t todo = ballot(mine < nb && tl[min(mine, nb - 1)] != 0ull);
        int blk = 0, pb = 0, pe = 0;   // the block to take, its rows' offsets on the way
        if (todo) {
            blk = wave + nw * (__ffsll((long long)todo) - 1);
            pb = ptr[min(blk * 64 + l, n)];
            pe = ptr[min(blk * 64 + l + 1, n)];
        }
        while (todo) {
            did = true;
            const int w = blk * 64 + l;
            unsigned long long f = 0;
            if (l == 0) f = atomicExch(&tl[blk], 0ull);
            // R is read after the bits are taken: what grows later sets them again
            asm volatile("" ::: "memory");
            const unsigned f0 = __builtin_amdgcn_readfirstlane((int)(unsigned)f);
            const unsigned f1 = __builtin_amdgcn_readfirstlane((int)(unsigned)(f >> 32));
            unsigned g = 0u;
            int b = 0, e = 0;
            if ((l < 32 ? f0 >> l : f1 >> (l - 32)) & 1u) {
                b = pb;
                e = pe;
                if (b < 0 || e > m || e < b) {
                    b2 = true;
                    b = e = 0;
                }
                g = tc_get<BITS>(R, w);
                if (w >= u0 && w < u0 + rows) g |= 1u << (w - u0);
            }
            todo &= todo - 1;
            if (todo) {
                blk = wave + nw * (__ffsll((long long)todo) - 1);
                pb = ptr[min(blk * 64 + l, n)];
                pe = ptr[min(blk * 64 + l + 1, n)];
            }
            const bool wide = e - b > TC_LONG;
            if (!__any(e - b > TC_SHORT)) {
                int x[TC_SHORT];
                unsigned have[TC_SHORT];
#pragma unroll
                for (int j = 0; j < TC_SHORT; ++j) x[j] = b + j < e ? dst[b + j] : 0;
#pragma unroll
                for (int j = 0; j < TC_SHORT; ++j) {
                    if ((unsigned)x[j] >= (unsigned)n) {
                        b2 = true;
                        x[j] = 0;
                    }
                    have[j] = tc_get<BITS>(R, x[j]);
                }
#pragma unroll
                for (int j = 0; j < TC_SHORT; ++j)
                    if (b + j < e && (g & ~have[j])) tc_set<BITS>(R, act, x[j], g);
                continue;
            }
            for (unsigned k0 = b; !wide && k0 < (unsigned)e; k0 += 8) {
                int x[8];
                unsigned have[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = dst[min(k0 + j, (unsigned)e - 1)];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if ((unsigned)x[j] >= (unsigned)n) {
                        b2 = true;
                        x[j] = w;
                    }
                    have[j] = tc_get<BITS>(R, x[j]);
                }
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k0 + j < (unsigned)e && (g & ~have[j])) tc_set<BITS>(R, act, x[j], g);
            }
            for (uint64_t q = ballot(wide); q; q &= q - 1) {
                const int src = __ffsll((long long)q) - 1;
                const unsigned eb = shfl(b, src), ee = shfl(e, src);
                const unsigned gg = (unsigned)shfl((int)g, src);
                for (unsigned k0 = eb + l; k0 < ee; k0 += 4 * LLP_WAVE) {
                    int x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = dst[min(k0 + j * LLP_WAVE, ee - 1)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if ((unsigned)x[j] >= (unsigned)n) b2 = true;
                        else if (gg & ~tc_get<BITS>(R, x[j])) tc_set<BITS>(R, act, x[j], gg);
                    }
                }
            }
        }
        if (did && l == 0) any[r % 3] = 1;
        if (b2) bad[r % 3] = 1;
        __syncthreads();
        failed = bad[r % 3] != 0;
        if (!any[r % 3] || failed) break;
    }
    // transpose: 64 columns per step, the words of row u0 + s in lane s
    const int words = (n + 31) >> 5;
    for (int blk = wave; blk < nb; blk += nw) {
        const int v = blk * 64 + l;
        const unsigned g = v < n ? tc_get<BITS>(R, v) : 0u;
        uint64_t out = 0;
        if (rows == BITS) {
#pragma unroll
            for (int s = 0; s < BITS; ++s) {
                const uint64_t col = ballot((g >> s) & 1u);
                out = l == s ? col : out;
            }
        } else {
            for (int s = 0; s < rows; ++s) {
                const uint64_t col = ballot((g >> s) & 1u);
                out = l == s ? col : out;
            }
        }
        if (l < rows && u0 + l < n) {
            unsigned* row = bits + (long long)(u0 + l) * words + 2 * blk;
            row[0] = (unsigned)out;
            if (2 * blk + 1 < words) row[1] = (unsigned)(out >> 32);
        }
    }
    if (t == 0) {
        if (failed) {
            set_status(&ctl->status, LLP_E_INPUT);
            record_diag(ctl->diag, 81, u0, n, 0, 0);
        }
        atomicAdd((unsigned long long*)&ctl->rounds, (unsigned long long)(r + 1));
    }
}

size_t tc_workspace_bytes(int64_t) { return 256; }

int solve_tc(int32_t n, int64_t m, const int32_t* out_ptr, const int32_t* out_dst, uint32_t* bits,
             const llp_opts* opts) {
    if (n <= 0 || n > TC_MAX_N) return fail(LLP_E_ARG, "n must be in [1, %d] (got %d)", TC_MAX_N, n);
    if (m < 0 || m > 0x7fffffffll) return fail(LLP_E_ARG, "m out of range");
    if (!out_ptr || !bits || (m > 0 && !out_dst)) return fail(LLP_E_ARG, "out_ptr, out_dst and bits are required");
    llp_opts o = opts_or_default(opts);
    hipStream_t st = (hipStream_t)o.stream;
    void* ws = nullptr;
    int s = get_workspace(o, 256, &ws);
    if (s) return s;
    TCtrl* ctl = (TCtrl*)ws;
    // 32 rows per group while their words fit in LDS (132 KB at n = 32768), else 16
    const bool narrow = n > 32768;
    // or fewer, one group per CU
    int rows = narrow ? 16 : 32;
    while (rows > 1 && n <= (int64_t)device_info().cus * (rows / 2)) rows /= 2;
    const size_t lds = (size_t)((n + 63) / 64) * 8 + (narrow ? (size_t)(n + 1) / 2 : (size_t)n) * 4;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool timing = (o.flags & LLP_TIMING) && o.stats;
    if (timing) {
        LLP_HIP(hipEventCreate(&ev0));
        LLP_HIP(hipEventCreate(&ev1));
        LLP_HIP(hipEventRecord(ev0, st));
    }
    hipLaunchKernelGGL(k_tc_init, dim3(1), dim3(64), 0, st, ctl);
    auto* kernel = narrow ? k_tc_rows<16> : k_tc_rows<32>;
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3((n + rows - 1) / rows),
                       dim3(std::min(TC_BLOCK, (n + 63) / 64 * 64)), lds, st, n, (int)m, rows, out_ptr, out_dst, bits,
                       ctl);
    LLP_HIP(hipGetLastError());
    if (timing) LLP_HIP(hipEventRecord(ev1, st));
    TCtrl h;
    s = readback(st, ctl, &h, sizeof(h));
    if (s) return s;
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = h.rounds;
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
    if (h.status) return fail(h.status, "malformed out-CSR (offsets or ids out of range on a path from rows %d and up)", h.diag[1]);
    return LLP_OK;
}

// --------------------------------------------------------------- reduction
constexpr int RB = 256;

// What bounds the sum is the rate of the reads: 16 bytes per thread and step,
// consecutive over the whole grid, so that the grid reads the array in order
// (2 loads in flight per thread, each over its own stretch: 30.8 us at 2^24
// words, 4: 31.7, 8: 34.3).  A first word off the 16-byte alignment and the
// last word are added apart.  The tiles are counted by the launch boundary:
// with a counter whose last arrival sums them, each of the 2048 workgroups'
// release and acquire flushed its L2, and 2^22 words took 61 us.  Both launches
// together, from HBM: 13.4 us at 2^22 words, 28.1 us at 2^24 (4.8 TB/s; 76.6 us
// with the counter and 8-byte loads), 87.7 us at 2^26 (6.1 TB/s; 142 us).
// Sum over the workgroup, valid in thread 0.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long s, unsigned long long* ws) {
    s = (unsigned long long)wave_sum64((long long)s);
    if (lane() == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    unsigned long long b = 0;
    if (threadIdx.x == 0)
        for (int k = 0; k < RB / LLP_WAVE; ++k) b += ws[k];
    return b;
}

__global__ void __launch_bounds__(RB) k_reduce_tiles(long long n, const unsigned long long* x,
                                                     unsigned long long* partial) {
    __shared__ unsigned long long ws[RB / LLP_WAVE];
    unsigned long long s = 0;
    const long long head = n > 0 && ((uintptr_t)x & 15) ? 1 : 0;
    const ulonglong2* v = (const ulonglong2*)(x + head);
    const long long pairs = (n - head) / 2;
    const long long tid = (long long)blockIdx.x * RB + threadIdx.x, nt = (long long)gridDim.x * RB;
#pragma unroll 1
    for (long long i = tid; i < pairs; i += nt) s += v[i].x + v[i].y;
    if (tid == 0) {
        if (head) s += x[0];
        if (head + 2 * pairs < n) s += x[n - 1];
    }
    s = block_sum(s, ws);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The root: one workgroup over the published tiles.
__global__ void __launch_bounds__(RB) k_reduce_root(int tiles, const unsigned long long* partial,
                                                    unsigned long long* result, int* status_dev) {
    __shared__ unsigned long long ws[RB / LLP_WAVE];
    unsigned long long s = 0;
    for (int k = threadIdx.x; k < tiles; k += RB) s += partial[k];
    s = block_sum(s, ws);
    if (threadIdx.x == 0) {
        *result = s;
        if (status_dev) *status_dev = 0;
    }
}

static int reduce_grid(int64_t n) {
    long long g = (n + RB * 8 - 1) / (RB * 8);
    long long cap = (long long)device_info().cus * 8;
    if (g > cap) g = cap;
    return (int)(g < 1 ? 1 : g);
}

size_t reduce_workspace_bytes(int64_t) { return 256 + (size_t)2048 * 8; }

int solve_reduce(int64_t n, const uint64_t* x, uint64_t* result, const llp_opts* opts) {
    if (n < 0) return fail(LLP_E_ARG, "n must be >= 0");
    if (!result || (n > 0 && !x)) return fail(LLP_E_ARG, "x and result are required");
    llp_opts o = opts_or_default(opts);
    hipStream_t st = (hipStream_t)o.stream;
    const int grid = reduce_grid(n);
    if (grid > 2048) return fail(LLP_E_ARG, "too many tiles");
    void* ws = nullptr;
    int s = get_workspace(o, reduce_workspace_bytes(n), &ws);
    if (s) return s;
    unsigned long long* partial = (unsigned long long*)((char*)ws + 256);
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool timing = (o.flags & LLP_TIMING) && o.stats;
    if (timing) {
        LLP_HIP(hipEventCreate(&ev0));
        LLP_HIP(hipEventCreate(&ev1));
        LLP_HIP(hipEventRecord(ev0, st));
    }
    hipLaunchKernelGGL(k_reduce_tiles, dim3(grid), dim3(RB), 0, st, (long long)n, (const unsigned long long*)x, partial);
    hipLaunchKernelGGL(k_reduce_root, dim3(1), dim3(RB), 0, st, grid, (const unsigned long long*)partial,
                       (unsigned long long*)result, (o.flags & LLP_ASYNC) ? o.status_dev : nullptr);
    LLP_HIP(hipGetLastError());
    if (timing) LLP_HIP(hipEventRecord(ev1, st));
    if (o.flags & LLP_ASYNC) return LLP_OK;
    LLP_HIP(hipStreamSynchronize(st));
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = 2;
        o.stats->advances = grid + 1;
        if (timing) {
            float ms = 0.f;
            LLP_HIP(hipEventElapsedTime(&ms, ev0, ev1));
            o.stats->device_ms = ms;
            o.stats->kernel_ms = ms;
        }
    }
    if (timing) {
        (void)hipEventDestroy(ev0);
        (void)hipEventDestroy(ev1);
    }
    return LLP_OK;
}

// ---------------------------------------------------------------- no-allocation reduction
// The same reduction with its scratch (one partial per tile) in a file-scope
// device array instead of a workspace: for callers that cannot allocate.
// Each GPU holds its own copy of the array; its device address is looked up once per device (host code never passes the
// array's name itself to a kernel).  Calls on one GPU share the array, so
// calls that overlap on one GPU race; every call writes the partials it reads.
constexpr int REDUCE_MAX_TILES = 2048;
constexpr size_t REDUCE_SCRATCH_BYTES = 256 + (size_t)REDUCE_MAX_TILES * 8;
static __device__ __align__(256) unsigned char scratch[REDUCE_SCRATCH_BYTES];

static std::mutex g_scratch_mu;
static std::map<int, void*> g_scratch;   // device -> device address of scratch

static int scratch_ptr(void** out) {
    int dev = 0;
    LLP_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch.find(dev);
    if (it == g_scratch.end()) {
        void* p = nullptr;
        LLP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(LLP_E_HIP, "no device address for the reduction scratch");
        it = g_scratch.emplace(dev, p).first;
    }
    *out = it->second;
    return LLP_OK;
}

int solve_reduce_noalloc(int64_t n, const uint64_t* x, uint64_t* result, const llp_opts* opts) {
    if (n < 0) return fail(LLP_E_ARG, "n must be >= 0");
    if (!result || (n > 0 && !x)) return fail(LLP_E_ARG, "x and result are required");
    llp_opts o = opts_or_default(opts);
    if (o.flags & LLP_TIMING) return fail(LLP_E_ARG, "LLP_TIMING is not available without allocation");
    hipStream_t st = (hipStream_t)o.stream;
    const int grid = reduce_grid(n);
    if (grid > REDUCE_MAX_TILES)
        return fail(LLP_E_ARG, "%d tiles exceed the %d partials of the static scratch", grid, REDUCE_MAX_TILES);
    void* sp = nullptr;
    int s = scratch_ptr(&sp);
    if (s) return s;
    unsigned long long* partial = (unsigned long long*)((char*)sp + 256);
    hipLaunchKernelGGL(k_reduce_tiles, dim3(grid), dim3(RB), 0, st, (long long)n, (const unsigned long long*)x, partial);
    hipLaunchKernelGGL(k_reduce_root, dim3(1), dim3(RB), 0, st, grid, (const unsigned long long*)partial,
                       (unsigned long long*)result, (o.flags & LLP_ASYNC) ? o.status_dev : nullptr);
    LLP_HIP(hipGetLastError());
    if (o.flags & LLP_ASYNC) return LLP_OK;
    LLP_HIP(hipStreamSynchronize(st));
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = 2;
        o.stats->advances = grid + 1;
    }
    return LLP_OK;
}

}  // namespace llp

extern "C" {

int llp_solve_reduce_noalloc(int64_t n, const uint64_t* x, uint64_t* result, const llp_opts* opts) {
    return llp::solve_reduce_noalloc(n, x, result, opts);
}

int llp_solve_tc(int32_t n, int64_t m, const int32_t* out_ptr, const int32_t* out_dst, uint32_t* bits,
                 const llp_opts* opts) {
    return llp::solve_tc(n, m, out_ptr, out_dst, bits, opts);
}

int llp_solve_reduce(int64_t n, const uint64_t* x, uint64_t* result, const llp_opts* opts) {
    return llp::solve_reduce(n, x, result, opts);
}

}  // extern "C"

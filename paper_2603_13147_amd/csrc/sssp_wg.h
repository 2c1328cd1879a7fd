// sssp_wg.h - single-source shortest paths of one small graph by one
// workgroup (paper Section 5.2), shared by the batch (batch.hip) and by small
// graphs solved alone (graph.hip).
//
// State G[v] = INF - d(v) in LDS (bottom 0, the source INF), the row offsets
// in LDS, and a bitmap of active vertices (their state rose since their arcs
// were last pushed).  Taking an active vertex u pushes single-arc partial
// advances G[x] <- max(G[x], G[u] - w) along its out-arcs with LDS atomicMax
// (Definition 3: a partial maximum is an alpha-forbidden advance) and makes x
// active where that raised it; no active vertex is the fixpoint.
//
// What bounds it is how the arcs are read: with a thread per vertex, each of
// its loads touched a line per lane and refetched it for every arc (5 clocks
// per arc and CU).  So a wave takes the active vertices of a block of 64
// together and walks their arcs edge by edge: positions 0 .. E-1 run over the
// block's arcs, lane l takes positions l + 64 j, and neighbouring lanes read
// neighbouring arcs.  A position's vertex comes from a table of 64 PER bytes per
// wave: every vertex writes its lane at its first position and a max-scan
// fills the rest.  A row of more than SW_LONG arcs needs no table.  4096
// graphs of 256 to 4096 vertices (80 M arcs): 681 us, against 1984 us with a
// thread per vertex.  There PER is 4, for four workgroups per CU (PER = 8
// needs more registers: 760 us), in workgroups of 512 threads (256: 934 us,
// 1024: 820).  Where no vertex of the step has more than one arc, the lanes of
// the batch read their own: chains are nothing but rounds, and 1001 vertices in
// one take 0.96 ms, 1.55 through the table (1.25 with a thread per vertex).
// A round is one scan of the bitmap; within a round waves see each other's
// advances, so a round is at least a synchronous one.
//
// SOLO: one graph alone on the chip, 16 waves, so a round lasts as long as its
// busiest wave, and three things spread the arcs:
//  - runs of four vertices are dealt to the blocks in turn, to at least one
//    block per wave (64 vertices of 97 arcs 42 us; 101 in one block), every
//    turn from another block on, as hubs often share their ids' low bits
//    (R-MAT scale 13, 8 arcs a vertex, ids not permuted: 234 us, 365 without).
//    Blocks of neighbouring vertices are up to 10% faster where they happen to
//    be even (R-MAT scale 11 with ids permuted 93 us, 102 dealt), and 355 there;
//  - a wave's blocks with few active vertices make one step together (R-MAT
//    scale 13, 8 arcs a vertex, BFS: 111 us, 147 without; 171 and 278 with ids
//    not permuted; uniform n = 4096, 8 arcs, SSSP: 118, 139 without);
//  - the long rows of a block that has more than SW_HUGE arcs in them are left
//    to all waves in the next round, in a list (one hub with half of 80000 arcs:
//    68 us, 212 without).  A list of every long row makes them wait too often
//    (R-MAT scale 10, 70 arcs a vertex: 111 us with a limit of 4096, 150 with 512).
// Going on with the blocks while few vertices are active, with or without a
// look at the other waves, saves rounds but pushes values too early: 5 to 40%
// longer throughout.  In the batch the other workgroups fill a wave's pauses.
#pragma once

#include "llp_dev.h"
#include "llp_host.h"

namespace llp {

constexpr int SW_LONG = 256;    // longest row taken through the table
// Flags: something was taken, and bad input was met, each by round modulo 3 (a
// wave past a round's only barrier may set the next round's before another has
// read this one's; the words it reads are cleared no sooner than two rounds
// on, so all waves leave by the same round); an arc overflowed; a distance did.
constexpr int SW_TAKEN = 0, SW_BAD = 3, SW_OVF_ARC = 6, SW_OVF = 7, SW_FLAGS = 8;
// SOLO: log2 of the waves; log2 of a run's vertices; arcs in a block's long rows
// above which all waves share them; rows listed for that, by round modulo 3, the
// length first.
constexpr int SW_SOLO_LG = 4, SW_SOLO_T = 64 << SW_SOLO_LG;
constexpr int SW_RUN = 2, SW_HUGE = 4096, SW_SHARED = 399, SW_SHARE_WORDS = 3 * (SW_SHARED + 1);

// LDS words needed for n vertices and T threads, n + 1 row offsets among them.
// per: arc positions per lane and step, a multiple of 4.
__host__ __device__ constexpr size_t sssp_wg_words(size_t n, size_t T, size_t per) {
    return 2 * ((n + 63) / 64) + T / 64 * (LLP_WAVE * per / 4) + n + n + 1;
}

struct SsspWg {
    int lg;                    // SOLO: log2 of the count of blocks, which is a multiple of the waves'
    unsigned long long* act;   // active vertices, a word per block of 64
    unsigned char* own;        // the wave's position table
    int* G;
    int* ptr;
};

// Blocks for n vertices.
template <bool SOLO>
__device__ __forceinline__ int sssp_wg_blocks(const SsspWg& s, int n) {
    return SOLO ? 1 << s.lg : (n + 63) >> 6;
}
// SOLO: where a turn of dealing runs to the blocks differs from the first.
__device__ __forceinline__ int sssp_wg_turn(const SsspWg& s, int turn) { return turn & ((1 << s.lg) - 1); }
// The vertex of a lane of a block.
template <bool SOLO>
__device__ __forceinline__ int sssp_wg_vertex(const SsspWg& s, int blk, int l) {
    if (!SOLO) return blk * 64 + l;
    const int turn = l >> SW_RUN;
    return (turn << s.lg | (blk ^ sssp_wg_turn(s, turn))) << SW_RUN | (l & ((1 << SW_RUN) - 1));
}
// The index of a vertex' bit in the bitmap.
template <bool SOLO>
__device__ __forceinline__ int sssp_wg_bit(const SsspWg& s, int v) {
    if (!SOLO) return v;
    const int run = v >> SW_RUN, turn = run >> s.lg, blk = (run & ((1 << s.lg) - 1)) ^ sssp_wg_turn(s, turn);
    return blk << 6 | turn << SW_RUN | (v & ((1 << SW_RUN) - 1));
}

// lds: 8-byte aligned, sssp_wg_words(n, blockDim.x, PER) words.
template <int PER, bool SOLO>
__device__ __forceinline__ SsspWg sssp_wg_carve(void* lds, int n) {
    SsspWg s;
    s.lg = SW_SOLO_LG;
    while (SOLO && 64 << s.lg < n) ++s.lg;
    s.act = (unsigned long long*)lds;
    unsigned char* own = (unsigned char*)(s.act + sssp_wg_blocks<SOLO>(s, n));
    s.own = own + (threadIdx.x >> 6) * LLP_WAVE * PER;
    s.G = (int*)(own + (blockDim.x >> 6) * LLP_WAVE * PER);
    s.ptr = s.G + n;
    return s;
}

// One arc's advance.
template <bool SOLO>
__device__ __forceinline__ void sssp_wg_push(const SsspWg& s, int x, int cand) {
    if (cand > s.G[x] && atomicMax(&s.G[x], cand) < cand) {
        const int b = sssp_wg_bit<SOLO>(s, x);
        atomicOr(&((unsigned*)s.act)[b >> 5], 1u << (b & 31));
    }
}

// Arcs ks[j] of tails with state gs[j] (j < PER, those with on[j]).  UNIT: every
// weight is 1.  NEG: negative weights are malformed input, else they are
// taken as they are.
template <int PER, bool UNIT, bool NEG, bool SOLO>
__device__ __forceinline__ void sssp_wg_arcs(const SsspWg& s, const int* dst, const int* wgt, int n, const int* ks,
                                             const int* gs, const bool* on, bool& bad, bool& ovf) {
    int x[PER], w[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        x[j] = on[j] ? dst[ks[j]] : 0;
        w[j] = UNIT ? 1 : (on[j] ? wgt[ks[j]] : 0);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (!on[j]) continue;
        if ((unsigned)x[j] >= (unsigned)n || (NEG && w[j] < 0)) {
            bad = true;
            continue;
        }
        const int cand = (int)((unsigned)gs[j] - (unsigned)w[j]);
        if (cand <= 0) ovf = true;
        else sssp_wg_push<SOLO>(s, x[j], cand);
    }
}

// Arcs of one row [zb, zb + zd) of a tail with state zg: positions k0, k0 +
// step, ... on, CHUNK at a time (uniform in the wave).
template <int PER, bool UNIT, bool NEG, bool SOLO>
__device__ __forceinline__ void sssp_wg_row(const SsspWg& s, const int* dst, const int* wgt, int n, int l, int zb, int zd, int zg,
                                            unsigned k0, unsigned step, bool& bad, bool& ovf) {
    for (; k0 < (unsigned)zd; k0 += step) {
        int ks[PER], gs[PER];
        bool on[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const unsigned k = k0 + 64 * j + l;
            on[j] = k < (unsigned)zd;
            ks[j] = zb + (int)k;
            gs[j] = zg;
        }
        sssp_wg_arcs<PER, UNIT, NEG, SOLO>(s, dst, wgt, n, ks, gs, on, bad, ovf);
    }
}

// Solves with the calling workgroup.  gptr[n + 1], dst[m],
// wgt[m]: out-CSR; dist[n]: the output (INF = unreached).  fl: LDS int[SW_FLAGS].
// share: LDS int[SW_SHARE_WORDS] (SOLO).  Returns the status, uniform in the
// workgroup.
template <int PER, bool UNIT, bool NEG, bool SOLO>
__device__ __forceinline__ int sssp_wg(const int* gptr, const int* dst, const int* wgt, int n, int m, int src,
                                       const SsspWg& s, int* fl, int* share, int* dist, long long max_rounds) {
    const int T = SOLO ? SW_SOLO_T : blockDim.x, t = threadIdx.x, l = lane(), wave = t >> 6, nw = T >> 6;
    constexpr int CHUNK = LLP_WAVE * PER;
    const int nb = sssp_wg_blocks<SOLO>(s, n), sb = sssp_wg_bit<SOLO>(s, src);
    for (int v = t; v < n; v += T) s.G[v] = v == src ? LLP_INF : 0;
    for (int v = t; v <= n; v += T) s.ptr[v] = gptr[v];
    for (int i = t; i < nb; i += T) s.act[i] = i == (sb >> 6) ? 1ull << (sb & 63) : 0ull;
    if (t < SW_FLAGS) fl[t] = 0;
    if (SOLO && t < 3) share[t * (SW_SHARED + 1)] = 0;
    __syncthreads();
    long long r = 0;
    int now = 0;   // r modulo 3
    bool more = true;
    int st = LLP_OK;
    for (; more && r < max_rounds; ++r) {
        const int next = now == 2 ? 0 : now + 1, last = now == 0 ? 2 : now - 1;
        bool bad = false, ovf = false, did = false;
        if (t == 0) fl[SW_TAKEN + next] = fl[SW_BAD + next] = 0;   // last read in round r - 2
        if constexpr (SOLO) {
            // the last round's long rows, with what their vertices have risen to
            // meanwhile; this round fills its own list, the next one's is free
            const int* list = share + last * (SW_SHARED + 1);
            const int rows = min(list[0], SW_SHARED);
            if (t == 0) share[next * (SW_SHARED + 1)] = 0;
            did = rows > 0;
            for (int i = 0; i < rows; ++i) {
                const int v = list[1 + i], zb = s.ptr[v], zd = s.ptr[v + 1] - zb, zg = s.G[v];
                sssp_wg_row<PER, UNIT, NEG, SOLO>(s, dst, wgt, n, l, zb, zd, zg, wave * CHUNK, nw * CHUNK, bad, ovf);
            }
        }
        for (int c = wave; c < nb; c += nw * LLP_WAVE) {   // lane l looks at block c + nw l
            // read once: what the step takes is what was counted
            const unsigned long long seen = c + nw * l < nb ? s.act[min(c + nw * l, nb - 1)] : 0ull;
            uint64_t todo = ballot(seen != 0ull), few = 0ull;
            if constexpr (SOLO) {
                // all blocks with few active vertices make one step: 1 << lp
                // blocks to a wave, lane l with vertex l >> lp of block l & (1 << lp) - 1
                const int lp = s.lg - SW_SOLO_LG;
                if (lp > 0) few = ballot(__popcll(seen) << lp <= LLP_WAVE) & todo;
                if ((few & (few - 1)) == 0ull) few = 0ull;
                todo &= ~few;
            }
            while (todo || few) {
                did = true;
                int b = 0, deg = 0, g = 0, v = 0;
                bool has;
                // take the bits, then read the states: what rises later sets its bit again
                if (SOLO && few) {
                    const int lp = s.lg - SW_SOLO_LG, i = l & ((1 << lp) - 1);
                    const bool in = (few >> l) & 1ull;
                    const unsigned long long mine = in ? seen : 0ull;
                    if (in) atomicAnd(&s.act[c + nw * l], ~mine);
                    unsigned long long f = (unsigned long long)__shfl((long long)mine, i, LLP_WAVE);
                    for (int k = l >> lp; k > 0; --k) f &= f - 1;
                    has = f != 0ull;
                    v = sssp_wg_vertex<SOLO>(s, c + nw * i, __ffsll((long long)f) - 1);
                    few = 0ull;
                } else {
                    const int blk = c + nw * (__ffsll((long long)todo) - 1);
                    const unsigned long long f = s.act[blk];
                    __builtin_amdgcn_wave_barrier();
                    if (l == 0) atomicAnd(&s.act[blk], ~f);
                    has = (f >> l) & 1ull;
                    v = sssp_wg_vertex<SOLO>(s, blk, l);
                    todo &= todo - 1;
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
                if (has) {
                    b = s.ptr[v];
                    const int e = s.ptr[v + 1];
                    if (b < 0 || e > m || e < b) bad = true;
                    else deg = e - b;
                    g = s.G[v];
                }
                if (!SOLO && !__any(deg > 1)) {   // (a graph alone has three arcs a vertex or more)
                    int ks[1] = {b}, gs[1] = {g};
                    bool on[1] = {deg > 0};
                    sssp_wg_arcs<1, UNIT, NEG, SOLO>(s, dst, wgt, n, ks, gs, on, bad, ovf);
                    continue;
                }
                const int len = deg <= SW_LONG ? deg : 0;
                const int incl = wave_incl_sum(len), E = shfl(incl, 63);
                const int start = incl - len, off = b - start;
                for (int base = 0; base < E; base += CHUNK) {
                    unsigned* cell = (unsigned*)(s.own + PER * l);   // the lane's own PER positions
#pragma unroll
                    for (int q = 0; q < PER / 4; ++q) cell[q] = 0u;
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
                    if (len > 0 && start < base + CHUNK && incl > base)
                        s.own[start > base ? start - base : 0] = (unsigned char)(l + 1);
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
                    int run = 0, o[PER];
#pragma unroll
                    for (int j = 0; j < PER; ++j) {
                        run = max(run, (int)((cell[j / 4] >> (8 * (j & 3))) & 255u));
                        o[j] = run;
                    }
                    int before = __shfl_up(wave_incl_max(run), 1, LLP_WAVE);
                    if (l == 0) before = 0;
#pragma unroll
                    for (int q = 0; q < PER / 4; ++q) {
                        unsigned z = 0u;
#pragma unroll
                        for (int j = 0; j < 4; ++j) z |= (unsigned)max(before, o[4 * q + j]) << (8 * j);
                        cell[q] = z;
                    }
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_wave_barrier();
                    int ks[PER], gs[PER];
                    bool on[PER];
#pragma unroll
                    for (int j = 0; j < PER; ++j) {
                        const int p = base + 64 * j + l;
                        on[j] = p < E;
                        const int w = on[j] ? s.own[64 * j + l] - 1 : 0;
                        ks[j] = p + shfl(off, w);
                        gs[j] = shfl(g, w);
                    }
                    sssp_wg_arcs<PER, UNIT, NEG, SOLO>(s, dst, wgt, n, ks, gs, on, bad, ovf);
                    __builtin_amdgcn_wave_barrier();
                }
                uint64_t big = ballot(deg > SW_LONG);
                if constexpr (SOLO) {
                    if (big && wave_sum64(deg > SW_LONG ? deg : 0) > SW_HUGE) {
                        if (deg > SW_LONG) {
                            int* list = share + now * (SW_SHARED + 1);
                            const int i = atomicAdd(&list[0], 1);
                            if (i < SW_SHARED) {
                                list[1 + i] = v;
                                deg = 0;
                            }
                        }
                        big = ballot(deg > SW_LONG);
                    }
                }
                // (not sssp_wg_row: k_batch then has 7 more scalar registers to
                // spill and its knapsacks take 5% longer)
                for (; big; big &= big - 1) {
                    const int z = __ffsll((long long)big) - 1;
                    const int zb = shfl(b, z), zd = shfl(deg, z), zg = shfl(g, z);
                    for (unsigned k0 = 0; k0 < (unsigned)zd; k0 += CHUNK) {
                        int ks[PER], gs[PER];
                        bool on[PER];
#pragma unroll
                        for (int j = 0; j < PER; ++j) {
                            const unsigned k = k0 + 64 * j + l;
                            on[j] = k < (unsigned)zd;
                            ks[j] = zb + (int)k;
                            gs[j] = zg;
                        }
                        sssp_wg_arcs<PER, UNIT, NEG, SOLO>(s, dst, wgt, n, ks, gs, on, bad, ovf);
                    }
                }
            }
        }
        if (did && l == 0) fl[SW_TAKEN + now] = 1;
        if (bad) fl[SW_BAD + now] = 1;
        if (ovf) fl[SW_OVF_ARC] = 1;
        __syncthreads();
        if (fl[SW_BAD + now]) st = LLP_E_INPUT;
        more = fl[SW_TAKEN + now] != 0 && st == LLP_OK;
        now = next;
    }
    if (more) st = LLP_E_NOT_CONVERGED;
    // overflow: an unreached vertex with a reached in-neighbour (every wave has
    // left the rounds: none sets the flag any more)
    if (st == LLP_OK && fl[SW_OVF_ARC]) {
        for (int u = t; u < n; u += T) {
            if (s.G[u] <= 0) continue;
            for (int k = max(s.ptr[u], 0); k < min(s.ptr[u + 1], m); ++k) {
                const int x = dst[k];
                if ((unsigned)x < (unsigned)n && s.G[x] == 0) fl[SW_OVF] = 1;
            }
        }
        __syncthreads();
        if (fl[SW_OVF]) st = LLP_E_OVERFLOW;
    }
    for (int v = t; v < n; v += T) {
        const int g = s.G[v];
        dist[v] = g > 0 ? LLP_INF - g : LLP_INF;
    }
    return st;
}

}  // namespace llp

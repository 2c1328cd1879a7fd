// sm.hip - the LLP sweep for the man-optimal stable matching (paper Section
// 5.4) on gfx950.
//
// State.  G[m] is the index of the woman man m currently targets in his list
// (bottom 0, bound n - 1).  m is forbidden when his target is also targeted
// by a man she ranks better; alpha(G, m) = G[m] + 1.
//
// The forbidden test is answered by best[w], the smallest key that has ever
// targeted woman w, key = rank << 32 | man << 16 | index (64-bit atomicMin).
// The man holding best[w] targets w at every moment (he can only be moved on
// by a better key, which then holds w), so a man whose key loses the minimum
// at w is forbidden in the current state and may advance; a man whose key
// wins displaces the previous holder, who becomes forbidden.  (The predicate
// counts every man who has reached w in his list; from the bottom only the
// current holder matters, and a warm start registers the proposals its
// indices imply before the sweep.)  Because the
// displaced key carries its index, the displacing thread knows where the
// displaced man resumes without reading his G.
//
// Schedules (all reach the same least fixpoint):
//  - chains (default): one thread per man; a thread whose man is rejected
//    advances him and proposes again, a thread whose man displaces another
//    carries on with the displaced man, and a thread ends when its man lands
//    on a woman nobody held.  opts->chunk > 0 bounds the proposals a thread
//    makes per launch; a man still forbidden at the bound is parked and the
//    next launch (round) resumes him.
//  - dense rounds (LLP_SCHED_FIXED + LLP_DENSE): every round evaluates every
//    man once at his current target and advances the forbidden ones by one.
//  - random rounds (LLP_SCHED_RANDOM): dense rounds in which each forbidden
//    man advances only on a seeded coin flip.
#include <string.h>

#include "llp_dev.h"
#include "llp_host.h"

namespace llp {

constexpr unsigned long long SM_EMPTY = ~0ull;
constexpr int SM_NFLAG = 64;
constexpr int SM_LOOKAHEAD = 4;   // women examined per round trip of a chain

struct SCtrl {
    int done;
    int status;
    int last_round;
    int pad;
    int diag[8];
    long long proposals;
    int flag[SM_NFLAG];   // flag[r & 63]: round r left work for round r + 1
};

struct SArgs {
    int n;
    const short* mpref;   // [n * n] woman ids
    const short* wrank;   // [n * n] rank of man m for woman w
    int* G;               // proposal index per man
    unsigned long long* best;
    int* pend;            // round in which a parked man resumes (chunked chains)
    SCtrl* ctrl;
    const int* warm;      // warm start (nullable): man m has proposed to his first warm[m] women
    int chunk;            // proposals per thread per launch, 0 = unbounded
    int random;           // random rounds
    unsigned long long seed;
    int* combo;           // n <= SM_LDS_MAX: [n * SM_COMBO] w | rank of m for w << 16, by man and list position
};

__device__ __forceinline__ unsigned long long sm_key(int rank, int man, int idx) {
    return ((unsigned long long)(unsigned)rank << 32) | ((unsigned long long)(unsigned)man << 16) |
           (unsigned long long)(unsigned)idx;
}

__device__ __forceinline__ unsigned long long amin64(unsigned long long* p, unsigned long long v) {
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_sm_init(SArgs a, const int* warm) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    for (long long i = tid; i < a.n; i += nt) {
        int g = 0;
        if (warm) {
            g = warm[i];
            if (g < 0 || g >= a.n) g = 0;
        }
        a.G[i] = g;
        a.best[i] = SM_EMPTY;
        a.pend[i] = 1;
    }
    if (tid == 0) memset(a.ctrl, 0, sizeof(SCtrl));
}

__device__ __forceinline__ int sm_warm(const SArgs& a, int m) {
    int g = a.warm[m];
    return (g < 0 || g >= a.n) ? 0 : g;
}

// Warm start: index G0[m] means man m has already proposed to the women
// before it (the predicate counts every man who has reached w in his list),
// so those proposals are registered before the sweep starts.
__global__ void k_sm_warm_register(SArgs a) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    for (long long m = tid; m < a.n; m += nt) {
        const int g0 = sm_warm(a, (int)m);
        for (int i = 0; i < g0; ++i) {
            int w = guard(a.mpref[m * a.n + i], a.n, a.ctrl->diag, 9, (int)m, i);
            int rk = guard(a.wrank[(long long)w * a.n + m], a.n, a.ctrl->diag, 10, w, (int)m);
            amin64(&a.best[w], sm_key(rk, (int)m, i));
        }
    }
}

// One workgroup per list (men's lists first, then women's rank rows): every
// row must be a permutation of 0..n-1.  n <= 32767, so a row's bitmap fits
// in 4 KB of LDS.
__global__ void k_sm_validate(SArgs a) {
    __shared__ unsigned bits[1024];
    const int row = blockIdx.x;
    const short* p = row < a.n ? a.mpref + (long long)row * a.n : a.wrank + (long long)(row - a.n) * a.n;
    const int words = (a.n + 31) >> 5;
    for (int i = threadIdx.x; i < words; i += blockDim.x) bits[i] = 0u;
    __syncthreads();
    bool bad = false;
    for (int i = threadIdx.x; i < a.n; i += blockDim.x) {
        int x = p[i];
        if (x < 0 || x >= a.n) {
            bad = true;
            continue;
        }
        unsigned old = atomicOr(&bits[x >> 5], 1u << (x & 31));
        if (old & (1u << (x & 31))) bad = true;
    }
    if (bad) set_status(&a.ctrl->status, LLP_E_INPUT);
}

// Chains.  Launch r resumes the men whose pend stamp is r (round 1: all).
__global__ void k_sm_chain(SArgs a, int r) {
    SCtrl* c = a.ctrl;
    if (ld_relaxed(&c->done) || ld_relaxed(&c->status)) return;
    if (r > 1 && ld_relaxed(&c->flag[(r - 1) & (SM_NFLAG - 1)]) == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c->done = 1;
            c->last_round = r - 1;
        }
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) c->flag[(r + 1) & (SM_NFLAG - 1)] = 0;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    long long made = 0;
    if (t < a.n && a.pend[t] == r) {
        const int n = a.n;
        int m = t;
        int g = guard(a.G[m], n, c->diag, 8, m);
        const long long cap = a.chunk > 0 ? a.chunk : (long long)n * n + n;
        for (;;) {
            if (g >= n) {
                set_status(&c->status, LLP_E_INFEASIBLE);
                break;
            }
            if (made >= cap) {
                // park m, still to propose at index g, for the next launch
                amax(&a.G[m], g);
                a.pend[m] = r + 1;
                st_relaxed(&c->flag[r & (SM_NFLAG - 1)], 1);
                break;
            }
            // look ahead: the next women on m's list, their ranks of m and their
            // current best keys are independent loads; a woman whose best key
            // already beats m's rejects him without an atomic (best only
            // decreases), so a run of rejections costs one round trip
            const int la = (int)min((long long)SM_LOOKAHEAD, min((long long)(n - g), cap - made));
            int wv[SM_LOOKAHEAD];
            unsigned long long kv[SM_LOOKAHEAD], bv[SM_LOOKAHEAD];
#pragma unroll
            for (int i = 0; i < SM_LOOKAHEAD; ++i) {
                if (i < la) {
                    wv[i] = guard(a.mpref[(long long)m * n + g + i], n, c->diag, 1, m, g + i);
                } else {
                    wv[i] = 0;
                }
            }
#pragma unroll
            for (int i = 0; i < SM_LOOKAHEAD; ++i) {
                kv[i] = ~0ull;
                bv[i] = 0ull;
                if (i < la) {
                    int rk = guard(a.wrank[(long long)wv[i] * n + m], n, c->diag, 2, wv[i], m);
                    kv[i] = sm_key(rk, m, g + i);
                    bv[i] = a.best[wv[i]];
                }
            }
            int skip = 0;
#pragma unroll
            for (int i = 0; i < SM_LOOKAHEAD; ++i)
                if (skip == i && i < la && bv[i] < kv[i]) skip = i + 1;
            if (skip == la) {   // every looked-at woman holds a better man
                g += la;
                made += la;
                continue;
            }
            g += skip;
            made += skip + 1;
            int w = 0;
            unsigned long long key = 0;
#pragma unroll
            for (int i = 0; i < SM_LOOKAHEAD; ++i)
                if (i == skip) {
                    w = wv[i];
                    key = kv[i];
                }
            unsigned long long old = amin64(&a.best[w], key);
            if (old < key) {        // w holds a better man: m is forbidden
                ++g;
                continue;
            }
            amax(&a.G[m], g);       // m targets w and is not forbidden
            if (old == SM_EMPTY || old == key) break;
            // the previous holder is now forbidden at w: carry him on, unless
            // the key was registered for a warm start (he is already past w)
            m = guard((int)((old >> 16) & 0xffffull), n, c->diag, 3, w, (int)(old & 0xffff));
            g = (int)(old & 0xffffull) + 1;
            if (a.warm && g - 1 < sm_warm(a, m)) break;
        }
    }
    long long tot = wave_sum64(made);
    if (lane() == 0 && tot) atomicAdd((unsigned long long*)&c->proposals, (unsigned long long)tot);
}

// One workgroup runs every chain of a cold start with n <= SM_LDS_MAX: the
// women's best keys and the men's positions live in LDS, so the displacement
// atomic and the reads of the keys stay on the CU (across XCDs an atomic must
// reach the memory side).  See k_sm_lds.
constexpr int SM_LDS_MAX = 12288;   // 10 B of LDS per man: 120 KB
constexpr int SM_COMBO = 64;        // list positions per man held as (woman, rank) pairs
constexpr int SM_LDS_LOOKAHEAD = 6;   // women examined per round trip of a thread's chain in k_sm_lds
constexpr unsigned SM_FREE = ~0u;   // key of a woman nobody holds
constexpr int SM_MAN_BITS = 14;     // a key is rank << 14 | man (n <= SM_LDS_MAX < 2^14)
constexpr int SM_MAN = (1 << SM_MAN_BITS) - 1;
constexpr int SM_HOPS = 16;         // steps of a thread's chain in the first pass
// The passes after it (see k_sm_lds):
constexpr int SM_MANY = 128;        // chains from which a pass may go by threads
constexpr int SM_TRIES = 128;       // positions tried per man displaced below which it does
constexpr int SM_PASS_HOPS = 64;    // and its steps per chain
constexpr int SM_FEW = 64;          // chains up to which a wave runs each to its end
constexpr int SM_WAVE_HOPS = 16;    // men a wave's chain displaces per pass while there are more
constexpr int SM_LDS_THREADS = 1024;

// The i-th woman w on m's list and her rank of m, as w | rank << 16.
__device__ __forceinline__ int sm_pair(const SArgs& a, int m, int i) {
    const int n = a.n;
    const int w = guard(a.mpref[(long long)m * n + i], n, a.ctrl->diag, 4, m, i);
    const int rk = guard(a.wrank[(long long)w * n + m], n, a.ctrl->diag, 5, w, m);
    return w | (rk << 16);
}

// combo[m * SM_COMBO + i] = sm_pair(m, i) for the first SM_COMBO positions of
// every list (men make about log n proposals on average): a chain step there
// reads one entry (woman and her rank of m together) instead of a list entry
// and then a rank; later positions read both.  One thread per entry.
__global__ void k_sm_combo(SArgs a) {
    const int n = a.n;
    const int k = min(n, SM_COMBO);
    const long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= (long long)n * k) return;
    const int m = (int)(x / k), i = (int)(x % k);
    a.combo[(long long)m * SM_COMBO + i] = sm_pair(a, m, i);
}

// Adds the wave's x and y to words in LDS.
__device__ __forceinline__ void sm_add(int* px, int x, int* py, int y) {
    const int sx = (int)wave_sum64(x), sy = (int)wave_sum64(y);
    if (lane() == 0) {
        atomicAdd(px, sx);
        atomicAdd(py, sy);
    }
}

// Up to `hops` steps of a thread's chain from man m at position g on, while g
// is below the table's end (PAST: the list's).  Returns whether the chain is
// unfinished: m then stands at g.  tries, moves: positions tried, men displaced.
template <bool PAST>
__device__ __forceinline__ bool sm_thread_chain(const SArgs& a, unsigned* best, unsigned short* nx, int hops, int& m, int& g,
                                                int& tries, int& moves) {
    const int k = min(a.n, SM_COMBO), end = PAST ? a.n : k;
    for (int hop = 0; hop < hops && g < end; ++hop) {
        // positions past the end read the last entry, whose woman is then
        // taken only at her own position
        int cw[SM_LDS_LOOKAHEAD];
        unsigned bv[SM_LDS_LOOKAHEAD];
        if (!PAST || g + SM_LDS_LOOKAHEAD <= k) {
#pragma unroll
            for (int i = 0; i < SM_LDS_LOOKAHEAD; ++i) cw[i] = a.combo[m * SM_COMBO + min(g + i, k - 1)];
        } else {
#pragma unroll
            for (int i = 0; i < SM_LDS_LOOKAHEAD; ++i) cw[i] = sm_pair(a, m, min(g + i, end - 1));
        }
#pragma unroll
        for (int i = 0; i < SM_LDS_LOOKAHEAD; ++i) bv[i] = best[cw[i] & 0xffff];
        int at = -1, w = 0;
        unsigned key = 0;
#pragma unroll
        for (int i = SM_LDS_LOOKAHEAD - 1; i >= 0; --i) {
            const unsigned ki = ((unsigned)cw[i] >> 16 << SM_MAN_BITS) | (unsigned)m;
            if (g + i < end && ki < bv[i]) {
                at = g + i;
                w = cw[i] & 0xffff;
                key = ki;
            }
        }
        if (at < 0) {
            tries += min(SM_LDS_LOOKAHEAD, end - g);
            g = min(g + SM_LDS_LOOKAHEAD, end);
            continue;
        }
        tries += at + 1 - g;
        nx[m] = (unsigned short)(at + 1);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        const unsigned old = atomicMin(&best[w], key);
        if (old == SM_FREE) return false;
        if (old > key) {
            ++moves;
            m = (int)(old & SM_MAN);
            g = nx[m];
        } else {
            g = at + 1;
        }
    }
    return true;
}

// Up to `hops` displacements of a wave's chain (m and g uniform in the wave).
// Returns whether the chain is unfinished: m then stands at g.  bad is set
// where a man exhausts his list.
template <bool LIMIT>
__device__ __forceinline__ bool sm_wave_chain(const SArgs& a, unsigned* best, unsigned short* nx, int* bad, int hops, int& m,
                                              int& g, int& tries, int& moves) {
    const int n = a.n, k = min(n, SM_COMBO), l = lane();
    int row = l < k ? a.combo[m * SM_COMBO + l] : 0;
    for (int hop = 0; !LIMIT || hop < hops;) {
        // the first of m's women from position g on who prefers him
        int at = -1, w = row & 0xffff;
        unsigned key = ((unsigned)row >> 16 << SM_MAN_BITS) | (unsigned)m;
        unsigned bv = l >= g && l < k ? best[w] : 0u;
        uint64_t ok = ballot(key < bv);
        for (int b = max(g, k); !ok && b < n; b += LLP_WAVE) {   // past the table: the list and the rank
            const int p = b + l < n ? sm_pair(a, m, b + l) : 0;
            w = p & 0xffff;
            key = ((unsigned)p >> 16 << SM_MAN_BITS) | (unsigned)m;
            bv = b + l < n ? best[w] : 0u;
            ok = ballot(key < bv);
            at = b;
        }
        if (!ok) {
            if (l == 0) *bad = 1;   // he exhausted his list
            return false;
        }
        const int i = __ffsll((long long)ok) - 1;
        at = max(at, 0) + i;
        if constexpr (LIMIT) tries += at + 1 - g;
        const int wi = __builtin_amdgcn_readlane(w, i);
        const unsigned ki = (unsigned)__builtin_amdgcn_readlane((int)key, i);
        const unsigned seen = (unsigned)__builtin_amdgcn_readlane((int)bv, i);
        // her holder's row and position, on the way while he is displaced
        const int m2 = seen == SM_FREE ? m : (int)(seen & SM_MAN);
        const int row2 = l < k ? a.combo[m2 * SM_COMBO + l] : 0;
        const int g2 = nx[m2];
        unsigned old = 0;
        if (l == 0) {
            nx[m] = (unsigned short)(at + 1);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            old = atomicMin(&best[wi], ki);
        }
        old = (unsigned)__builtin_amdgcn_readfirstlane((int)old);
        if (old == SM_FREE) return false;
        if (old == seen) {
            m = m2;
            row = row2;
            g = __builtin_amdgcn_readfirstlane(g2);
            if constexpr (LIMIT) ++hop, ++moves;
        } else if (old < ki) {   // another chain was first: m tries on
            g = at + 1;
        } else {                 // another chain's man is displaced instead
            m = (int)(old & SM_MAN);
            row = l < k ? a.combo[m * SM_COMBO + l] : 0;
            g = __builtin_amdgcn_readfirstlane((int)nx[m]);
            if constexpr (LIMIT) ++hop, ++moves;
        }
    }
    return true;
}

// A chain step takes the man displaced last, finds the first woman on the
// rest of his list whose key his own beats, and displaces her holder.  It is
// bound by latency: a row of the table from the L2, the women's keys from
// LDS, and the next man is known.  Two forms:
//  - a thread per chain, 6 women per step;
//  - a wave per chain: a lane per list position, so a man's whole row of 64 is
//    one load and a ballot finds his woman, however many reject him.  Her
//    holder is in the key read, so his row is loaded before the atomicMin that
//    displaces him returns; if another chain came between, the row is dropped.
// The first pass starts every man by a thread, SM_HOPS steps inside the table,
// and a pass leaves its unfinished chains to the next.  In a random market few
// are left, and waves end them.  Where many are, waves displace at most
// SM_WAVE_HOPS men per chain and pass, so that good ranks settle before the
// rest try on, and while a displaced man tries few positions (SM_TRIES), many
// chains at once by threads are the faster.  That is what lists and ranks much
// alike need: all lists and ranks the same, n = 3000 18.7 ms (ranks reversed
// 18.3, shuffled 23.0), n = 8192 117 (119, 184), against 47.6 (182, 194) and 444
// (1590, 1630) with every chain run to its end by a wave, and 15.8 (21.9, 29.6)
// and 91 (151, 243) with a thread per chain throughout.  Lists alike with random
// ranks want waves: n = 8192 39.8 ms against 53.4 by threads.  Limits of 24 to
// 200 positions and 64 to 256 chains measure within 10% of each other but for
// lists and ranks strongly alike at n = 1000 (0.56 ms; 1.10 with 24) and lists
// alike at n = 300 (0.09; 0.18 with 64 chains).
// A man's position nx (the next one to try) is written before the atomicMin
// that places him (LDS operations of a wave stay in order), so whoever reads
// his key reads his position too.
// Random markets, three each: n = 8192 330-521 us (0.73-1.62 ms with a thread per
// chain throughout), n = 3000 143-239 (335-663), n = 1000 91-109 (192-270).  With 4
// or 64 steps in the first pass 10% more or the same at n = 8192; without
// touching the table first 10% more.
__global__ void __launch_bounds__(SM_LDS_THREADS) k_sm_lds(SArgs a) {
    __shared__ unsigned best[SM_LDS_MAX];
    __shared__ unsigned short nx[SM_LDS_MAX];
    __shared__ unsigned short pend[2][SM_LDS_MAX];
    // by pass modulo 3: unfinished chains, positions tried and men displaced in
    // the pass before, chains taken by the waves
    __shared__ int npend[3], ntry[3], nmove[3], head[3], bad;
    SCtrl* c = a.ctrl;
    const int n = a.n, k = min(n, SM_COMBO), l = lane();
    for (int i = threadIdx.x; i < n; i += SM_LDS_THREADS) {
        best[i] = SM_FREE;
        nx[i] = 0;
    }
    if (threadIdx.x < 3) npend[threadIdx.x] = ntry[threadIdx.x] = nmove[threadIdx.x] = head[threadIdx.x] = 0;
    if (threadIdx.x == 0) bad = 0;
    // one word of every line of the table, so that a chain's first visit to a
    // row finds it in this XCD's L2 (the table was written from all of them)
    int x = 0;
    for (int i = threadIdx.x * 32; i < n * SM_COMBO; i += SM_LDS_THREADS * 32) x |= a.combo[i];
    asm volatile("" ::"v"(x));
    __syncthreads();
    {
        int tries = 0, moves = 0;
        for (int t = threadIdx.x; t < n; t += SM_LDS_THREADS) {
            int m = t, g = 0;
            if (sm_thread_chain<false>(a, best, nx, SM_HOPS, m, g, tries, moves)) {
                nx[m] = (unsigned short)g;
                pend[0][atomicAdd(&npend[0], 1)] = (unsigned short)m;
            }
        }
        sm_add(&ntry[0], tries, &nmove[0], moves);
    }
    __syncthreads();
    for (int pass = 0;; ++pass) {
        const int i = pass % 3, nxt = (pass + 1) % 3, clr = (pass + 2) % 3;
        const int np = npend[i];
        if (np == 0) break;
        const bool by_thread = np >= SM_MANY && (long long)SM_TRIES * nmove[i] > ntry[i];
        const unsigned short* from = pend[pass & 1];
        unsigned short* to = pend[(pass + 1) & 1];
        if (threadIdx.x == 0) npend[clr] = ntry[clr] = nmove[clr] = head[clr] = 0;   // last read in the pass before
        int tries = 0, moves = 0;
        if (by_thread) {
            for (int t = threadIdx.x; t < np; t += SM_LDS_THREADS) {
                int m = from[t], g = nx[m];
                if (!sm_thread_chain<true>(a, best, nx, SM_PASS_HOPS, m, g, tries, moves)) continue;
                if (g >= n) {
                    bad = 1;   // he exhausted his list
                    continue;
                }
                nx[m] = (unsigned short)g;
                to[atomicAdd(&npend[nxt], 1)] = (unsigned short)m;
            }
        } else {
            for (;;) {
                int q = 0;
                if (l == 0) q = atomicAdd(&head[i], 1);
                q = __builtin_amdgcn_readfirstlane(q);
                if (q >= np) break;
                int m = __builtin_amdgcn_readfirstlane((int)from[q]);
                int g = __builtin_amdgcn_readfirstlane((int)nx[m]);
                if (np <= SM_FEW) {
                    sm_wave_chain<false>(a, best, nx, &bad, 0, m, g, tries, moves);
                } else if (sm_wave_chain<true>(a, best, nx, &bad, SM_WAVE_HOPS, m, g, tries, moves) && l == 0) {
                    nx[m] = (unsigned short)g;
                    to[atomicAdd(&npend[nxt], 1)] = (unsigned short)m;
                }
            }
            if (l) tries = moves = 0;   // counted once for the wave
        }
        sm_add(&ntry[nxt], tries, &nmove[nxt], moves);
        __syncthreads();
    }
    if (bad && threadIdx.x == 0) set_status(&c->status, LLP_E_INFEASIBLE);
    // a man's proposals are the positions he tried
    long long made = 0;
    for (int i = threadIdx.x; i < n; i += SM_LDS_THREADS) {
        a.G[i] = max((int)nx[i] - 1, 0);
        made += nx[i];
    }
    const long long tot = wave_sum64(made);
    if (l == 0 && tot) atomicAdd((unsigned long long*)&c->proposals, (unsigned long long)tot);
    if (threadIdx.x == 0) {
        c->done = 1;
        c->last_round = 1;
    }
}

__device__ __forceinline__ unsigned long long sm_mix(unsigned long long x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// Dense round r: every man registers his current proposal and advances by one
// if it loses (on a coin flip for random rounds).
__global__ void k_sm_round(SArgs a, int r) {
    SCtrl* c = a.ctrl;
    if (ld_relaxed(&c->done) || ld_relaxed(&c->status)) return;
    if (r > 1 && ld_relaxed(&c->flag[(r - 1) & (SM_NFLAG - 1)]) == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c->done = 1;
            c->last_round = r - 1;
        }
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) c->flag[(r + 1) & (SM_NFLAG - 1)] = 0;
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    const int n = a.n;
    long long tot = wave_sum64(m < n ? 1 : 0);
    if (lane() == 0 && tot) atomicAdd((unsigned long long*)&c->proposals, (unsigned long long)tot);
    if (m >= n) return;
    int g = guard(a.G[m], n, c->diag, 7, m);
    int w = guard(a.mpref[(long long)m * n + g], n, c->diag, 4, m, g);
    int rk = guard(a.wrank[(long long)w * n + m], n, c->diag, 5, w, m);
    unsigned long long key = sm_key(rk, m, g);
    unsigned long long old = amin64(&a.best[w], key);
    // m displaced the previous holder, who is now forbidden: he finds out by
    // re-registering in the next round
    if (old != SM_EMPTY && old > key) st_relaxed(&c->flag[r & (SM_NFLAG - 1)], 1);
    if (old < key) {
        // forbidden: any later round also sees it (best[w] only decreases)
        st_relaxed(&c->flag[r & (SM_NFLAG - 1)], 1);
        bool go = true;
        if (a.random) go = (sm_mix(a.seed ^ ((unsigned long long)r << 32) ^ (unsigned)m) & 1ull) != 0;
        if (go) {
            if (g + 1 >= n) set_status(&c->status, LLP_E_INFEASIBLE);
            else a.G[m] = g + 1;
        }
    }
}

__global__ void k_sm_decode(SArgs a, int* wife) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    for (long long m = tid; m < a.n; m += nt) {
        int g = guard(a.G[m], a.n, a.ctrl->diag, 6, (int)m);
        wife[m] = a.mpref[m * a.n + g];
    }
}

// --------------------------------------------------------------- host
static size_t sm_ws(int64_t n, SArgs* a, char* base, size_t cap) {
    Carver cv{base, cap, 0, base == nullptr};
    unsigned long long* best = cv.take<unsigned long long>(n);
    int* G = cv.take<int>(n);
    int* pend = cv.take<int>(n);
    SCtrl* ctrl = cv.take<SCtrl>(1);
    int* combo = cv.take<int>(n <= SM_LDS_MAX ? (size_t)n * SM_COMBO : 0);
    if (a) {
        a->combo = combo;
        a->best = best;
        a->G = G;
        a->pend = pend;
        a->ctrl = ctrl;
    }
    return cv.used;
}

size_t sm_workspace_bytes(int64_t n) { return sm_ws(n, nullptr, nullptr, 0); }

static int grid_for(int64_t work, int block) {
    int64_t g = (work + block - 1) / block;
    return (int)(g < 1 ? 1 : (g > 65535 * 4 ? 65535 * 4 : g));
}

int solve_sm(int32_t n, const int16_t* men_pref, const int16_t* women_rank, int32_t* wife,
             int32_t* proposal_idx, const llp_opts* opts) {
    if (n <= 0 || n > 32767) return fail(LLP_E_ARG, "n must be in [1, 32767] (got %d)", n);
    if (!men_pref || !women_rank || !wife) return fail(LLP_E_ARG, "men_pref, women_rank and wife are required");
    llp_opts o = opts_or_default(opts);
    if (o.sched > LLP_SCHED_RANDOM) return fail(LLP_E_ARG, "unknown schedule %u", o.sched);
    if (o.sched == LLP_SCHED_LEARNED || o.sched == LLP_SCHED_HYBRID)
        return fail(LLP_E_ARG, "stable marriage supports the plain, fixed and random schedules");
    if (o.chunk < 0) return fail(LLP_E_ARG, "chunk must be >= 0");
    hipStream_t st = (hipStream_t)o.stream;
    SArgs a;
    memset(&a, 0, sizeof(a));
    a.n = n;
    a.mpref = men_pref;
    a.wrank = women_rank;
    a.chunk = o.chunk;
    a.random = o.sched == LLP_SCHED_RANDOM;
    a.seed = o.seed;
    a.warm = o.warm_start;
    const bool rounds = a.random || (o.sched == LLP_SCHED_FIXED && (o.flags & LLP_DENSE));

    size_t need = sm_ws(n, nullptr, nullptr, 0);
    void* ws = nullptr;
    int s = get_workspace(o, need, &ws);
    if (s) return s;
    sm_ws(n, &a, (char*)ws, need);
    if (proposal_idx) a.G = proposal_idx;

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool timing = (o.flags & LLP_TIMING) && o.stats;
    if (timing) {
        LLP_HIP(hipEventCreate(&ev0));
        LLP_HIP(hipEventCreate(&ev1));
        LLP_HIP(hipEventRecord(ev0, st));
    }
    const int blk = 64;
    hipLaunchKernelGGL(k_sm_init, dim3(grid_for(n, 256)), dim3(256), 0, st, a, o.warm_start);
    if (o.flags & LLP_VALIDATE) hipLaunchKernelGGL(k_sm_validate, dim3(2 * n), dim3(256), 0, st, a);
    if (a.warm) hipLaunchKernelGGL(k_sm_warm_register, dim3(grid_for(n, 64)), dim3(64), 0, st, a);
    LLP_HIP(hipGetLastError());

    // Unbounded chains finish in one launch; chunked chains and dense rounds
    // need at most n * n proposals in all, hence the default round limit.
    const int64_t max_rounds = o.max_rounds > 0 ? o.max_rounds : (int64_t)n * n + 2;
    SCtrl h;
    memset(&h, 0, sizeof(h));
    int64_t r = 1;
    int batch = rounds || a.chunk > 0 ? 8 : 2;
    int status = LLP_OK;
    const bool lds = !rounds && a.chunk == 0 && !a.warm && n <= SM_LDS_MAX;
    if (lds) {
        const long long entries = (long long)n * (n < SM_COMBO ? n : SM_COMBO);
        hipLaunchKernelGGL(k_sm_combo, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, st, a);
        hipLaunchKernelGGL(k_sm_lds, dim3(1), dim3(SM_LDS_THREADS), 0, st, a);
        ++r;
    }
    while (!lds) {
        for (int i = 0; i < batch && r <= max_rounds; ++i, ++r) {
            if (rounds) hipLaunchKernelGGL(k_sm_round, dim3(grid_for(n, blk)), dim3(blk), 0, st, a, (int)r);
            else hipLaunchKernelGGL(k_sm_chain, dim3(grid_for(n, blk)), dim3(blk), 0, st, a, (int)r);
        }
        LLP_HIP(hipGetLastError());
        s = readback(st, a.ctrl, &h, sizeof(h));
        if (s) return s;
        if (h.status || h.done) break;
        if (o.abort_host && *o.abort_host) { status = LLP_E_ABORTED; break; }
        if (r > max_rounds) { status = LLP_E_NOT_CONVERGED; break; }
        if (batch < 64) batch *= 2;
    }
    hipLaunchKernelGGL(k_sm_decode, dim3(grid_for(n, 256)), dim3(256), 0, st, a, wife);
    LLP_HIP(hipGetLastError());
    if (timing) LLP_HIP(hipEventRecord(ev1, st));
    s = readback(st, a.ctrl, &h, sizeof(h));
    if (s) return s;
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = h.done ? h.last_round : (r - 1);
        o.stats->candidates = h.proposals;
        o.stats->advances = h.proposals;
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
    if (h.diag[0])
        return fail(LLP_E_INPUT, "index guard %d fired: index %d bound %d context %d %d", h.diag[0], h.diag[1],
                    h.diag[2], h.diag[3], h.diag[4]);
    if (h.status == LLP_E_INPUT) return fail(LLP_E_INPUT, "a preference list is not a permutation of 0..n-1");
    if (h.status == LLP_E_INFEASIBLE) return fail(LLP_E_INFEASIBLE, "a man exhausted his list (malformed lists)");
    if (h.status) return fail(h.status, "device status %d", h.status);
    if (status == LLP_E_NOT_CONVERGED) return fail(status, "not converged after %lld rounds", (long long)max_rounds);
    if (status == LLP_E_ABORTED) return fail(status, "aborted by the host flag");
    return LLP_OK;
}

}  // namespace llp

extern "C" int llp_solve_sm(int32_t n, const int16_t* men_pref, const int16_t* women_rank, int32_t* wife,
                            int32_t* proposal_idx, const llp_opts* opts) {
    return llp::solve_sm(n, men_pref, women_rank, wife, proposal_idx, opts);
}

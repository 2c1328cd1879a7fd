// jobs.hip - earliest start times of a job DAG (paper Section 5.5) on gfx950,
// with the paper's readiness counters.
//
// State.  S[j] is the start time of job j (bottom 0); alpha(S, j) is the
// largest S[p] + dur[p] over its predecessors p.  The paper adds readiness to
// the predicate: a job is only evaluated once every predecessor is fixed, so
// each job is advanced exactly once, to its final value, and the work is
// proportional to the arcs.
//
// Rounds.  Round r consumes the list R[r-1] of jobs that became ready (fixed)
// in round r-1 and walks their successor arcs, edge-balanced across waves:
// each arc (p -> j) publishes S[p] + dur[p] into S[j] with atomicMax and
// decrements j's counter of unfixed predecessors; the arc that brings the
// counter to zero appends j to R[r].  Every contribution to S[j] is made in an
// earlier launch than the one that reads S[j] (j is read only when R[r] is
// consumed by round r+1), so the kernel boundary orders them.  A round with
// an empty input list ends the sweep; a job whose counter never reached zero
// lies on (or after) a cycle.  The pull form of the sweep (LLP_JOBS_PULL)
// runs in the generic graph sweep.
//
// Narrow levels.  A level of at most JN_ARCS arcs (most levels of a deep DAG
// are a few jobs wide) is run by workgroup 0 alone, which keeps running the
// following levels in the same launch, with both lists in LDS, while they
// stay that narrow (at most JN_LEVELS per launch, so the host's abort flag
// and round limit are seen in time).  Its rounds are separated by a full
// wait on its memory operations and a workgroup barrier: a job made ready in
// round r is read in round r + 1 through agent-scope loads, after every
// atomicMax on it has completed, so the launch boundary is not needed there.
// The launch hands the first wide level's list to the next launch through
// one of two small hand-over lists (alternating, so a launch never writes the
// list it was given: a late workgroup of it may still be reading the list's
// totals).  Every launch takes its level and its input list from the slots
// the previous launch wrote (lvl / src, by launch parity).
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include "llp_host.h"
#include "llp_lists.h"

namespace llp {

constexpr int JB = 256;            // threads per workgroup
constexpr int JW = JB / LLP_WAVE;  // waves per workgroup
constexpr int J_MAX_SEG = 1024;
constexpr int JN_ARCS = 1024;      // widest level (arcs) run in the narrow form
constexpr int JN_LEVELS = 64;      // narrow levels per launch at most
constexpr int JN_PER = JN_ARCS / JB;

struct JCtrl {
    int done;
    int status;
    int last_round;
    int over;           // a level past the round limit had jobs to run
    int diag[8];
    long long rounds, ready, edges;
    int lvl[2];         // launch k runs level lvl[k & 1] ...
    int src[2];         // ... from list src[k & 1]: 0 = R[level - 1], 1 / 2 = hand-over list h0 / h1
    int end_k;          // the launch that ended the sweep
    int pad2;
};

struct JArgs {
    int n, E;
    const int* pred_ptr;
    const int* pred_idx;
    const int* dur;
    const int* succ_ptr;
    const int* succ_idx;
    int* S;
    int* cnt;          // unfixed predecessors per job
    ListRef l0, l1;
    ListRef h0, h1;    // hand-over lists of the narrow form (segment 0 only, JN_ARCS entries)
    int nseg;
    int narrow;        // widest level run in the narrow form (arcs), 0 = none
    long long max_rounds;
    JCtrl* ctrl;
};

struct JShared {
    int cpre[J_MAX_SEG + 1];
    int epre[J_MAX_SEG + 1];
    int own[JW][64];
    unsigned long long ctr;
    int tot_edges, tot_count;
    int tmp[JW + 1];
    // narrow form: the current and the next level's entries {job, first
    // successor arc, -, successor count}, per entry of the current level
    // its first arc (exclusive prefix) and completion time
    int4 q[2][JN_ARCS];
    int qpre[JN_ARCS + 1];
    int qcm[JN_ARCS];
    int qn[2], qe[2];
    int ovf;
};

__device__ __forceinline__ ListRef jl_of(const JArgs& a, int r) { return (r & 1) ? a.l1 : a.l0; }

__global__ void k_jobs_init(JArgs a, const int* warm) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    for (long long j = tid; j < a.n; j += nt) {
        int s = warm ? warm[j] : 0;
        a.S[j] = s > 0 ? s : 0;
        a.cnt[j] = a.pred_ptr[j + 1] - a.pred_ptr[j];
    }
    for (long long s = tid; s < a.nseg; s += nt) {
        a.l0.seg[s] = 0ull;
        a.l1.seg[s] = 0ull;
        a.h0.seg[s] = 0ull;
        a.h1.seg[s] = 0ull;
    }
    if (tid == 0) {
        JCtrl c;
        memset(&c, 0, sizeof(c));
        c.lvl[0] = 1;   // the first launch runs level 1 from R[0]
        *a.ctrl = c;
    }
}

// Validation: row offsets, ids, durations, and that the successor lists hold
// the same arcs as the predecessor lists (per-job counts; cnt is the
// scratch counter here and is re-initialised afterwards).
__global__ void k_jobs_validate_count(JArgs a) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    bool bad = false;
    for (long long j = tid; j <= a.n; j += nt) {
        int p = a.pred_ptr[j], q = a.succ_ptr[j];
        if (j == 0 && (p != 0 || q != 0)) bad = true;
        if (j == a.n && (p != a.E || q != a.E)) bad = true;
        if (j < a.n) {
            if (a.pred_ptr[j + 1] < p || a.succ_ptr[j + 1] < q) bad = true;
            if (a.dur[j] < 0) bad = true;
        }
    }
    for (long long e = tid; e < a.E; e += nt) {
        int x = a.pred_idx[e], y = a.succ_idx[e];
        if (x < 0 || x >= a.n || y < 0 || y >= a.n) {
            bad = true;
            continue;
        }
        aadd(&a.cnt[y], -1);
    }
    if (bad) set_status(&a.ctrl->status, LLP_E_INPUT);
}

__global__ void k_jobs_validate_check(JArgs a) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    for (long long j = tid; j < a.n; j += nt)
        if (a.cnt[j] != 0) set_status(&a.ctrl->status, LLP_E_INPUT);
}

// R[0]: the jobs without predecessors.  Workgroup b seeds a contiguous block
// of jobs into its own segment.
__global__ void __launch_bounds__(JB) k_jobs_seed(JArgs a) {
    __shared__ unsigned long long ctr;
    if (ld_relaxed(&a.ctrl->status)) return;
    if (threadIdx.x == 0) ctr = 0ull;
    __syncthreads();
    const int per = (a.n + gridDim.x - 1) / gridDim.x;
    const int b = blockIdx.x * per, e = min(b + per, a.n);
    for (int base = b; base < e; base += JB) {
        int j = base + threadIdx.x;
        bool ready = false;
        int sb = 0, deg = 0;
        if (j < e) {
            ready = a.pred_ptr[j + 1] == a.pred_ptr[j];
            sb = a.succ_ptr[j];
            deg = a.succ_ptr[j + 1] - sb;
        }
        append(ready && deg > 0, j, sb, deg, &ctr, a.l0, &a.ctrl->status);
    }
    __syncthreads();
    if (threadIdx.x == 0) a.l0.seg[blockIdx.x] = ctr;
}

__device__ __forceinline__ void jobs_wave_range(int total, int& wb, int& we) {
    const long long W = (long long)gridDim.x * JW;
    const long long w = (long long)blockIdx.x * JW + (threadIdx.x >> 6);
    wb = (int)((long long)total * w / W);
    we = (int)((long long)total * (w + 1) / W);
}

// Block-wide exclusive prefix of the successor counts of the n entries in
// q (JN_PER per thread, in order); returns the total.
__device__ int jn_prefix(const int4* q, int n, int* pre, int* tmp) {
    const int t = threadIdx.x, b = t * JN_PER;
    int d[JN_PER], sum = 0;
#pragma unroll
    for (int i = 0; i < JN_PER; ++i) {
        d[i] = b + i < n ? q[b + i].w : 0;
        sum += d[i];
    }
    const int incl = wave_incl_sum(sum);
    if (lane() == LLP_WAVE - 1) tmp[t >> 6] = incl;
    __syncthreads();
    int before = incl - sum, tot = 0;
    for (int w = 0; w < JW; ++w) {
        if (w < (t >> 6)) before += tmp[w];
        tot += tmp[w];
    }
#pragma unroll
    for (int i = 0; i < JN_PER; ++i) {
        if (b + i < n) pre[b + i] = before;
        before += d[i];
    }
    __syncthreads();   // tmp is reused by the caller
    return tot;
}

// The narrow form, run by workgroup 0 of launch k from level r (input list
// in, holding at most JN_ARCS entries and arcs).  See the file comment.
__device__ void jobs_narrow(const JArgs& a, int k, int r, const ListRef& in, int si, JShared& sh) {
    JCtrl* c = a.ctrl;
    const int t = threadIdx.x;
    if (t == 0) {
        sh.qn[0] = sh.qn[1] = 0;
        sh.qe[0] = sh.qe[1] = 0;
        sh.ovf = 0;
    }
    __syncthreads();
    // stage R[r-1] into q[0] (entries in any segments, in any order)
    for (int sg = t; sg < a.nseg; sg += JB) {
        const int cs = min(sh.cpre[sg + 1] - sh.cpre[sg], in.cap);
        if (cs > 0) {
            const int b = atomicAdd(&sh.qn[0], cs);
            for (int i = 0; i < cs; ++i) sh.q[0][b + i] = in.ent[(long long)sg * in.cap + i];
        }
    }
    __syncthreads();
    int cur = 0, lv = r, levels = 0;
    long long ready = 0, edges = 0;
    for (;;) {
        const int n_in = sh.qn[cur], nx = cur ^ 1;
        // completion time of every entry (agent-scope loads: its start time
        // was raised by atomics of this workgroup's previous round)
        for (int i = t; i < n_in; i += JB) {
            const int p = guard(sh.q[cur][i].x, a.n, c->diag, 74);
            const long long cm = (long long)ld_i32<true>(a.S + p) + a.dur[p];
            if (cm > LLP_INF) sh.ovf = 1;
            sh.qcm[i] = cm > LLP_INF ? LLP_INF : (int)cm;
        }
        const int T = jn_prefix(sh.q[cur], n_in, sh.qpre, sh.tmp);
        ready += n_in;
        edges += T;
        // the level's arcs, JN_PER per thread: every load before any is used
        int j[JN_PER], cm[JN_PER];
        bool act[JN_PER], rd[JN_PER];
#pragma unroll
        for (int q4 = 0; q4 < JN_PER; ++q4) {
            const int e = t + q4 * JB;
            act[q4] = e < T;
            j[q4] = 0;
            cm[q4] = 0;
            if (act[q4]) {
                int lo = 0, hi = n_in;   // last entry whose first arc is <= e
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (sh.qpre[mid] <= e) lo = mid;
                    else hi = mid;
                }
                const int4 en = sh.q[cur][lo];
                cm[q4] = sh.qcm[lo];
                const int ea = guard(en.y + (e - sh.qpre[lo]), a.E, c->diag, 75, en.x);
                j[q4] = guard(a.succ_idx[ea], a.n, c->diag, 76, ea);
            }
        }
#pragma unroll
        for (int q4 = 0; q4 < JN_PER; ++q4)
            if (act[q4]) amax(&a.S[j[q4]], cm[q4]);
#pragma unroll
        for (int q4 = 0; q4 < JN_PER; ++q4) rd[q4] = act[q4] && aadd(&a.cnt[j[q4]], -1) == 1;
#pragma unroll
        for (int q4 = 0; q4 < JN_PER; ++q4) {
            if (rd[q4]) {
                const int sb = a.succ_ptr[j[q4]];
                const int deg = a.succ_ptr[j[q4] + 1] - sb;
                if (deg > 0) {
                    const int idx = atomicAdd(&sh.qn[nx], 1);   // < JN_ARCS: one per arc at most
                    atomicAdd(&sh.qe[nx], deg);
                    sh.q[nx][idx] = make_int4(j[q4], sb, 0, deg);
                }
            }
        }
        // every atomic of the round has completed before the barrier
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        ++levels;
        const int n_out = sh.qn[nx], e_out = sh.qe[nx];
        const bool stop = sh.ovf != 0;
        const bool end = n_out == 0;
        const bool wide = e_out > a.narrow || levels >= JN_LEVELS || (long long)lv + 1 > a.max_rounds;
        if (stop || end || wide) {
            if (t == 0) {
                c->rounds = lv;
                c->ready += ready;
                c->edges += edges;
                if (stop) set_status(&c->status, LLP_E_OVERFLOW);
                if (end) {
                    c->done = 1;
                    c->last_round = lv;
                    c->end_k = k;
                }
            }
            if (!stop && !end) {
                // the next level's list: into the hand-over list this launch
                // was not given, segment 0, arc offsets in order
                const ListRef h = si == 1 ? a.h1 : a.h0;
                const int tot = jn_prefix(sh.q[nx], n_out, sh.qpre, sh.tmp);
                for (int i = t; i < n_out; i += JB) {
                    int4 en = sh.q[nx][i];
                    en.z = sh.qpre[i];
                    h.ent[i] = en;
                }
                if (t == 0) {
                    h.seg[0] = (unsigned long long)(unsigned)n_out | ((unsigned long long)(unsigned)tot << 32);
                    c->lvl[(k + 1) & 1] = lv + 1;
                    c->src[(k + 1) & 1] = si == 1 ? 2 : 1;
                }
            }
            return;
        }
        if (t == 0) {
            sh.qn[cur] = 0;
            sh.qe[cur] = 0;
        }
        __syncthreads();
        cur = nx;
        ++lv;
    }
}

// Launch k: level r = lvl[k & 1] from its input list; a narrow level starts
// the narrow form in workgroup 0, and the other workgroups return.
__global__ void __launch_bounds__(JB) k_jobs_level(JArgs a, int k) {
    __shared__ JShared sh;
    JCtrl* c = a.ctrl;
    if (ld_relaxed(&c->done) || ld_relaxed(&c->status)) return;
    const int r = c->lvl[k & 1], si = c->src[k & 1];
    const ListRef in = si == 0 ? jl_of(a, r - 1) : (si == 1 ? a.h0 : a.h1);
    load_segments(in.seg, a.nseg, sh.cpre, sh.epre, sh.tmp, &sh.tot_edges, &sh.tot_count);
    if (sh.tot_count == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c->done = 1;
            c->last_round = r - 1;
            c->end_k = k;
        }
        return;
    }
    if ((long long)r > a.max_rounds) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c->over = 1;
            c->done = 1;
            c->last_round = r - 1;
        }
        return;
    }
    if (sh.tot_edges <= a.narrow && sh.tot_count <= JN_ARCS) {
        if (blockIdx.x == 0) jobs_narrow(a, k, r, in, si, sh);
        return;
    }
    const ListRef out = jl_of(a, r);
    if (threadIdx.x == 0) sh.ctr = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->rounds = r;
        c->ready += sh.tot_count;
        c->edges += sh.tot_edges;
        c->lvl[(k + 1) & 1] = r + 1;
        c->src[(k + 1) & 1] = 0;
    }
    __syncthreads();
    SegView sv{in.ent, in.cap, a.nseg, sh.cpre, sh.epre, sh.tot_edges, sh.tot_count};
    ListSrc src{sv, c->diag};
    int wb, we;
    jobs_wave_range(sh.tot_edges, wb, we);
    int* own = sh.own[threadIdx.x >> 6];
    bool ovf = false;
    for_edges(src, wb, we, own, [&](const EdgeCtx& x) {
        // completion time of each window entry, handed to its arcs
        long long cm = 0;
        if (x.mine_valid) {
            int p = guard(x.mine.x, a.n, c->diag, 71);
            cm = (long long)a.S[p] + a.dur[p];
        }
        if (cm > LLP_INF) {
            ovf = true;
            cm = LLP_INF;
        }
        int cp = shfl((int)cm, x.j);
        bool ready = false;
        int j = 0, sb = 0, deg = 0;
        if (x.active) {
            int e = guard(x.csr, a.E, c->diag, 72, x.own.x, x.own.y);
            j = guard(a.succ_idx[e], a.n, c->diag, 73, e);
            amax(&a.S[j], cp);
            ready = aadd(&a.cnt[j], -1) == 1;
            if (ready) {
                sb = a.succ_ptr[j];
                deg = a.succ_ptr[j + 1] - sb;
            }
        }
        append(ready && deg > 0, j, sb, deg, &sh.ctr, out, &c->status);
    });
    __syncthreads();
    if (threadIdx.x == 0) out.seg[blockIdx.x] = sh.ctr;
    if (__any(ovf) && lane() == 0) set_status(&c->status, LLP_E_OVERFLOW);
}

// Completion times must fit int32; a job never made ready lies on a cycle.
__global__ void k_jobs_final(JArgs a) {
    const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long nt = (long long)gridDim.x * blockDim.x;
    bool ovf = false, cyc = false;
    for (long long j = tid; j < a.n; j += nt) {
        if ((long long)a.S[j] + a.dur[j] > LLP_INF) ovf = true;
        if (a.cnt[j] != 0) cyc = true;
    }
    if (cyc) set_status(&a.ctrl->status, LLP_E_CYCLE);
    if (ovf) set_status(&a.ctrl->status, LLP_E_OVERFLOW);
}

// --------------------------------------------------------------- host
struct JobsLayout {
    int nseg;
    int cap;
};

// One list segment (and workgroup) per CU: a level is a chain of round trips,
// and half the workgroups of two per CU scan half the totals and end sooner.
// At 2^20, 2^18, 2^16 and 10^4 jobs on 256 CUs: one per CU 2117, 1326, 944 and
// 602 us, two 2125, 1345, 1004 and 616, three 2152, 1421, 1065 and 637 (while a
// window of entries ended with its segment two were the better: 2.57 ms
// against 2.61).  The scratch asked for is that of two, which is never smaller.
constexpr int JOBS_PER_CU = 1, JOBS_SCRATCH_PER_CU = 2;
static JobsLayout jobs_layout(int64_t n, int64_t E, int per_cu) {
    JobsLayout L;
    L.nseg = device_info().cus * per_cu;
    if (L.nseg > J_MAX_SEG) L.nseg = J_MAX_SEG;
    if (L.nseg < 1) L.nseg = 1;
    long long W = (long long)L.nseg * JW;
    long long per_wave = (E + W - 1) / W;
    long long cap_level = JW * per_wave + JW * 2 + 64;
    long long cap_seed = (n + L.nseg - 1) / L.nseg + 64;
    L.cap = (int)(cap_level > cap_seed ? cap_level : cap_seed);
    return L;
}

static size_t jobs_ws(int64_t n, int64_t E, int per_cu, JArgs* a, char* base, size_t cap) {
    JobsLayout L = jobs_layout(n, E, per_cu);
    Carver cv{base, cap, 0, base == nullptr};
    int* cnt = cv.take<int>(n);
    JCtrl* ctrl = cv.take<JCtrl>(1);
    ListRef lists[4];
    for (int i = 0; i < 4; ++i) {
        // lists 2 and 3 hand a narrow launch's last list over (segment 0)
        const int cap = i < 2 ? L.cap : JN_ARCS;
        lists[i].seg = cv.take<unsigned long long>(L.nseg);
        lists[i].ent = cv.take<int4>((size_t)L.nseg * cap);
        lists[i].cap = cap;
        lists[i].segmin = nullptr;
    }
    if (a) {
        a->cnt = cnt;
        a->ctrl = ctrl;
        a->l0 = lists[0];
        a->l1 = lists[1];
        a->h0 = lists[2];
        a->h1 = lists[3];
        a->nseg = L.nseg;
    }
    return cv.used;
}

// the pull form shares the graph sweep's workspace
size_t graph_workspace_bytes(int64_t n, int64_t m, int chunk);

size_t jobs_workspace_bytes(int64_t n, int64_t E, int chunk) {
    size_t a = jobs_ws(n, E, JOBS_SCRATCH_PER_CU, nullptr, nullptr, 0);
    size_t b = graph_workspace_bytes(n, E, chunk);
    return a > b ? a : b;
}

int solve_jobs_pull(int32_t n, const int32_t* pred_ptr, const int32_t* pred_idx, const int32_t* dur,
                    const int32_t* succ_ptr, const int32_t* succ_idx, int32_t* start, const llp_opts* opts,
                    int64_t E);

// level launches of the last sweep, by (predecessor and successor arrays, n,
// arc count, narrow limit)
using JobsKey = std::tuple<const void*, const void*, int, int, int>;
static std::mutex g_jmu;
static std::map<JobsKey, int> g_jhist;

static int grid1(int64_t work) {
    int64_t g = (work + 255) / 256;
    if (g < 1) g = 1;
    int cap = device_info().cus * 8;
    return (int)(g < cap ? g : cap);
}

int solve_jobs(int32_t n, const int32_t* pred_ptr, const int32_t* pred_idx, const int32_t* dur,
               const int32_t* succ_ptr, const int32_t* succ_idx, int32_t* start, const llp_opts* opts) {
    if (n <= 0) return fail(LLP_E_ARG, "n must be positive (got %d)", n);
    if (!pred_ptr || !dur || !succ_ptr || !start)
        return fail(LLP_E_ARG, "pred_ptr, dur, succ_ptr and start are required");
    llp_opts o = opts_or_default(opts);
    hipStream_t st = (hipStream_t)o.stream;
    // the arc count is the last row offset
    int E = 0;
    int s = readback(st, pred_ptr + n, &E, sizeof(int));
    if (s) return s;
    if (E < 0) return fail(LLP_E_INPUT, "pred_ptr[n] is negative");
    if (E > 0 && (!pred_idx || !succ_idx)) return fail(LLP_E_ARG, "pred_idx and succ_idx are required");
    if (o.flags & LLP_JOBS_PULL) return solve_jobs_pull(n, pred_ptr, pred_idx, dur, succ_ptr, succ_idx, start, opts, E);
    if (o.sched != LLP_SCHED_PLAIN)
        return fail(LLP_E_ARG, "the readiness schedule takes no schedule options (use LLP_JOBS_PULL)");

    JArgs a;
    memset(&a, 0, sizeof(a));
    a.n = n;
    a.E = E;
    a.pred_ptr = pred_ptr;
    a.pred_idx = pred_idx;
    a.dur = dur;
    a.succ_ptr = succ_ptr;
    a.succ_idx = succ_idx;
    a.S = start;
    a.narrow = o.chunk < 0 ? 0 : (o.chunk == 0 ? JN_ARCS : std::min<int>(o.chunk, JN_ARCS));
    a.max_rounds = o.max_rounds > 0 ? o.max_rounds : (int64_t)n + 2;
    size_t need = jobs_ws(n, E, JOBS_SCRATCH_PER_CU, nullptr, nullptr, 0);
    void* ws = nullptr;
    s = get_workspace(o, need, &ws);
    if (s) return s;
    jobs_ws(n, E, JOBS_PER_CU, &a, (char*)ws, need);

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool timing = (o.flags & LLP_TIMING) && o.stats;
    if (timing) {
        LLP_HIP(hipEventCreate(&ev0));
        LLP_HIP(hipEventCreate(&ev1));
        LLP_HIP(hipEventRecord(ev0, st));
    }
    const int g1 = grid1((int64_t)n > E ? n : E);
    hipLaunchKernelGGL(k_jobs_init, dim3(grid1(n)), dim3(256), 0, st, a, o.warm_start);
    if (o.flags & LLP_VALIDATE) {
        hipLaunchKernelGGL(k_jobs_validate_count, dim3(g1), dim3(256), 0, st, a);
        hipLaunchKernelGGL(k_jobs_validate_check, dim3(grid1(n)), dim3(256), 0, st, a);
        JCtrl h0;
        s = readback(st, a.ctrl, &h0, sizeof(h0));
        if (s) return s;
        if (h0.status) return fail(LLP_E_INPUT, "job lists failed validation (offsets, ids, durations or arc sets)");
        hipLaunchKernelGGL(k_jobs_init, dim3(grid1(n)), dim3(256), 0, st, a, o.warm_start);
    }
    hipLaunchKernelGGL(k_jobs_seed, dim3(a.nseg), dim3(JB), 0, st, a);
    LLP_HIP(hipGetLastError());

    const int64_t max_rounds = o.max_rounds > 0 ? o.max_rounds : (int64_t)n + 2;
    JCtrl h;
    memset(&h, 0, sizeof(h));
    // every launch runs at least one level or ends the sweep (a level past
    // the limit sets over)
    const int64_t max_launches = max_rounds + 2;
    int64_t k = 0;
    int batch = 8;
    // the level launches the last sweep of the same arrays needed: the first
    // batch is sized from it, so a repeated solve enqueues few launches past
    // its end (each costs a few microseconds); outputs do not depend on it
    const JobsKey key((const void*)pred_ptr, (const void*)succ_ptr, n, E, a.narrow);
    {
        std::lock_guard<std::mutex> lk(g_jmu);
        auto it = g_jhist.find(key);
        if (it != g_jhist.end()) batch = std::max(2, it->second + 1);
    }
    int status = LLP_OK;
    if (o.abort_host && *o.abort_host) status = LLP_E_ABORTED;   // set before the solve: no launch
    for (; status == LLP_OK;) {
        for (int i = 0; i < batch && k < max_launches; ++i, ++k)
            hipLaunchKernelGGL(k_jobs_level, dim3(a.nseg), dim3(JB), 0, st, a, (int)k);
        LLP_HIP(hipGetLastError());
        s = readback(st, a.ctrl, &h, sizeof(h));
        if (s) return s;
        if (h.status) break;
        if (h.done) {
            if (h.over) status = LLP_E_NOT_CONVERGED;
            break;
        }
        if (o.abort_host && *o.abort_host) { status = LLP_E_ABORTED; break; }
        if (k >= max_launches) { status = LLP_E_NOT_CONVERGED; break; }
        if (batch < 64) batch *= 2;
    }
    if (status == LLP_OK && h.status == 0 && h.done && !h.over) {
        std::lock_guard<std::mutex> lk(g_jmu);
        if (g_jhist.size() >= 256) g_jhist.clear();
        g_jhist[key] = h.end_k + 1;
    }
    if (status == LLP_OK && h.status == 0) hipLaunchKernelGGL(k_jobs_final, dim3(grid1(n)), dim3(256), 0, st, a);
    LLP_HIP(hipGetLastError());
    if (timing) LLP_HIP(hipEventRecord(ev1, st));
    s = readback(st, a.ctrl, &h, sizeof(h));
    if (s) return s;
    if (o.stats) {
        memset(o.stats, 0, sizeof(*o.stats));
        o.stats->rounds = h.rounds;
        o.stats->candidates = h.ready;
        o.stats->advances = h.ready;
        o.stats->edges_inspected = h.edges;
        o.stats->states_gathered = h.edges;
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
    if (h.status == LLP_E_CYCLE) return fail(LLP_E_CYCLE, "the job arcs contain a cycle");
    if (h.status == LLP_E_OVERFLOW) return fail(LLP_E_OVERFLOW, "a completion time does not fit int32");
    if (h.status) return fail(h.status, "device status %d", h.status);
    if (status == LLP_E_NOT_CONVERGED) return fail(status, "not converged after %lld rounds", (long long)max_rounds);
    if (status == LLP_E_ABORTED) return fail(status, "aborted by the host flag");
    return LLP_OK;
}

}  // namespace llp

extern "C" int llp_solve_jobs(int32_t n, const int32_t* pred_ptr, const int32_t* pred_idx, const int32_t* dur,
                              const int32_t* succ_ptr, const int32_t* succ_idx, int32_t* start,
                              const llp_opts* opts) {
    return llp::solve_jobs(n, pred_ptr, pred_idx, dur, succ_ptr, succ_idx, start, opts);
}

"""The calls whose speed is measured: one case per problem family of the library,
at the sizes its benchmark, tests and training run use.

Every call goes through the Python binding, with the output buffers and the
workspace that a program solving repeatedly keeps.  Inputs are synthetic and
made on the GPU from the seed: R-MAT graphs with relabelled vertices, uniform
graphs with a Hamiltonian cycle, 4-neighbour grids, random preference lists,
random job DAGs, knapsack instances, 64-bit words and scheduler features.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2603_13147_amd as llp

DEV = "cuda"
SCHED = {"plain": llp.SCHED_PLAIN, "hybrid": llp.SCHED_HYBRID, "learned": llp.SCHED_LEARNED}


def listed():
    return [
        # one small query on a small graph: the launches and the latency count
        {"name": "sssp_uniform_4096", "kind": "sssp", "graph": "uniform", "n": 4096, "sched": "hybrid"},
        # the headline benchmark's two sweeps: a power-law graph of 71 M arcs
        {"name": "sssp_rmat22", "kind": "sssp", "graph": "rmat", "scale": 22, "sched": "hybrid"},
        {"name": "bfs_rmat22", "kind": "bfs", "graph": "rmat", "scale": 22, "sched": "hybrid"},
        # a road-like mesh: a long diameter and hundreds of narrow rounds
        {"name": "sssp_grid_2048", "kind": "sssp", "graph": "grid", "rows": 2048, "cols": 2048, "sched": "hybrid"},
        # what a call without options runs: the plain schedule
        {"name": "sssp_rmat18_plain", "kind": "sssp", "graph": "rmat", "scale": 18, "sched": "plain"},
        # a matching market of the benchmark's size (134 MB of lists)
        {"name": "marriage_8192", "kind": "sm", "n": 8192},
        # a sparse job DAG of a million jobs, about 8 prerequisites each
        {"name": "jobs_2e20", "kind": "jobs", "n": 1 << 20, "pull": False},
        # one knapsack of the largest published size
        {"name": "knapsack_4000x6400", "kind": "knapsack", "items": 4000, "W": 6400},
        # reachability of a sparse digraph
        {"name": "closure_8192", "kind": "tc", "n": 8192, "m": 65536},
        # a bulk reduction
        {"name": "reduce_2e24", "kind": "reduce", "n": 1 << 24},
        # thousands of small instances in one captured launch
        {"name": "batch_8192", "kind": "batch", "knapsacks": 4096, "graphs": 4096},
        # one full-batch training step of the scheduler's network on the
        # number of rounds its training run labels
        {"name": "train_step_859", "kind": "mlp", "rows": 859},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["uniform", "rmat", "rmat", "grid", "sm", "jobs", "knapsack", "tc", "reduce", "batch", "mlp"])
    if kind == "uniform":
        return {"kind": rng.choice(["sssp", "bfs"]), "graph": "uniform", "n": _log_int(rng, 64, 65536),
                "sched": rng.choice(["hybrid", "plain"])}
    if kind == "rmat":
        return {"kind": rng.choice(["sssp", "bfs"]), "graph": "rmat", "scale": rng.randint(10, 21),
                "sched": rng.choice(["hybrid", "hybrid", "plain", "learned"])}
    if kind == "grid":
        return {"kind": rng.choice(["sssp", "bfs"]), "graph": "grid", "rows": _log_int(rng, 16, 1024),
                "cols": _log_int(rng, 16, 2048), "sched": "hybrid"}
    if kind == "sm":
        return {"kind": "sm", "n": _log_int(rng, 10, 8192)}
    if kind == "jobs":
        # the readiness sweep and, less often, the pull form on smaller DAGs
        pull = rng.random() < 0.25
        return {"kind": "jobs", "n": _log_int(rng, 100, 1 << 16 if pull else 1 << 20), "pull": pull}
    if kind == "knapsack":
        return {"kind": "knapsack", "items": _log_int(rng, 16, 4000), "W": _log_int(rng, 256, 6400)}
    if kind == "tc":
        n = _log_int(rng, 32, 8192)
        return {"kind": "tc", "n": n, "m": n * rng.randint(1, 8) + rng.randint(0, 7)}
    if kind == "reduce":
        return {"kind": "reduce", "n": _log_int(rng, 1000, 1 << 24)}
    if kind == "batch":
        return {"kind": "batch", "knapsacks": _log_int(rng, 64, 4096), "graphs": _log_int(rng, 64, 4096)}
    return {"kind": "mlp", "rows": _log_int(rng, 64, 1 << 18)}


# ---------------------------------------------------------------- inputs
def _gen(seed, device=DEV):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _ints(g, n, lo, hi):
    return torch.randint(lo, hi + 1, (n,), generator=g, device=DEV, dtype=torch.int32)


def _rows(key, n, *cols):
    """Row offsets of the arcs sorted by key (stable), and the columns in that order."""
    order = torch.sort(key, stable=True).indices
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(key, minlength=n), 0)
    return (ptr.int(),) + tuple(c[order] for c in cols)


def _csr(n, src, dst, w):
    in_ptr, in_src, in_w = _rows(dst, n, src, w)
    out_ptr, out_dst, out_w = _rows(src, n, dst, w)
    return SimpleNamespace(n=n, m=src.numel(), in_ptr=in_ptr, in_src=in_src, in_w=in_w, out_ptr=out_ptr,
                           out_dst=out_dst, out_w=out_w)


def _with_cycle(n, src, dst):
    i = torch.arange(n, device=DEV, dtype=torch.int32)
    return torch.cat([src, i]), torch.cat([dst, (i + 1) % n])


def _uniform_arcs(g, n, m):
    """m arcs with uniform tails, each to another vertex."""
    src = _ints(g, m, 0, n - 1)
    dst = (src + _ints(g, m, 1, max(n - 1, 1))) % n
    return src, dst


def _graph(case, seed):
    """(arrays, source) of the case's graph."""
    g = _gen(seed)
    if case["graph"] == "uniform":
        n = case["n"]
        src, dst = _with_cycle(n, *_uniform_arcs(g, n, 8 * n))
        return _csr(n, src, dst, _ints(g, src.numel(), 1, 100)), 0
    if case["graph"] == "grid":
        rows, cols = case["rows"], case["cols"]
        v = torch.arange(rows * cols, device=DEV, dtype=torch.int32).view(rows, cols)
        a = torch.cat([v[:, :-1].reshape(-1), v[:-1].reshape(-1)])
        b = torch.cat([v[:, 1:].reshape(-1), v[1:].reshape(-1)])
        src, dst = torch.cat([a, b]), torch.cat([b, a])
        source = int(_ints(g, 1, 0, rows * cols - 1))
        return _csr(rows * cols, src, dst, _ints(g, src.numel(), 1, 1000)), source
    # R-MAT with (a, b, c, d) = (.57, .19, .19, .05), 16 arcs per vertex,
    # vertices relabelled, plus a Hamiltonian cycle; from the highest out-degree
    n = 1 << case["scale"]
    m = 16 * n
    src = torch.zeros(m, dtype=torch.int32, device=DEV)
    dst = torch.zeros(m, dtype=torch.int32, device=DEV)
    for _ in range(case["scale"]):
        r = torch.rand(m, generator=g, device=DEV)
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    p = torch.randperm(n, generator=g, device=DEV, dtype=torch.int32)
    src, dst = _with_cycle(n, p[src], p[dst])
    c = _csr(n, src.int(), dst.int(), _ints(g, src.numel(), 1, 255))
    return c, int(torch.argmax(c.out_ptr[1:] - c.out_ptr[:-1]))


def _prepare_graph(case, seed):
    c, source = _graph(case, seed)
    bfs = case["kind"] == "bfs"
    dg = llp.DeviceGraph(c, weighted=not bfs)
    if case["sched"] == "learned":
        llp.set_sched_weights(np.load(llp.default_sched_weights_path()))
    return SimpleNamespace(solve=llp.bfs if bfs else llp.sssp, dg=dg, source=source, sched=SCHED[case["sched"]],
                           out=torch.empty(dg.n, dtype=torch.int32, device=DEV),
                           ws=llp.workspace(llp.KIND_BFS if bfs else llp.KIND_SSSP, dg.n, dg.m))


def _run_graph(s):
    return s.solve(s.dg, s.source, out=s.out, ws=s.ws, sched=s.sched)


def _prepare_sm(case, seed):
    g, n = _gen(seed), case["n"]
    mpref = torch.rand(n, n, generator=g, device=DEV).argsort(dim=1).short()
    wrank = torch.rand(n, n, generator=g, device=DEV).argsort(dim=1).short()
    return SimpleNamespace(mpref=mpref, wrank=wrank, wife=torch.empty(n, dtype=torch.int32, device=DEV),
                           prop=torch.empty(n, dtype=torch.int32, device=DEV), ws=llp.workspace(llp.KIND_SM, n, 0))


def _run_sm(s):
    return llp.stable_marriage(s.mpref, s.wrank, wife=s.wife, prop=s.prop, ws=s.ws)


def _prepare_jobs(case, seed):
    g, n = _gen(seed), case["n"]
    j = torch.arange(n, device=DEV)
    k = torch.minimum(torch.poisson(torch.full((n,), 8.0, device=DEV), generator=g).long(), j)
    child = torch.repeat_interleave(j, k)
    parent = (torch.rand(child.numel(), generator=g, device=DEV, dtype=torch.float64) * child).long()
    arcs = torch.unique(child * n + parent)   # distinct parents
    child, parent = (arcs // n).int(), (arcs % n).int()
    pp, pi = _rows(child, n, parent)
    sp, si = _rows(parent, n, child)
    return SimpleNamespace(args=(pp, pi, _ints(g, n, 1, 1000), sp, si), pull=case["pull"],
                           out=torch.empty(n, dtype=torch.int32, device=DEV),
                           ws=llp.workspace(llp.KIND_JOBS, n, pi.numel()))


def _run_jobs(s):
    if s.pull:
        return llp.jobs(*s.args, out=s.out, ws=s.ws, pull=True, sched=llp.SCHED_HYBRID)
    return llp.jobs(*s.args, out=s.out, ws=s.ws)


def _prepare_knapsack(case, seed):
    g, items, W = _gen(seed), case["items"], case["W"]
    return SimpleNamespace(wt=_ints(g, items, 1, max(W // 4, 1)), val=_ints(g, items, 1, 1000), W=W,
                           ws=llp.workspace(llp.KIND_KNAPSACK, items, W))


def _run_knapsack(s):
    return llp.knapsack(s.wt, s.val, s.W, row=True, ws=s.ws)


def _prepare_tc(case, seed):
    n = case["n"]
    src, dst = _uniform_arcs(_gen(seed), n, case["m"])
    ptr, dst = _rows(src, n, dst)
    return SimpleNamespace(n=n, ptr=ptr, dst=dst, ws=llp.workspace(llp.KIND_TC, n, dst.numel()))


def _run_tc(s):
    return llp.transitive_closure(s.n, s.ptr, s.dst, ws=s.ws)


def _prepare_reduce(case, seed):
    x = torch.randint(-(2**63), 2**63 - 1, (case["n"],), generator=_gen(seed), device=DEV)
    return SimpleNamespace(x=x, ws=llp.workspace(llp.KIND_REDUCE, case["n"], 0))


def _run_reduce(s):
    v = llp.reduce_sum(s.x, ws=s.ws)
    return v - 2**64 if v >= 2**63 else v   # the same 64 bits, as a signed number


def _prepare_batch(case, seed):
    """Knapsacks (16-256 items, W 256-4096) and graphs (256-4096 vertices, 8 uniform
    arcs per vertex and a cycle), shuffled.  The sizes and the order are the
    case's, the contents the seed's."""
    shape = np.random.default_rng([case["knapsacks"], case["graphs"]])
    rng = np.random.default_rng(seed)
    items = []
    for _ in range(case["knapsacks"]):
        k, W = int(shape.integers(16, 257)), int(shape.integers(256, 4097))
        items.append(("knapsack", rng.integers(1, W // 4 + 1, k, np.int32), rng.integers(1, 1001, k, np.int32), W))
    ns = shape.integers(256, 4097, case["graphs"])
    # the arcs of all graphs at once, on the GPU, ordered by tail
    g = _gen(seed)
    n = torch.from_numpy(ns).to(DEV)
    first = torch.cumsum(n, 0) - n
    own = torch.repeat_interleave(torch.arange(ns.size, device=DEV), 8 * n)
    src = (torch.rand(own.numel(), generator=g, device=DEV, dtype=torch.float64) * n[own]).long()
    step = 1 + (torch.rand(own.numel(), generator=g, device=DEV, dtype=torch.float64) * (n[own] - 1)).long()
    dst = (src + step) % n[own]
    all_n = int(ns.sum())
    vown = torch.repeat_interleave(torch.arange(ns.size, device=DEV), n)
    v = torch.arange(all_n, device=DEV) - first[vown]
    tail = torch.cat([first[own] + src, first[vown] + v])
    order = torch.sort(tail, stable=True).indices
    src = torch.cat([src, v])[order].int().cpu().numpy()
    dst = torch.cat([dst, (v + 1) % n[vown]])[order].int().cpu().numpy()
    w = _ints(g, src.size, 1, 100).cpu().numpy()
    at = 0
    for k in ns:
        e = at + 9 * int(k)
        items.append(("sssp", SimpleNamespace(n=int(k), src=src[at:e], dst=dst[at:e], w=w[at:e]), 0))
        at = e
    return llp.Batch([items[i] for i in shape.permutation(len(items))])


def _run_batch(b):
    b.solve(graph=True)
    return b.out, b.status


def _mlp_inputs(case, seed):
    g, B = _gen(seed), case["rows"]
    p = torch.zeros(llp.MLP_PARAMS, device=DEV)
    at = 0
    for size, fan in ((64 * 12, 12), (64, 0), (64 * 64, 64), (64, 0), (5 * 64, 64), (5, 0)):
        if fan:
            p[at:at + size] = torch.randn(size, generator=g, device=DEV) * math.sqrt(2.0 / fan)
        at += size
    x = torch.rand(B, llp.MLP_IN, generator=g, device=DEV)
    y = _ints(g, B, 0, 2) | (_ints(g, B, 0, 2) << 8)
    m1 = torch.randn(llp.MLP_PARAMS, generator=g, device=DEV) * 1e-3
    m2 = torch.rand(llp.MLP_PARAMS, generator=g, device=DEV) * 1e-4 + 1e-6
    return p, x, y, m1, m2


LR, STEP = 3e-4, 100   # the training run's rate; a step well after the moments' start


def _prepare_mlp(case, seed):
    p, x, y, m1, m2 = _mlp_inputs(case, seed)
    return SimpleNamespace(p=p, x=x, y=y, m1=m1, m2=m2, grad=torch.empty_like(p), step=STEP)


def _run_mlp(s):
    logits, act = llp.mlp_forward(s.p, s.x)
    loss, dl = llp.mlp_loss(logits, s.y)
    s.grad.zero_()
    llp.mlp_backward(s.p, s.x, act, dl, s.grad)
    llp.mlp_adam(s.grad, s.p, s.m1, s.m2, s.step, LR)
    s.step += 1
    return {"logits": logits, "loss": loss, "dlogits": dl, "grad": s.grad, "p": s.p, "m1": s.m1, "m2": s.m2}


_KINDS = {"sssp": (_prepare_graph, _run_graph), "bfs": (_prepare_graph, _run_graph), "sm": (_prepare_sm, _run_sm),
          "jobs": (_prepare_jobs, _run_jobs), "knapsack": (_prepare_knapsack, _run_knapsack),
          "tc": (_prepare_tc, _run_tc), "reduce": (_prepare_reduce, _run_reduce),
          "batch": (_prepare_batch, _run_batch), "mlp": (_prepare_mlp, _run_mlp)}


def prepare(case, seed):
    make, run_it = _KINDS[case["kind"]]
    return SimpleNamespace(state=make(case, seed), run=run_it)


def run(state):
    return state.run(state.state)


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    k = case["kind"]
    if k in ("sssp", "bfs"):
        if case["graph"] == "uniform":
            n, m = case["n"], 9 * case["n"]
        elif case["graph"] == "rmat":
            n, m = 1 << case["scale"], 17 << case["scale"]
        else:
            r, c = case["rows"], case["cols"]
            n, m = r * c, 4 * r * c - 2 * (r + c)
        # each arc's head (and weight) and the row offsets once, the output once
        return {"bytes": 4 * (n + 1) + 4 * n + (8 if k == "sssp" else 4) * m, "flops": 0}
    if k == "sm":
        # the proposals made, about n ln n: a list entry and a rank each; the outputs
        n = case["n"]
        return {"bytes": 4 * n * max(math.log(n), 1.0) + 8 * n, "flops": 0}
    if k == "jobs":
        n = case["n"]
        return {"bytes": 4 * 8 * n + 4 * 2 * (n + 1) + 4 * n + 4 * n, "flops": 8 * n}
    if k == "knapsack":
        return {"bytes": 8 * case["items"] + 4 * (case["W"] + 2), "flops": 2 * case["items"] * (case["W"] + 1)}
    if k == "tc":
        n, m = case["n"], case["m"]
        return {"bytes": 4 * (n + 1 + m) + 4 * n * ((n + 31) // 32), "flops": 0}
    if k == "reduce":
        return {"bytes": 8 * case["n"] + 8, "flops": case["n"]}
    if k == "batch":
        # means of the drawn sizes: 136 items, W 2176; 2176 vertices
        kn, gr = case["knapsacks"], case["graphs"]
        return {"bytes": kn * (8 * 136 + 4) + gr * (4 * 2177 + 8 * 9 * 2176 + 4 * 2176) + 44 * (kn + gr),
                "flops": 2 * kn * 136 * 2177 + 2 * gr * 9 * 2176}
    B = case["rows"]
    mac = 64 * 12 + 64 * 64 + 5 * 64
    return {"bytes": B * (48 + 4 + 20 + 20) + 4 * llp.MLP_PARAMS * 7,
            "flops": 2 * B * (2 * mac + 64 * 64 + 5 * 64)}


# ---------------------------------------------------------------- 64-bit values
def exact(case, seed):
    """The training step in float64 (its bf16 roundings kept: they are the
    network's definition).  Every other output is a whole number."""
    if case["kind"] != "mlp":
        return None
    p, x, y, m1, m2 = (t.cpu() for t in _mlp_inputs(case, seed))

    def bf(t):
        return t.float().bfloat16().double()

    W1, b1, W2, b2, W3, b3 = torch.split(p, [768, 64, 4096, 64, 320, 5])
    W1, W2, W3 = bf(W1).view(64, 12), bf(W2).view(64, 64), bf(W3).view(5, 64)
    X, B = bf(x), x.shape[0]
    h1 = bf(torch.relu(X @ W1.T + bf(b1)))
    h2 = bf(torch.relu(h1 @ W2.T + bf(b2)))
    o = h2 @ W3.T + bf(b3)
    mode, dc = y.long() & 3, ((y.long() >> 8) & 3).clamp(max=2)
    t = torch.stack([mode == 2, mode == 1], 1).double()
    ls = torch.log_softmax(o[:, 2:], 1)
    loss = (torch.nn.functional.softplus(o[:, :2]) - o[:, :2] * t).sum() - ls.gather(1, dc[:, None]).sum()
    d = torch.cat([torch.sigmoid(o[:, :2]) - t, ls.exp() - torch.nn.functional.one_hot(dc, 3)], 1) / B
    d2 = (d @ W3) * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    grad = torch.cat([(d1.T @ X).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), (d.T @ h2).reshape(-1),
                      d.sum(0)])
    m1 = 0.9 * m1.double() + 0.1 * grad
    m2 = 0.999 * m2.double() + 0.001 * grad * grad
    p = p.double() - LR * (m1 / (1 - 0.9 ** STEP)) / ((m2 / (1 - 0.999 ** STEP)).sqrt() + 1e-8)
    return {"logits": o, "loss": (loss / B).view(1), "dlogits": d, "grad": grad, "p": p, "m1": m1, "m2": m2}

"""Timed cases of the evaluation path: the calls a user makes, over the sizes they are made at.

A case names a training graph, a candidate count and a call. Graphs and
fractional matrices S* come from the package's seeded generators (the shapes
and distributions of its standard workloads). Every output is an integer and
is compared exactly.

  round      ckm_round_eval_async: thresholds, randomized rounding, repair,
             simulation, argmin and the best rows, everything on the device
  sync       ckm_round_eval: the same from host arrays to host arrays
  schedules  ckm_eval_schedules_async: K given checkpoint matrices
  threshold  ckm_threshold_eval_async: one candidate per threshold
  batch      quantize, evaluate and ckm_max_batch_async: largest batch
  plan       ckm_plan_async: the execution plan of one schedule

`size` counts a graph's layers, blocks, ops per level or forward nodes;
`pct` is the memory budget in percent of the checkpoint-all memory.
"""
import math

import numpy as np
import torch

from paper_1910_02653_amd import ckm
from paper_1910_02653_amd import workloads as wl


def listed():
    return [
        # a short chain: a call of a few launches, where their latency counts
        dict(name="chain n=17 K=64", call="round", graph="chain", size=8, K=64, det0=False, pct=80.0),
        # a residual network, a size that a search asks for again and again
        dict(name="resnet n=129 K=256", call="round", graph="resnet", size=32, K=256, det0=False, pct=40.0),
        # long skips, candidate 0 rounded deterministically, an odd count
        dict(name="unet n=337 K=501 det0", call="round", graph="unet", size=8, K=501, det0=True, pct=75.0),
        # the named benchmark: a 24-block transformer at its own budget
        dict(name="transformer n=1009 K=1024", call="round", graph="transformer", size=24, K=1024, det0=False, pct=25.0),
        # the deepest graph and the largest call
        dict(name="random n=4001 K=4096", call="round", graph="random", size=2000, K=4096, det0=False, pct=70.0),
        # many samples of a middling graph, the last group of candidates ragged
        dict(name="random n=747 K=3000", call="round", graph="random", size=373, K=3000, det0=False, pct=70.0),
        # a program without device arrays: S* from host memory, results back
        dict(name="sync transformer n=505 K=300", call="sync", graph="transformer", size=12, K=300, det0=False, pct=75.0),
        # schedules from another source (heuristics, a solver's pool), judged
        dict(name="schedules n=1009 K=512", call="schedules", graph="transformer", size=24, K=512, det0=False, pct=60.0),
        # a sweep of the deterministic rounding's threshold
        dict(name="threshold n=1009 K=200", call="threshold", graph="transformer", size=24, K=200, det0=False, pct=75.0),
        # the largest-batch experiment
        dict(name="batch unet n=337 K=1024", call="batch", graph="unet", size=8, K=1024, det0=False, pct=3000.0),
        # the chosen schedule's program
        dict(name="plan n=1009", call="plan", graph="transformer", size=24, K=1, det0=False, pct=100.0),
    ]


NODES = {"chain": lambda s: 2 * s + 1, "resnet": lambda s: 4 * s + 1, "unet": lambda s: 40 * s + 17,
         "transformer": lambda s: 42 * s + 1, "random": lambda s: 2 * s + 1}
SIZES = {"chain": (8, 500), "resnet": (4, 300), "unet": (1, 30), "transformer": (1, 30), "random": (10, 2000)}
VISITS = 4001 * 4001 * 4096   # no drawn case does more node visits than the largest listed one


def draw(rng):
    call = rng.choice(["round"] * 4 + ["sync", "schedules", "threshold", "batch", "plan"])
    graph = rng.choice(sorted(SIZES))
    lo, hi = SIZES[graph]
    size = _log(rng, lo, hi)
    n = NODES[graph](size)
    most = min(4096, VISITS // (n * n))
    if call == "schedules":
        most = min(most, (256 << 20) // (n * ((n + 63) // 64) * 8))   # K whole matrices in device memory
    K = 1 if call == "plan" else _log(rng, 1, max(1, most))
    return dict(call=call, graph=graph, size=size, K=K, det0=call in ("round", "sync") and rng.random() < 0.3,
                pct=3000.0 if call == "batch" else float(rng.randint(20, 95)))


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _workload(case, seed):
    kw = dict(seed=seed % 1000003, K=case["K"], pct=case["pct"])
    size, graph = case["size"], case["graph"]
    if graph == "chain":
        return wl.linear_chain(layers=size, **kw)
    if graph == "resnet":
        return wl.resnet_like(blocks=size, **kw)
    if graph == "unet":
        return wl.unet_like(ops_per_level=size, **kw)
    if graph == "transformer":
        return wl.transformer_stack(blocks=size, **kw)
    return wl.random_dag_stress(F=size, **kw)


def _schedules(n, K, seed):
    """K checkpoint matrices as bit rows: each value is kept with probability
    0.3, from its first stage to a uniformly drawn last one."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = (n + 63) // 64
    i = torch.arange(64 * W, device="cuda")
    t = torch.arange(n, device="cuda")[:, None]
    one = torch.ones(64, dtype=torch.int64, device="cuda") << torch.arange(64, device="cuda")
    out = torch.empty((K, n, W), dtype=torch.int64, device="cuda")
    for k in range(K):
        keep = torch.rand(64 * W, generator=gen, device="cuda") < 0.3
        end = i + 1 + (torch.rand(64 * W, generator=gen, device="cuda") * (n - i).clamp(min=0)).long()
        bits = keep & (i < n) & (t > i) & (t < end)
        out[k] = (bits.view(n, W, 64) * one).sum(2)
    return out


def prepare(case, seed):
    w = _workload(case, seed)
    g = ckm.Graph.from_workload(w)
    call, K = case["call"], case["K"]
    st = dict(call=call, g=g, w=w, K=K, flags=ckm.F_DET0 if case["det0"] else 0)
    if call == "sync":
        return st
    st["work"] = g.alloc_work(K)
    if call in ("round", "threshold", "batch"):
        st["s"] = torch.from_numpy(w.s_frac).cuda()
    if call in ("round", "threshold", "schedules"):
        st["out"] = g.alloc_outputs(K)
    if call == "threshold":
        p = np.random.default_rng(seed).random(K)   # any order
        st["p"] = torch.from_numpy(p).cuda()
    if call in ("schedules", "plan"):
        st["S"] = _schedules(w.n, K, seed)
    if call == "batch":
        st["cap"] = int(w.cost.sum()) * w.n // 3
        st["out"] = dict(batch=torch.empty(K, dtype=torch.int64, device="cuda"),
                         best_k=torch.empty(1, dtype=torch.int32, device="cuda"),
                         best_batch=torch.empty(1, dtype=torch.int64, device="cuda"),
                         status=torch.empty(1, dtype=torch.int32, device="cuda"))
    if call == "plan":
        # the schedule and its recomputations, from the evaluation before it
        out = g.alloc_outputs(1)
        g.eval_schedules_async(st["S"], 1, 1 << 62, out, st["work"])
        st["R"] = out["best_R"]
        st["most"] = most = w.n * (w.n + 1)   # statements any plan can have
        st["out"] = dict(P=torch.zeros((most, 4), dtype=torch.int32, device="cuda"),
                         mem=torch.zeros(most, dtype=torch.int64, device="cuda"),
                         count=torch.zeros(1, dtype=torch.int64, device="cuda"),
                         status=torch.zeros(1, dtype=torch.int32, device="cuda"))
    return st


def run(st):
    g, w, call, K = st["g"], st["w"], st["call"], st["K"]
    if call == "sync":
        r = g.round_eval(w.s_frac, K, w.seed, w.budget, st["flags"])
        return dict(r, best_S=r["best_S"].view(np.int64), best_R=r["best_R"].view(np.int64))
    out, work = st["out"], st["work"]
    if call == "round":
        g.round_eval_async(st["s"], K, w.seed, w.budget, st["flags"], out, work)
    elif call == "threshold":
        g.threshold_eval_async(st["s"], st["p"], w.budget, out, work)
    elif call == "schedules":
        g.eval_schedules_async(st["S"], K, w.budget, out, work)
        return {k: out[k] for k in out if k != "best_S"}   # the matrices are the caller's: no S rows come back
    elif call == "batch":
        g.quantize_async(st["s"], work)
        g.evaluate_async(K, w.seed, 0, work)
        g.max_batch_async(K, w.budget, st["cap"], out["batch"], out["best_k"], out["best_batch"], out["status"], work)
    else:
        g.plan_async(st["S"][0], st["R"], False, out["P"], st["most"], out["count"], out["mem"], out["status"], work)
    return out


def work(case):
    """Each input and output once; per candidate, stage and node at or below
    the stage: a rounding decision, a memory update, its maximum and a cost
    update (the plan: a memory update per statement, about two per node)."""
    n, K, call = NODES[case["graph"]](case["size"]), case["K"], case["call"]
    tri, rows = n * (n + 1) // 2, n * ((n + 63) // 64) * 8
    graph = 40 * n
    if call == "plan":
        return dict(bytes=graph + 2 * rows + 24 * 2 * tri * 3 // 10, flops=2 * tri)
    s = K * rows // 2 if call == "schedules" else 8 * tri
    out = 8 * K if call == "batch" else 17 * K + (rows if call == "schedules" else 2 * rows)
    return dict(bytes=graph + s + out, flops=4 * K * tri)


def tolerance(case):
    return "exact"


def exact(case, seed):
    """Peak, cost, feasibility and the argmin of the rounding calls on small
    graphs, by the definitions, for all candidates at once in int64."""
    n, K = NODES[case["graph"]](case["size"]), case["K"]
    if case["call"] not in ("round", "sync") or n > 140 or n * n * K > 1 << 23:
        return None
    w = _workload(case, seed)
    S = np.zeros((n + 1, n, K), bool)
    for t in range(n):
        for b in range((t + 7) // 8):
            u = _philox(b, t, np.arange(K, dtype=np.uint64), w.seed)
            for j in range(min(8, t - 8 * b)):
                i = 8 * b + j
                S[t, i] = u[j] < int(math.floor(min(max(w.s_frac[t, i], 0.0), 1.0) * 65536.0))
                if case["det0"]:
                    S[t, i, 0] = w.s_frac[t, i] > 0.5
    users = [[] for _ in range(n)]
    for j in range(n):
        for i in w.deps(j):
            users[int(i)].append(j)
    peak, cost = np.zeros(K, np.int64), np.zeros(K, np.int64)
    for t in range(n):
        R = np.zeros((n, K), bool)
        R[t] = True
        for v in range(t - 1, -1, -1):
            need = S[t + 1, v].copy()
            for u in users[v]:
                need |= R[u]
            R[v] = need & ~S[t, v]
        cost += (R * w.cost[:, None]).sum(0)
        mem = w.m_input + 2 * w.m_param + (S[t] * w.size[:, None]).sum(0)
        for v in range(t + 1):
            mem = mem + R[v] * w.size[v]
            peak = np.maximum(peak, mem)
            for i in list(w.deps(v)) + [v]:
                free = R[v] & ~S[t + 1, i]
                for u in users[int(i)]:
                    if u > v:
                        free = free & ~R[u]
                mem = mem - free * w.size[i]
    feasible = peak <= w.budget
    best = min(((int(cost[k]), int(peak[k]), k) for k in range(K) if feasible[k]), default=(0, 0, -1))[2]
    return dict(peak=peak, cost=cost, feasible=feasible.astype(np.uint8), best_k=best, best_S=None, best_R=None,
                status=None)


def _philox(block, stage, k, seed):
    """Eight 16-bit draws per candidate: Philox4x32-10 of (block, stage, k, 0)."""
    mask = np.uint64(0xFFFFFFFF)
    c = [np.full_like(k, block), np.full_like(k, stage), k, np.zeros_like(k)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & mask, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return [(c[j // 2] >> np.uint64(16 * (j % 2))) & np.uint64(0xFFFF) for j in range(8)]

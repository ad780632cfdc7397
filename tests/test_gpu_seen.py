"""Parity with the oracle on graphs with many relations between far nodes: a
node with 120 users more than 32 nodes above it, a dependency with dozens of
far later users, a node with 60 dependencies, and graphs up to the largest
size whose every node has a far user. None of them fits the node data of the
mask path, so they take the tile path, the first ones with hub words. Small
graphs are compared over every candidate; large ones on sampled candidates,
the argmin and the best rows.
"""
import numpy as np
import pytest

from paper_1910_02653_amd import workloads as wl
from test_gpu_parity import check_full, check_rows, gpu_round_eval, lexi_best, log, oracle_candidates
import test_gpu_schedules as sched
import test_gpu_threshold as thr

pytestmark = pytest.mark.gpu


def workload(name, deps, seed, K, m_in=5, m_param=3):
    n = len(deps)
    ptr, idx = wl.csr_from_deps([sorted(d) for d in deps])
    rng = np.random.default_rng(seed)
    size = rng.integers(1, 1000, n).astype(np.int64)
    cost = rng.integers(1, 1000, n).astype(np.int64)
    return wl.Workload(name, n, ptr, idx, cost, size, m_in, m_param, wl.s_frac_uniform(n, seed), K, seed, 1 << 40)


def hub_graph():
    """300 nodes on a chain, plus: node 5 used by 121 nodes from 40 up (far
    users of one node); node 10 used by 251 .. 299, so node 250's slot for it
    sees up to 48 far later users; node 250 with 3 dependencies (slots 2-3)
    and node 290 with 60 (the overflow list)."""
    n = 300
    deps = [set() if v == 0 else {v - 1} for v in range(n)]
    for u in range(40, 281, 2):
        deps[u].add(5)
    deps[250] |= {10, 11}
    for u in range(251, 300):
        deps[u].add(10)
    deps[290] |= set(range(0, 240, 4))
    return workload("hub", deps, seed=300, K=70)


def test_hub_graph_all_candidates():
    w = hub_graph()
    log("far users: hub graph n=%d K=%d" % (w.n, w.K))
    peak, _ = check_full(w, gpu_round_eval(w))
    med = int(np.median(peak))
    check_full(w, gpu_round_eval(w, budget=med), budget=med)


def test_fan_in_fan_out_all_candidates():
    """A random DAG with up to 12 dependencies per node and users anywhere above."""
    w = wl.random_dag(200, seed=17, K=96, max_deg=12, window=200, max_size=1000, max_cost=1000,
                      s_kind="uniform", budget_pct=60.0)
    log("far users: fan-in/out n=%d K=%d" % (w.n, w.K))
    peak, _ = check_full(w, gpu_round_eval(w))
    med = int(np.median(peak))
    check_full(w, gpu_round_eval(w, budget=med), budget=med)


def sampled(w, ks=(0, 1, 33, 63, 64, 69)):
    got = gpu_round_eval(w)
    orc = oracle_candidates(w, list(ks))
    for k in ks:
        assert (int(got["peak"][k]), int(got["cost"][k])) == orc[k], k
    budget = int(np.median(got["peak"]))
    got2 = gpu_round_eval(w, budget=budget)
    assert np.array_equal(got2["peak"], got["peak"]) and np.array_equal(got2["cost"], got["cost"])
    bk = lexi_best(got2["peak"], got2["cost"], budget)
    assert got2["best_k"] == bk >= 0
    assert (int(got2["peak"][bk]), int(got2["cost"][bk])) == oracle_candidates(w, [bk])[bk]
    check_rows(w, got2, bk)


def test_mirrored_training_graph():
    """A random forward DAG of 750 ops (1-3 predecessors within 16) with its
    mirrored backward pass: n = 1501, every forward op far-used by its
    gradient."""
    rng = np.random.default_rng(1501)
    F = 750
    fwd = [[]] + [sorted(set(rng.integers(max(0, v - 16), v, rng.integers(1, 4)).tolist())) for v in range(1, F)]
    deps, size, cost, _ = wl.mirror_training_graph(fwd, rng.integers(1, 1 << 20, F), rng.integers(1, 5000, F), 4, 7)
    ptr, idx = wl.csr_from_deps(deps)
    n = len(deps)
    w = wl.Workload("mirror1501", n, ptr, idx, np.asarray(cost, np.int64), np.asarray(size, np.int64), 1 << 20,
                    1 << 19, wl.s_frac_uniform(n, 5), 70, 5, 1 << 40)
    log("far users: mirrored n=%d" % n)
    sampled(w)


def test_far_users_of_the_largest_graph():
    """n = 4096, every node used 40 nodes above it."""
    n = 4096
    deps = [set() if v == 0 else {v - 1} for v in range(n)]
    for v in range(40, n):
        deps[v].add(v - 40)
    w = workload("skip40", deps, seed=4096, K=70)
    log("far users: n=%d" % n)
    sampled(w, ks=(0, 63, 69))


def far_users_graph(K):
    """n = 1400, every node used by the next and by the node 40 above it."""
    n = 1400
    deps = [set() if v == 0 else {v - 1} for v in range(n)]
    for v in range(40, n):
        deps[v].add(v - 40)
    return workload("skip40_1400", deps, seed=1400, K=K)


def test_far_users_rounding_all_candidates():
    """K = 520 (9 groups, the last ragged): every candidate at two budgets."""
    w = far_users_graph(520)
    log("far users: rounding n=%d K=%d" % (w.n, w.K))
    peak, _ = check_full(w, gpu_round_eval(w))
    med = int(np.median(peak))
    check_full(w, gpu_round_eval(w, budget=med), budget=med)


def test_far_users_thresholds_all_candidates():
    w = far_users_graph(520)
    p = thr.grid(520, 9)
    log("far users: thresholds n=%d K=520" % w.n)
    peak, _ = thr.check(w, p, thr.gpu_eval(w, p, w.budget), w.budget)
    med = int(np.median(peak))
    thr.check(w, p, thr.gpu_eval(w, p, med), med)


def test_far_users_schedules_all_candidates():
    w = far_users_graph(520)
    rows = wl.random_schedules(w.n, 520, seed=520, density=0.3, kind="intervals")
    log("far users: supplied schedules n=%d K=520" % w.n)
    peak, _ = sched.check(w, rows, sched.gpu_eval(w, rows, w.budget), w.budget)
    med = int(np.median(peak))
    sched.check(w, rows, sched.gpu_eval(w, rows, med), med)

"""The tile path (32 stages to a word, a candidate to a lane) where it can go
wrong: sizes around the tile and block edges, every count of near users, far
users and dependencies its tables treat apart, hub words, and both sides of
each launch rule. Every result is an integer and compared for equality, with
the oracle and with the per-lane scan, which a work buffer without the row
arrays takes.
"""
import numpy as np
import pytest
import torch

from paper_1910_02653_amd import ckm
from paper_1910_02653_amd import workloads as wl
from test_gpu_parity import check_full, gpu_round_eval, log, oracle_candidates

pytestmark = pytest.mark.gpu


def graph(n, offsets, seed, K, hubs=()):
    """Node v uses v - o for every o of offsets, and `hubs` = (node, first user, step)."""
    deps = [{v - o for o in offsets if o <= v} for v in range(n)]
    for node, first, step in hubs:
        for u in range(max(first, node + 1), n, step):
            deps[u].add(node)
    ptr, idx = wl.csr_from_deps([sorted(d) for d in deps])
    rng = np.random.default_rng(seed)
    return wl.Workload("tiles", n, ptr, idx, rng.integers(1, 1000, n).astype(np.int64),
                       rng.integers(1, 1000, n).astype(np.int64), 5, 3, 0.6 * wl.s_frac_uniform(n, seed), K, seed, 1 << 40)


def both_paths(w, flags=0, budget=None):
    """ckm_round_eval_async with the row arrays and without them: equal results."""
    g = ckm.Graph.from_workload(w)
    budget = w.budget if budget is None else budget
    s = torch.from_numpy(w.s_frac).cuda()
    res = []
    for rows in (True, False):
        out = g.alloc_outputs(w.K)
        g.round_eval_async(s, w.K, w.seed, budget, flags, out, g.alloc_work(w.K, rows=rows))
        torch.cuda.synchronize()
        res.append({k: v.cpu() for k, v in out.items()})
    g.close()
    for k in res[0]:
        assert torch.equal(res[0][k], res[1][k]), k
    return res[0]


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 129])
def test_sizes(n):
    w = graph(n, (1, 33), n, 65)
    log("tiles: n=%d" % n)
    peak, _ = check_full(w, gpu_round_eval(w, flags=ckm.F_DET0), flags=ckm.F_DET0)
    both_paths(w, budget=int(np.median(peak)))


@pytest.mark.parametrize("offsets", [
    (), (1, 2, 3), (4, 9), (4, 9, 31), (5, 8, 30, 31), (4, 5, 6, 7, 31), (4, 5, 6, 7, 8, 30), (64, 65), (64, 65, 96),
    (64, 65, 66, 67, 68, 69, 70, 71, 72, 73, 74, 75), (1, 40, 63, 64, 100)], ids=str)
def test_users_and_dependencies(offsets):
    """2 to 6 near users, 2 to 12 far ones (the fifth and the third open lists), 0 to 12 dependencies."""
    w = graph(170, offsets, 7 + len(offsets), 64)
    log("tiles: users at %s" % (offsets,))
    peak, _ = check_full(w, gpu_round_eval(w))
    both_paths(w, budget=int(np.median(peak)))


@pytest.mark.parametrize("hubs", [[(0, 120, 10)], [(0, 110, 10)], [(3, 4, 1)], [(0, 1, 2), (40, 41, 3), (100, 130, 5)]],
                         ids=["5 users", "6 users", "all above", "three hubs"])
def test_hubs(hubs):
    w = graph(170, (1, 2) if len(hubs) > 1 else (), 11, 70, hubs=hubs)
    log("tiles: hubs %s" % (hubs,))
    peak, _ = check_full(w, gpu_round_eval(w))
    both_paths(w, budget=int(np.median(peak)))


@pytest.mark.parametrize("K", [6528, 6529, 8128, 8129, 16320, 16321])
def test_launch_rules(K):
    """n = 97 (4 tiles, 10 rounding items): 102 and 103 groups are either side
    of the byte rounding, 127 and 128 of eight stages a wave, 255 and 256 of
    eight parts a tile."""
    w = graph(97, (1, 3, 40), K, K, hubs=[(2, 50, 4)])
    log("tiles: K=%d" % K)
    got = both_paths(w, flags=ckm.F_DET0)
    ks = [0, 1, 63, 64, K // 2, K - 2, K - 1]
    for k, r in oracle_candidates(w, ks, flags=ckm.F_DET0).items():
        assert (int(got["peak"][k]), int(got["cost"][k])) == r, k


@pytest.mark.parametrize("K", [1, 1025, 8192, 8193])
def test_largest_batch_launches(K):
    """One block up to 8192 candidates, block maxima beyond: the multipliers and
    the best one from the evaluation's peaks and costs."""
    w = graph(33, (1, 3), K, K)
    log("largest batch: K=%d" % K)
    g = ckm.Graph.from_workload(w)
    r = g.round_eval(w.s_frac, K, w.seed, 1 << 40)
    base = w.m_input + 2 * w.m_param
    budget, cap = base + 3 * int(r["peak"].min() - base), int(np.median(r["cost"]))
    B = np.where((r["cost"] <= cap) & (r["peak"] <= budget), (budget - base) // (r["peak"] - base), 0)
    best = min((-int(B[k]), int(r["cost"][k]), int(r["peak"][k]), k) for k in range(K) if B[k])
    got = g.max_batch(w.s_frac, K, w.seed, budget, cap)
    g.close()
    assert np.array_equal(got["batch"], B)
    assert (got["best_k"], got["best_batch"]) == (best[3], -best[0])

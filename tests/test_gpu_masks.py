"""The mask path of small graphs, on either side of the rules that choose it:
every call against the per-lane scan, which a work buffer without the row
arrays takes, and some candidates against the oracle. Every result is an
integer and compared for equality.
"""
import numpy as np
import pytest
import torch

from paper_1910_02653_amd import ckm
from paper_1910_02653_amd import workloads as wl
from test_gpu_parity import log, oracle_candidates
from test_gpu_tiles import graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,offsets", [
    (1, 70, ()), (2, 1, (1,)), (7, 65, (1, 2)), (8, 64, (1, 3)), (33, 130, (1, 2, 3, 32)), (64, 200, (1, 33)),
    # the first size past the small ones, with few candidates and with many
    (112, 300, (1, 2, 5, 40)), (113, 300, (1, 2, 5, 40)), (113, 1151, (1, 40)), (113, 1152, (1, 40)),
    # the largest size, and the first past it
    (224, 1152, (2, 7, 50)), (225, 1152, (2, 7, 50)),
    # K n^2 on either side of 140 Mi: 35,840 candidates of 64 nodes
    (64, 35840, (1, 40)), (64, 35841, (1, 40)),
    # what the path's records do not hold: five dependencies, two far users, two later far users
    (100, 70, (1, 2, 3, 4, 5)), (100, 70, (1, 40, 50)), (100, 70, (33, 66))], ids=str)
def test_rules(n, K, offsets):
    w = graph(n, offsets, n + K, K)
    g = ckm.Graph.from_workload(w)
    s = torch.from_numpy(w.s_frac).cuda()
    p = torch.from_numpy(np.random.default_rng(1).random(K)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(5)
    S = torch.randint(-2 ** 63, 2 ** 63 - 1, (K, n, (n + 63) // 64), generator=gen, device="cuda")   # above the diagonal too
    probe = g.alloc_outputs(K)
    g.round_eval_async(s, K, w.seed, 1 << 60, 0, probe, g.alloc_work(K))
    budget = int(probe["peak"].median())
    res = []
    for rows in (True, False):
        log("masks: n=%d K=%d rows=%d" % (n, K, rows))
        work = torch.full((g.workspace_size(K, rows=rows),), 0xA5, dtype=torch.uint8, device="cuda")
        out = [g.alloc_outputs(K) for _ in range(5)]
        g.round_eval_async(s, K, w.seed, budget, ckm.F_DET0, out[0], work)
        g.threshold_eval_async(s, p, budget, out[1], work)
        g.eval_schedules_async(S, K, 1 << 60, out[2], work)
        g.quantize_async(s, work)
        g.round_async(K, w.seed + 1, 0, work)
        g.evaluate_async(K, w.seed + 1, ckm.F_ROUNDED, work)
        g.select_async(K, w.seed + 1, budget, 0, out[3], work)
        g.evaluate_async(K, w.seed, 0, work, stage_splits=min(3, n))
        g.select_async(K, w.seed, budget, 0, out[4], work)
        torch.cuda.synchronize()
        res.append([{k: v.cpu() for k, v in o.items() if not (i == 2 and k == "best_S")} for i, o in enumerate(out)])
    g.close()
    for i, (a, b) in enumerate(zip(*res)):
        for k in a:
            assert torch.equal(a[k], b[k]), (i, k)
    ks = sorted({0, min(1, K - 1), min(63, K - 1), min(64, K - 1), K // 2, K - 1})
    for k, r in oracle_candidates(w, ks, flags=ckm.F_DET0).items():
        assert (int(res[0][0]["peak"][k]), int(res[0][0]["cost"][k])) == r, k

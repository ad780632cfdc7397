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

from oracle import ref
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


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 112, 113])
def test_sizes_two_far_users(n):
    """The same sizes where nodes have two users more than 32 above them, which
    the mask path of small graphs does not take (from 42 nodes on)."""
    w = graph(n, (1, 33, 41), n, 65)
    log("tiles: n=%d, two far users" % n)
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


@pytest.mark.parametrize("K", [2752, 2753, 3776, 3777, 4800, 4801, 6528, 6529, 8128, 8129, 11712, 11713, 16320, 16321])
def test_launch_rules(K):
    """n = 97 (4 tiles, 10 rounding items): 59 and 60 groups are either side
    of the byte rounding, 43 and 44 of eight parts of few tiles, 75 and 76 of
    eight stages a wave, 183 and 184 of eight parts a tile."""
    w = graph(97, (1, 3, 40), K, K, hubs=[(2, 50, 4)])
    log("tiles: K=%d" % K)
    got = both_paths(w, flags=ckm.F_DET0)
    ks = [0, 1, 63, 64, K // 2, K - 2, K - 1]
    for k, r in oracle_candidates(w, ks, flags=ckm.F_DET0).items():
        assert (int(got["peak"][k]), int(got["cost"][k])) == r, k


@pytest.mark.parametrize("K", [1, 1025, 6144, 6145, 8192, 8193])
def test_largest_batch_launches(K):
    """One block up to 6144 candidates, block maxima beyond: the multipliers and
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


def complete(n, K):
    return graph(n, range(1, n), n, K)


def by_definition(w, S):
    """R, peak and cost of a schedule of a graph with many edges, where the
    oracle's scan of all users takes minutes: a value is freed right after the
    last node computed that uses it (or itself), unless the next stage keeps it."""
    n = w.n
    use = np.zeros((n, n), bool)   # [i, u]: u uses i
    for u in range(n):
        use[w.deps(u), u] = True
    S = np.vstack([np.asarray(S, bool)[:, :n], np.zeros((1, n), bool)])
    R, peak, cost = np.zeros((n, n), bool), 0, 0
    for t in range(n):
        r = R[t]
        r[t] = True
        for v in range(t - 1, -1, -1):
            r[v] = (S[t + 1, v] or (use[v] & r).any()) and not S[t, v]
        last = np.where(use & r, np.arange(n), -1).max(1)
        last = np.maximum(last, np.where(r, np.arange(n), -1))
        gone = np.bincount(last[(last >= 0) & ~S[t + 1]], w.size[(last >= 0) & ~S[t + 1]], n).astype(np.int64)
        mem = w.m_input + 2 * w.m_param + int(w.size[S[t]].sum())
        # before a node's own allocation its predecessors' releases are done
        peak = max(peak, int((mem + np.cumsum(w.size * r) - np.concatenate([[0], np.cumsum(gone)[:-1]]))[r].max()))
        cost += int(w.cost[r].sum())
    return R, peak, cost


def test_dense_graphs():
    """Graphs of many users per node: rounding, thresholds and supplied
    schedules. Hub words four users apart (n = 370) and five apart with the
    users between in lists (n = 740); the reference against the oracle first."""
    for n, K in ((60, 3), (370, 5), (740, 2)):
        w = complete(n, K)
        log("dense: n=%d" % n)
        q = ref.quantize(w.s_frac)
        S = [ref.round_random(q, w.seed, k) for k in range(K)]
        want = [by_definition(w, x) for x in S]
        if n == 60:
            for k in range(K):
                peak, cost, _, R = ref.eval_candidate(w, k, want_rows=True)
                assert (int(peak), int(cost)) == want[k][1:] and np.array_equal(np.asarray(R, bool)[:, :n], want[k][0])
        p = np.linspace(0.1, 0.5, 3)
        T = [ref.round_threshold(w.s_frac, x) for x in p]
        mats = wl.random_schedules(n, K, seed=3, density=0.3, kind="intervals")
        U = np.tril(wl.unpack_schedules(mats, n), -1)
        g = ckm.Graph.from_workload(w)
        top = 1 << 60
        for name, got, mine in (("rounding", g.round_eval(w.s_frac, K, w.seed, top), want),
                                ("thresholds", g.threshold_eval(w.s_frac, p, top), [by_definition(w, x) for x in T]),
                                ("schedules", g.eval_schedules(mats, top), [by_definition(w, x) for x in U])):
            assert [(int(a), int(b)) for a, b in zip(got["peak"], got["cost"])] == [x[1:] for x in mine], (n, name)
            assert np.array_equal(got["best_R"], ref.pack_rows(mine[got["best_k"]][0])), (n, name)
        g.close()


def test_room_for_hub_words():
    """A work buffer asks for a bounded room for hub words, and one with less
    room (down to the largest pair of a group and a tile, and less) gives the
    same results in more launches; so does the area that allocates nothing."""
    w = complete(150, 128)
    g, plain = ckm.Graph.from_workload(w), ckm.Graph.from_workload(graph(150, (1, 40, 64), 1, 1))   # tiles, no hubs
    for K in (1, 128, 4096, 65536):
        assert g.workspace_size(K) <= plain.workspace_size(K) + (1 << 30) + 256
    full = g.workspace_size(w.K)
    room = full - plain.workspace_size(w.K)
    most = 256 * (1 + sum((m - 1) // 4 for m in range(6, w.n)))   # the last tile's
    assert most < 64 * w.num_edges and 2 * most < room < 10 * most
    s = torch.from_numpy(w.s_frac).cuda()
    want = None
    for less in (0, 256, room // 2, room - 2 * most, room - most - 256, room - most, room - most + 256, None):
        log("hub words: room for %s bytes" % (less and room - less))
        out = g.alloc_outputs(w.K)
        if less is None:
            g.round_eval_noalloc(s, w.K, w.seed, w.budget, 0, out)
        else:
            work = torch.full((full - less,), 0xA5, dtype=torch.uint8, device="cuda")
            g.round_eval_async(s, w.K, w.seed, w.budget, 0, out, work)
        torch.cuda.synchronize()
        res = {k: v.cpu() for k, v in out.items()}
        want = want or res
        for k in want:
            assert torch.equal(res[k], want[k]), (less, k)
    got = {k: ckm.rows_to_numpy(v) if k in ("best_S", "best_R") else v.numpy() for k, v in want.items()}
    check_full(w, dict(got, best_k=int(got["best_k"][0])))
    g.close()
    plain.close()


@pytest.mark.parametrize("hubs", [(), [(0, 20, 9), (5, 6, 1)]], ids=["no hubs", "hubs"])
def test_room_for_groups(hubs):
    """A buffer with room for the tiles of fewer groups than the call has: the
    groups are evaluated in passes of at least 512 pairs of a group and a tile
    (five tiles: 103 of the 401 groups), with the same results as in one; with
    less room the per-lane scan."""
    n, K = 129, 400 * 64 + 5
    w = graph(n, (1, 33), 3, K, hubs=hubs)
    g = ckm.Graph.from_workload(w)
    s = torch.from_numpy(w.s_frac).cuda()
    p = torch.from_numpy(np.random.default_rng(1).random(K)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(5)
    S = torch.randint(-2 ** 63, 2 ** 63 - 1, (K, n, 3), generator=gen, device="cuda")   # above the diagonal too
    budget = int(np.median(g.round_eval(w.s_frac, K, w.seed, 1 << 60, ckm.F_DET0)["peak"]))
    low, full = g.workspace_size(K, rows=False), g.workspace_size(K)

    def calls(work):
        out = [g.alloc_outputs(K) for _ in range(4)]
        g.round_eval_async(s, K, w.seed, budget, ckm.F_DET0, out[0], work)
        g.threshold_eval_async(s, p, budget, out[1], work)
        g.eval_schedules_async(S, K, 1 << 60, out[2], work)
        g.quantize_async(s, work)
        g.round_async(K, w.seed + 1, 0, work)
        g.evaluate_async(K, w.seed + 1, ckm.F_ROUNDED, work)
        g.select_async(K, w.seed + 1, budget, 0, out[3], work)
        batch = torch.empty(K, dtype=torch.int64, device="cuda")
        best = torch.empty(1, dtype=torch.int32, device="cuda")
        g.max_batch_async(K, 2 * budget, 1 << 60, batch, best, None, None, work)
        torch.cuda.synchronize()
        return [{k: v.cpu() for k, v in o.items() if not (i == 2 and k == "best_S")} for i, o in enumerate(out)] + [
            {"batch": batch.cpu(), "best": best.cpu()}]

    want = calls(torch.empty(full, dtype=torch.uint8, device="cuda"))
    assert all(int(o["best_k"]) >= 0 for o in want[:4])
    for part in (1.0, 0.99, 0.7, 0.4, 0.28, 0.25, 0.0):
        log("passes: %d of %d bytes" % (part * (full - low), full - low))
        work = torch.full((low + int(part * (full - low)),), 0xA5, dtype=torch.uint8, device="cuda")
        for a, b in zip(want, calls(work)):
            for k in a:
                assert torch.equal(a[k], b[k]), (part, k)
    g.close()

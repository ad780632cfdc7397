"""The tile path's host tables (CPU): a closure and a simulation that read
nothing but the tables give the oracle's R, peak and cost, on graphs with every
count of near users, far users, dependencies and hub words that they treat
apart; and a bound on the hub words of any graph."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT
from oracle import ref
from paper_1910_02653_amd import workloads as wl

CSRC = os.path.join(ROOT, "paper_1910_02653_amd", "csrc")
WRAP = r"""
#include "ckm_tiles.h"
using namespace ckm;
template <typename V> static long put(const V& v, void* out) {
  if (out) __builtin_memcpy(out, v.data(), v.size() * sizeof(v[0]));
  return (long)(v.size() * sizeof(v[0]));
}
extern "C" long tiles(int n, const int64_t* M, const int64_t* C, const int32_t* dp, const int32_t* di,
                      const int32_t* up, const int32_t* ui, long max_words, int which, void* out) {
  TileTables T;
  build_tiles(n, M, C, dp, di, up, ui, T, max_words);
  switch (which) {
    case 0: return put(T.desc, out);
    case 1: return put(T.near_more, out);
    case 2: return put(T.far, out);
    case 3: return put(T.far_more, out);
    case 4: return put(T.ops, out);
    case 5: return put(T.refs, out);
    case 6: return put(T.tile_rec, out);
    case 7: return put(T.hub_ptr, out);
    case 8: return put(T.hub, out);
    case 9: return put(T.hub_at, out);
    default: return T.step;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "wrap.cpp").write_text(WRAP)
    so = str(d / "libtiles.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "wrap.cpp"),
                    os.path.join(CSRC, "ckm_tiles.cpp"), "-o", so], check=True)
    f = ctypes.CDLL(so).tiles
    f.restype = ctypes.c_long
    return f


def tables(f, w, max_words=65535):
    users = [[] for _ in range(w.n)]
    for j in range(w.n):
        for i in w.deps(j):
            users[int(i)].append(j)
    up, ui = wl.csr_from_deps(users)
    arrs = [np.ascontiguousarray(w.size, np.int64), np.ascontiguousarray(w.cost, np.int64)] + [
        np.ascontiguousarray(a, np.int32) for a in (w.dep_ptr, w.dep_idx, up, ui)]
    args = [ctypes.c_int(w.n)] + [a.ctypes.data_as(ctypes.c_void_p) for a in arrs] + [ctypes.c_long(max_words)]

    def get(which, dtype):
        out = np.empty(f(*args, which, None), np.uint8)
        f(*args, which, out.ctypes.data_as(ctypes.c_void_p))
        return out.view(dtype)

    u32, i32 = np.uint32, np.int32
    refs = np.dtype([("v", "u2"), ("s", "u2", 2), ("more", "u2"), ("u", "u2", (2, 4)), ("list", "u4", 2)])
    ops = np.dtype([("M", "f8"), ("Mk", "f8", 2), ("C", "u8")])
    return dict(desc=get(0, u32).reshape(-1, 32), near_more=get(1, u32), far=get(2, u32).reshape(-1, 64),
                far_more=get(3, u32), ops=get(4, ops), refs=get(5, refs), tile_rec=get(6, i32),
                hub_ptr=get(7, i32), hub=get(8, u32).reshape(-1, 2), hub_at=get(9, i32), step=f(*args, 10, None),
                users=arrs[5])


PAIRS = {(3, 2): 0, (3, 1): 1, (3, 0): 2, (2, 1): 3, (2, 0): 4, (1, 0): 5}   # (user, node) of a chunk


def users_of(t, v):
    """Node v's users as the closure finds them: within its chunk, near, far."""
    c, j = divmod(v, 4)
    d, half = t["desc"][c], t["far"][v // 16]
    # a ring slot holds the last node at or above it that was decided: at most two blocks up
    near = list(d[4 * j:4 * j + 4]) + list(t["near_more"][d[17 + 2 * j]:][:d[18 + 2 * j]])
    block = v // 32 * 32
    out = [4 * c + x for x in range(j + 1, 4) if d[16] >> PAIRS[x, j] & 1]
    for o in near:
        slot = int(o) // 256
        if slot < 64:
            out.append(next(u for u in range(block, block + 64) if u % 64 == slot))
    k = v % 16
    far = [half[k], half[16 + k]] + list(t["far_more"][half[32 + k]:][:half[48 + k]])
    return out + [int(o) // 256 - 1 for o in far if o]


def evaluate(t, w, S):
    """R, peak and cost of the bits S by the tables."""
    n = w.n
    peak, cost, R = 0, 0, np.zeros((n, n), bool)
    users = [users_of(t, v) for v in range(n)]
    for s in range(n):
        nxt = S[s + 1] if s + 1 < n else np.zeros(n, bool)
        R[s, s] = True
        for v in range(s - 1, -1, -1):
            R[s, v] = (nxt[v] or any(u < n and R[s, u] for u in users[v])) and not S[s, v]
        end = s // 32 * 32 + 32
        at = lambda u: u < n and u < end and R[s, u]   # a user past the tile's end computes nothing
        words = {0: False}
        for h in range(len(t["hub_ptr"]) - 1):
            acc, hub = False, t["hub"][t["hub_ptr"][h]:t["hub_ptr"][h + 1]]
            assert (np.diff(hub[:, 0].astype(int)) < 0).all()
            for r, x in hub:
                u = int(r) // 256 - 1
                if u < end:
                    acc |= at(u)
                    if x:
                        words[int(x) // 256] = acc
        if len(t["hub_at"]):
            assert sorted(words) == list(range(-np.diff(t["hub_at"])[s // 32]))
        U = top = 0.0
        U0 = float(w.m_input + 2 * w.m_param)
        for r in range(t["tile_rec"][s // 32]):
            f, (M, Mk, C) = t["refs"][r], t["ops"][r]
            v = int(f["v"])
            cost += int(C) * bool(R[s, v])
            U0 += M * S[s, v]
            U += M * R[s, v]
            top = max(top, U)
            for k in range(2):
                u, more = [int(x) for x in f["u"][k]], int(f["more"])
                more >>= k
                above = u[:2] + ([u[2]] if more & 1 else []) + ([u[3]] if more & 64 else [])
                later = any(at(x - 1) for x in above if x)
                if more & 4:
                    assert not more & 64
                    later |= bool(words.get(u[3], False))
                if more & 16:
                    assert not more & 1
                    later |= any(at(int(x)) for x in t["users"][f["list"][k]:f["list"][k] + u[2]])
                i = int(f["s"][k])
                U -= Mk[k] * (R[s, v] and not (nxt[i] or later))
        peak = max(peak, U0 + top)
    return R, int(peak), cost


def graph(n, offsets, hubs):
    deps = [{v - o for o in offsets if o <= v} for v in range(n)]
    for node, step in hubs:
        for u in range(node + step, n, step):
            deps[u].add(node)
    ptr, idx = wl.csr_from_deps([sorted(d) for d in deps])
    rng = np.random.default_rng(n)
    return wl.Workload("tables", n, ptr, idx, rng.integers(1, 1000, n).astype(np.int64),
                       rng.integers(1, 1000, n).astype(np.int64), 5, 3, 0.6 * wl.s_frac_uniform(n, n), 2, n, 1 << 40)


def check(t, w):
    for k in range(2):
        peak, cost, S, R = ref.eval_candidate(w, k, want_rows=True)
        r, p, c = evaluate(t, w, np.asarray(S, bool)[:, :w.n])
        assert np.array_equal(r, np.asarray(R, bool)[:, :w.n])
        assert (p, c) == (int(peak), int(cost))


@pytest.mark.parametrize("n,offsets,hubs", [
    (1, (), ()), (33, (1,), ()), (64, (1, 2, 3), ()), (70, (4, 5, 6, 7, 31), ()), (97, (4, 5, 6, 7, 8, 30, 33), ()),
    (150, (64, 65, 66, 67, 68), ()), (100, (1, 40, 63, 64), ((3, 5),)), (80, (), ((0, 12), (1, 13), (2, 1))),
    (70, range(1, 70), ())], ids=str)
def test_tables(lib, n, offsets, hubs):
    w = graph(n, offsets, hubs)
    check(tables(lib, w), w)


@pytest.mark.parametrize("max_words,step", [(560, 4), (559, 5), (100, 18), (1, 68), (0, 69)])
def test_hub_words_bound(lib, max_words, step):
    """Fewer words, each further from the next, with the users between in
    lists: 560 words is what the complete graph of 70 nodes takes four apart."""
    w = graph(70, range(1, 70), ())
    t = tables(lib, w, max_words)
    assert (t["step"], len(t["hub"]) > 0) == (step, max_words > 0)
    check(t, w)


@pytest.mark.parametrize("users,step", [(7, 1), (8, 2), (12, 2), (13, 3), (21, 3), (22, 4)])
def test_hub_words_per_node(lib, users, step):
    """100 nodes with about this many users each: at most four words per node
    while a smaller step than four allows it."""
    w = graph(100, [3 * k + 1 for k in range(users)], ())
    m = np.bincount(w.dep_idx)
    words = [(((m - 1) // s)[m > 5] - (2 if s == 1 else 0)).sum() for s in (1, 2, 3)]   # step 1 from three users on
    t = tables(lib, w)
    assert t["step"] == step == next((s for s in (1, 2, 3) if words[s - 1] <= 400), 4)
    check(t, w)


@pytest.mark.parametrize("n,step", [(100, 4), (365, 4), (727, 4), (728, 5), (1500, 17)])
def test_hub_words_of_dense_graphs(lib, n, step):
    """Complete graphs: a tile's hub words are at most a quarter of the edges
    and never more than record slots can name."""
    t = tables(lib, graph(n, range(1, n), ()))
    words = -np.diff(t["hub_at"]) - 1
    assert t["step"] == step and (np.diff(words) >= 0).all()
    assert words[-1] == sum((m - 1) // step for m in range(6, n)) <= min(65535, n * (n - 1) // 8)
    assert words[0] < words[-1] // 8 or n < 200   # a tile makes those that cover a node of it
    assert t["refs"]["u"][:, :, 3].max() == words[-1]

// Host tables of the tile path (see ckm_tiles.h).
#include "ckm_tiles.h"

#include <algorithm>

namespace ckm {

void build_tiles(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                 const int32_t* user_ptr, const int32_t* user_idx, TileTables& T, int64_t max_hub_words) {
  T = TileTables();
  T.n = n;
  T.tiles = (n + kTile - 1) / kTile;

  // hub words: word w of a node with m users covers its highest w step, which are
  // three at least (or step) and below m (no dependency has all m above it)
  const auto first_of = [](int32_t step) { return step == 1 ? 3 : 1; };
  const auto words_at = [&](int32_t i, int32_t step) {
    const int32_t m = user_ptr[i + 1] - user_ptr[i];
    return m > kHubUsers ? (m - 1) / step + 1 - first_of(step) : 0;
  };
  for (;; ++T.step) {
    int64_t words = 0;
    for (int32_t i = 0; i < n; ++i) words += words_at(i, T.step);
    if (words <= (T.step < kHubStep ? std::min(max_hub_words, (int64_t)kHubWordsPerNode * n) : max_hub_words)) break;
  }
  const int32_t w0 = first_of(T.step);
  std::vector<int32_t> first_word(n + 1, 0);
  for (int32_t i = 0; i < n; ++i) first_word[i + 1] = first_word[i] + words_at(i, T.step);
  std::vector<int32_t> lowest(first_word[n]), order(first_word[n]), slot_of(first_word[n]);
  for (int32_t i = 0; i < n; ++i)
    for (int32_t w = first_word[i]; w < first_word[i + 1]; ++w)
      lowest[w] = user_idx[user_ptr[i + 1] - T.step * (w - first_word[i] + w0)];
  for (size_t w = 0; w < order.size(); ++w) order[w] = (int32_t)w;
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return lowest[a] < lowest[b]; });
  for (size_t k = 0; k < order.size(); ++k) slot_of[order[k]] = (int32_t)k + 1;
  if (!order.empty()) {
    T.hub_at.assign(T.tiles + 1, 0);
    for (int32_t k = T.tiles - 1, w = (int32_t)order.size(); k >= 0; --k) {
      while (w > 0 && lowest[order[w - 1]] >= kTile * (k + 1)) --w;
      T.hub_at[k] = T.hub_at[k + 1] + 1 + (uint32_t)w;
    }
  }
  T.hub_ptr.push_back(0);
  for (int32_t i = 0; i < n; ++i) {
    if (first_word[i] == first_word[i + 1]) continue;
    const int32_t used = T.step * (first_word[i + 1] - first_word[i] + w0 - 1);   // the users that some word covers
    for (int32_t k = 0; k < used; ++k) {
      const int32_t u = user_idx[user_ptr[i + 1] - 1 - k];
      const int32_t w = (k + 1) / T.step;
      T.hub.push_back({kRBase + node_off(u), (k + 1) % T.step || w < w0 ? 0u : node_off(slot_of[first_word[i] + w - w0])});
    }
    T.hub_ptr.push_back((int32_t)T.hub.size());
    ++T.nhub;
  }

  // the closure's users
  constexpr int kChunks = kTile / kChunk4;   // per block
  T.desc.assign((size_t)T.tiles * kChunks * kDescDwords, 0);
  T.far.assign((size_t)T.tiles * 2 * kFarDwords, 0);
  uint32_t block = 0;                        // flags of the block so far
  for (int32_t c = 0; c < T.tiles * kChunks; ++c) {
    uint32_t* d = T.desc.data() + (size_t)c * kDescDwords;
    uint32_t flags = 0;
    for (int j = 0; j < kChunk4; ++j) {
      const int32_t v = kChunk4 * c + j;
      uint32_t* near = d + 4 * j;
      for (int k = 0; k < 4; ++k) near[k] = kRingEmpty * kSlotBytes;
      if (v >= n) continue;
      uint32_t* far = T.far.data() + (size_t)(v / kFarNodes) * kFarDwords + v % kFarNodes;
      far[32] = (uint32_t)T.far_more.size();
      d[17 + 2 * j] = (uint32_t)T.near_more.size();
      int nn = 0, nf = 0;
      for (int32_t e = user_ptr[v]; e < user_ptr[v + 1]; ++e) {
        const int32_t u = user_idx[e];
        if (u / kChunk4 == c) {
          // pairs (3, 2), (3, 1), (3, 0), (2, 1), (2, 0), (1, 0)
          const int from = u % kChunk4;
          flags |= 1u << (from == 3 ? 2 - j : from == 2 ? 4 - j : 5);
        } else if (u / kTile <= v / kTile + 1) {
          const uint32_t slot = (uint32_t)(u % kRingNodes * kSlotBytes);
          if (nn < 4)
            near[nn] = slot;
          else
            T.near_more.push_back(slot);
          ++nn;
        } else {
          if (nf < 2)
            far[16 * nf] = kRBase + node_off(u);
          else
            T.far_more.push_back(kRBase + node_off(u));
          ++nf;
        }
      }
      far[48] = (uint32_t)T.far_more.size() - far[32];
      d[18 + 2 * j] = (uint32_t)T.near_more.size() - d[17 + 2 * j];
      if (nn > 2) block |= kBlockNear3;
      if (nn > 3) block |= kBlockNear4;
      if (nn > 4) block |= kBlockMany;
    }
    d[16] |= flags;
    if (c % kChunks == kChunks - 1) {
      for (int k = 0; k < kChunks; ++k) d[16 - k * kDescDwords] |= block;
      block = 0;
    }
  }

  // simulation records
  std::vector<int32_t> rec_end(n);
  for (int32_t v = 0; v < n; ++v) {
    const int32_t nd = dep_ptr[v + 1] - dep_ptr[v];
    for (int32_t a = 0; a < std::max(nd, 1); a += 2) {
      SimOps o{};
      SimRefs r{};
      r.v = r.s[0] = r.s[1] = (uint16_t)v;
      if (a == 0) {
        o.M = (double)M[v];
        o.C = (uint64_t)C[v];
      }
      for (int k = 0; k < 2 && a + k < nd; ++k) {
        const int32_t i = dep_idx[dep_ptr[v] + a + k];
        (k ? o.M1 : o.M0) = (double)M[i];
        r.s[k] = (uint16_t)i;
        const int32_t* above = std::upper_bound(user_idx + user_ptr[i], user_idx + user_ptr[i + 1], v);
        const int32_t na = (int32_t)(user_idx + user_ptr[i + 1] - above);
        const bool hub = na > 2 && first_word[i] < first_word[i + 1] && na >= T.step;
        const int32_t left = hub ? na % T.step : na;
        if (hub) {
          r.u[k][3] = (uint16_t)slot_of[first_word[i] + na / T.step - w0];
          r.more |= kMoreHub << k;
        }
        for (int32_t x = 0; x < left && x < 2; ++x) r.u[k][x] = (uint16_t)(above[x] + 1);
        if (left > 2 && T.step > kHubStep) {
          r.list[k] = (uint32_t)(above - user_idx) + 2;
          r.u[k][2] = (uint16_t)(left - 2);
          r.more |= kMoreList << k;
        } else if (left > 2) {
          r.u[k][2] = (uint16_t)(above[2] + 1);
          r.more |= kMoreThird << k;
          if (left > 3) {
            r.u[k][3] = (uint16_t)(above[3] + 1);
            r.more |= kMoreFourth << k;
          }
        }
      }
      T.ops.push_back(o);
      T.refs.push_back(r);
    }
    rec_end[v] = (int32_t)T.ops.size();
  }
  T.nrec = (int32_t)T.ops.size();
  for (int32_t k = 0; k < T.tiles; ++k) T.tile_rec.push_back(rec_end[std::min(kTile * (k + 1), n) - 1]);
  // records are read up to two past a tile's last
  for (int k = 0; k < 2; ++k) {
    T.ops.push_back(SimOps{});
    T.refs.push_back(SimRefs{});
  }
}

}  // namespace ckm

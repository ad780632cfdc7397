// Host tables of the tile path (see ckm_tiles.h).
#include "ckm_tiles.h"

#include <algorithm>

namespace ckm {

bool build_tiles(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                 const int32_t* user_ptr, const int32_t* user_idx, TileTables& T) {
  T = TileTables();
  T.n = n;
  T.tiles = (n + kTile - 1) / kTile;

  // hub words: their places first (they set rbase), then their tables
  uint32_t words = 0;
  std::vector<uint32_t> first_word(n, 0);
  if (n >= kMaxSlots) return false;
  for (int32_t i = 0; i < n; ++i) {
    const int32_t m = user_ptr[i + 1] - user_ptr[i];
    if (m <= kHubUsers) continue;
    first_word[i] = words;
    words += (uint32_t)(m - 3);
    if (1 + (int64_t)words + kTile * (int64_t)T.tiles > kMaxSlots) return false;
  }
  T.rbase = node_off((int32_t)(1 + words));
  const auto word_off = [](uint32_t x) { return node_off((int32_t)(1 + x)); };
  T.hub_ptr.push_back(0);
  for (int32_t i = 0; i < n; ++i) {
    const int32_t m = user_ptr[i + 1] - user_ptr[i];
    if (m <= kHubUsers) continue;
    for (int32_t k = 0; k < m; ++k) {   // k users above
      const int32_t u = user_idx[user_ptr[i + 1] - 1 - k];
      T.hub.push_back({T.rbase + node_off(u), k >= 3 ? word_off(first_word[i] + (uint32_t)(k - 3)) : 0u});
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
            far[16 * nf] = T.rbase + node_off(u);
          else
            T.far_more.push_back(T.rbase + node_off(u));
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
      const auto slot = [](uint32_t off) { return (uint16_t)(off / kSlotBytes); };
      r.v = r.s[0] = r.s[1] = (uint16_t)v;
      if (a == 0) {
        o.M = (double)M[v];
        r.C = (uint64_t)C[v];
      }
      for (int k = 0; k < 2 && a + k < nd; ++k) {
        const int32_t i = dep_idx[dep_ptr[v] + a + k];
        (k ? o.M1 : o.M0) = (double)M[i];
        r.s[k] = (uint16_t)i;
        const int32_t* b = user_idx + user_ptr[i];
        const int32_t* e = user_idx + user_ptr[i + 1];
        const int32_t* above = std::upper_bound(b, e, v);
        const int32_t na = (int32_t)(e - above);
        if (e - b > kHubUsers && na >= 3) {
          r.u[k][0] = slot(word_off(first_word[i] + (uint32_t)(na - 3)));
        } else {
          for (int32_t x = 0; x < na; ++x) r.u[k][x] = slot(T.rbase + node_off(above[x]));   // at most kHubUsers - 1
          if (na > 2) r.more = 1;
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
  return true;
}

}  // namespace ckm

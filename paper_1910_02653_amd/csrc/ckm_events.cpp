// Host tables of the event path (see ckm_events.h).
#include "ckm_events.h"

#include <algorithm>

namespace ckm {

namespace {

uint32_t slot_off(int slot) { return (uint32_t)slot * (uint32_t)kEvSlotBytes; }

}  // namespace

bool build_events(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                  const int32_t* user_ptr, const int32_t* user_idx, uint64_t max_tile_bytes, EventTables& T) {
  T = EventTables();
  T.n = n;
  T.np = (n + 3 + kEvChunk - 1) / kEvChunk * kEvChunk;
  T.chunks = T.np / kEvChunk;
  T.pairs = (n + 1) / 2;
  T.tiles = (2 * T.pairs + 63) / 64;
  const auto chunk = [](int32_t v) { return v / kEvChunk; };
  const auto is_far = [&](int32_t v, int32_t i) { return chunk(v) - chunk(i) > kEvNear; };

  // Pins: the nodes with the most far users that come within a chunk of each
  // other, or seven chunks above the node (its ring entry is loaded then).
  std::vector<int32_t> trouble(n, 0), pin_of(n, -1);
  for (int32_t i = 0; i < n; ++i) {
    for (int32_t e = user_ptr[i]; e < user_ptr[i + 1]; ++e) {
      const int32_t u = user_idx[e];
      if (!is_far(u, i)) continue;
      if (e + 1 < user_ptr[i + 1] && chunk(user_idx[e + 1]) <= chunk(u) + 1) ++trouble[i];
      if (chunk(u) == chunk(i) + kEvNear + 1) ++trouble[i];
    }
  }
  for (int32_t i = 0; i < n; ++i)
    if (trouble[i] > 0) T.pins.push_back(i);
  std::stable_sort(T.pins.begin(), T.pins.end(), [&](int32_t x, int32_t y) { return trouble[x] > trouble[y]; });
  if ((int32_t)T.pins.size() > kEvPins) T.pins.resize(kEvPins);
  for (size_t p = 0; p < T.pins.size(); ++p) pin_of[T.pins[p]] = (int32_t)p;

  // Far slots, and each node's lowest far user.
  std::vector<int32_t> fslot(n, -1), farmin(n, 0xFFFF);
  for (int32_t i = 0; i < n; ++i) {
    if (pin_of[i] >= 0) continue;
    for (int32_t e = user_ptr[i]; e < user_ptr[i + 1]; ++e)
      if (is_far(user_idx[e], i)) {
        farmin[i] = std::min(farmin[i], user_idx[e]);
        if (fslot[i] < 0) fslot[i] = T.nf++;
      }
  }
  // The far user of i next above v (0xFFFF: none).
  const auto far_above = [&](int32_t i, int32_t v) {
    const int32_t* b = user_idx + user_ptr[i];
    const int32_t* e = user_idx + user_ptr[i + 1];
    const int32_t* u = std::upper_bound(b, e, v);
    return u == e ? 0xFFFF : *u;   // a user above a far user is far too
  };

  T.desc.assign((size_t)T.chunks * 64, 0);
  T.main_rec.assign(T.np + 1, 0);
  struct Slots { int32_t d[4] = {-1, -1, -1, -1}; };
  std::vector<Slots> first(n);
  int32_t rec = 0;
  std::vector<int32_t> far, near;
  for (int32_t v = 0; v < T.np; ++v) {
    uint32_t* d = T.desc.data() + (size_t)v * kEvDescDw;
    T.main_rec[v] = rec;
    Slots s;
    far.clear();
    near.clear();
    if (v < n)
      for (int32_t e = dep_ptr[v]; e < dep_ptr[v + 1]; ++e) {
        const int32_t i = dep_idx[e];
        (is_far(v, i) && pin_of[i] < 0 ? far : near).push_back(i);
      }
    // slots 0 and 1 take far dependencies first; 2 and 3 near ones only
    size_t fa = 0, na = 0;
    for (int k = 0; k < 2; ++k) s.d[k] = fa < far.size() ? far[fa++] : na < near.size() ? near[na++] : -1;
    for (int k = 2; k < 4; ++k) s.d[k] = na < near.size() ? near[na++] : -1;
    uint32_t flags = 0, off[4];
    for (int k = 0; k < 4; ++k) {
      const int32_t i = s.d[k];
      if (i < 0) {
        off[k] = slot_off(kEvNone);
      } else if (pin_of[i] >= 0) {
        off[k] = slot_off(kEvPin + pin_of[i]);
      } else if (!is_far(v, i)) {
        off[k] = slot_off(i % kEvRing);
      } else {
        off[k] = slot_off(kEvStage + 2 * (v % 8) + k);   // k < 2
        const int32_t up = far_above(i, v);
        flags |= k ? kEvFar1 : kEvFar0;
        if (up != 0xFFFF && chunk(up) <= chunk(v) + 1) flags |= k ? kEvSync1 : kEvSync0;
        d[2] |= (uint32_t)fslot[i] << (16 * k);
        d[4 + k] = (uint32_t)i | (uint32_t)up << 16;
      }
    }
    d[0] = off[0] | off[1] << 16;
    d[8] = off[2] | off[3] << 16;
    if (s.d[2] >= 0) flags |= kEvSecond;
    const auto op = [&](int32_t a, int32_t b, bool main) {
      T.ops.push_back(main && v < n ? (double)M[v] : 0.0);
      T.ops.push_back(main && v < n ? (double)C[v] : 0.0);
      T.ops.push_back(a >= 0 ? (double)M[a] : 0.0);
      T.ops.push_back(b >= 0 ? (double)M[b] : 0.0);
      ++rec;
    };
    op(s.d[0], s.d[1], true);
    if (flags & kEvSecond) op(s.d[2], s.d[3], false);
    // records beyond the second
    std::vector<int32_t> rest(far.begin() + fa, far.end());
    rest.insert(rest.end(), near.begin() + na, near.end());
    d[3] = (uint32_t)(T.extra.size() / kEvExtraDw);
    uint32_t count = 0;
    for (size_t r = 0; r < rest.size(); r += 2, ++count) {
      uint32_t x[kEvExtraDw] = {0, 0, 0, 0, 0xFFFFFFFFu, 0, 0, 0};
      int32_t pair[2] = {rest[r], r + 1 < rest.size() ? rest[r + 1] : -1};
      uint32_t up16[2] = {0xFFFFu, 0xFFFFu};
      for (int k = 0; k < 2; ++k) {
        const int32_t i = pair[k];
        uint32_t o;
        if (i < 0) {
          o = slot_off(kEvNone);
        } else if (pin_of[i] >= 0) {
          o = slot_off(kEvPin + pin_of[i]);
        } else if (!is_far(v, i)) {
          o = slot_off(i % kEvRing);
        } else {
          o = slot_off(kEvXtra + k);
          x[1] |= k ? kEvFar1 : kEvFar0;
          x[2] |= (uint32_t)fslot[i] << (16 * k);
          x[3] |= (uint32_t)i << (16 * k);
          up16[k] = (uint32_t)far_above(i, v);
        }
        x[0] |= o << (16 * k);
      }
      x[4] = up16[0] | up16[1] << 16;
      T.extra.insert(T.extra.end(), x, x + kEvExtraDw);
      op(pair[0], pair[1], false);
    }
    d[1] = flags | count << 16;
    d[6] = 0xFFFF0000u;
    d[7] = slot_off(v % kEvRing);
    if (v < n) {
      if (pin_of[v] >= 0) d[7] = slot_off(kEvPin + pin_of[v]);
      if (fslot[v] >= 0) {
        d[6] = (uint32_t)fslot[v] | (uint32_t)farmin[v] << 16;
        for (int32_t e = user_ptr[v]; e < user_ptr[v + 1]; ++e)
          if (chunk(user_idx[e]) == chunk(v) + kEvNear + 1) d[1] |= kEvEntrySync;
      }
      first[v] = s;
    }
    if ((uint64_t)rec * kEvRecBytes * 64 > max_tile_bytes) return false;
  }
  T.main_rec[T.np] = rec;
  // node v + 1's first four slots against node v
  for (int32_t v = 0; v + 1 < n; ++v)
    for (int k = 0; k < 4; ++k)
      if (first[v + 1].d[k] == v) T.desc[(size_t)v * kEvDescDw + 1] |= kEvOwnFwd;
  for (int32_t c = 0; c < T.chunks; ++c) {
    uint32_t* d = T.desc.data() + (size_t)c * 64;
    uint32_t fl = 0;
    for (int j = 0; j < kEvChunk; ++j) {
      const uint32_t f = d[j * kEvDescDw + 1];
      if (((f & kEvFar0) && !(f & kEvSync0)) || ((f & kEvFar1) && !(f & kEvSync1))) fl |= kEvChunkFar;
      if (d[j * kEvDescDw + 6] != 0xFFFF0000u) fl |= kEvChunkEntry;
    }
    d[15] = fl;
    d[kEvDescDw + 15] = (uint32_t)T.main_rec[kEvChunk * (c + 1)];
  }
  // padded to a multiple of 4 records
  T.nrec = rec;
  while (T.nrec % 4) {
    T.ops.insert(T.ops.end(), 4, 0.0);
    ++T.nrec;
  }

  // rows of event records
  T.row_off.assign(2 * T.pairs + 1, 0);
  uint64_t at = 0;
  for (int32_t p = 0; p < T.pairs; ++p) {
    const int32_t last = std::min(2 * p + 1, n - 1);
    const uint64_t len = ((uint64_t)T.main_rec[last + 1] + 3) / 4 * 4;
    for (int h = 0; h < 2; ++h) {
      T.row_off[2 * p + h] = (uint32_t)at;
      at += len;
    }
  }
  if (at > UINT32_MAX) return false;
  T.row_off[2 * T.pairs] = (uint32_t)at;

  // the chunk of the node whose record ends the tile's longest row
  T.tile_chunk.assign(T.tiles, 0);
  for (int32_t k = 0; k < T.tiles; ++k) {
    const int32_t p = std::min(32 * k + 31, T.pairs - 1);
    const int32_t len = (int32_t)(T.row_off[2 * p + 1] - T.row_off[2 * p]);
    const int32_t v = (int32_t)(std::upper_bound(T.main_rec.begin(), T.main_rec.end() - 1, len - 1) -
                                T.main_rec.begin()) - 1;
    T.tile_chunk[k] = chunk(v);
  }
  return true;
}

}  // namespace ckm

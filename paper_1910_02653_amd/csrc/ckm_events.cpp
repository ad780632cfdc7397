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
  T.np = (n + kEvChunk - 1) / kEvChunk * kEvChunk;
  T.chunks = T.np / kEvChunk;
  T.tiles = (n + kEvTile - 1) / kEvTile;
  const auto chunk = [](int32_t v) { return v / kEvChunk; };
  const auto is_far = [&](int32_t v, int32_t i) { return chunk(v) - chunk(i) > kEvNear; };
  // A chunk's far accumulators are stored while the next chunk is decided, far
  // loads for chunk c issued then in chunk c + kEvAhead + 1, ring entries
  // loaded kEvAhead chunks before they are written (in the seventh chunk above
  // theirs): both miss the stores of a far user up to there.
  const auto too_close = [&](int32_t up, int32_t v) { return chunk(up) <= chunk(v) + kEvAhead + 1; };
  const auto above_ring = [&](int32_t u, int32_t i) {
    return is_far(u, i) && chunk(u) - chunk(i) <= kEvNear + 1 + kEvAhead;
  };

  // Pins: the nodes with the most such far users.
  std::vector<int32_t> trouble(n, 0), pin_of(n, -1);
  for (int32_t i = 0; i < n; ++i) {
    for (int32_t e = user_ptr[i]; e < user_ptr[i + 1]; ++e) {
      const int32_t u = user_idx[e];
      if (!is_far(u, i)) continue;
      if (e + 1 < user_ptr[i + 1] && too_close(user_idx[e + 1], u)) ++trouble[i];
      if (above_ring(u, i)) ++trouble[i];
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
  const int32_t spare = T.nf++;
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
        if (up != 0xFFFF && too_close(up, v)) flags |= k ? kEvSync1 : kEvSync0;
        d[7] |= (uint32_t)fslot[i] << (16 * k);
        d[4 + k] = (uint32_t)i | (uint32_t)up << 16;
      }
    }
    d[11] = 0;
    d[12] = (uint32_t)spare * (uint32_t)kEvSlotBytes;
    if (flags & kEvFar0) {
      d[11] = (uint32_t)(s.d[0] / 4 * kEvQuadBytes + 4 * (s.d[0] % 4));
      d[12] = (d[7] & 0xFFFFu) * (uint32_t)kEvSlotBytes;
    }
    d[0] = off[0];
    d[2] = off[1];
    d[3] = (uint32_t)rec * (uint32_t)kEvRecBytes;
    d[8] = off[2] | off[3] << 16;
    if (s.d[2] >= 0) flags |= kEvSecond;
    const auto op = [&](int32_t a, int32_t b, bool main) {
      T.ops.push_back({main && v < n ? (double)M[v] : 0.0, main && v < n ? (uint64_t)C[v] : 0u,
                       a >= 0 ? (double)M[a] : 0.0, b >= 0 ? (double)M[b] : 0.0});
      ++rec;
    };
    op(s.d[0], s.d[1], true);
    if (flags & kEvSecond) op(s.d[2], s.d[3], false);
    // records beyond the second
    std::vector<int32_t> rest(far.begin() + fa, far.end());
    rest.insert(rest.end(), near.begin() + na, near.end());
    d[9] = (uint32_t)(T.extra.size() / kEvExtraDw);
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
    if (v < n) {
      if (pin_of[v] >= 0) {
        d[1] |= kEvPinned;
        d[10] = slot_off(kEvPin + pin_of[v]);
      }
      if (fslot[v] >= 0) {
        d[6] = (uint32_t)fslot[v] | (uint32_t)farmin[v] << 16;
        for (int32_t e = user_ptr[v]; e < user_ptr[v + 1]; ++e)
          if (above_ring(user_idx[e], v)) d[1] |= kEvEntrySync;
      }
      first[v] = s;
    }
    if ((uint64_t)rec * kEvRecBytes > max_tile_bytes) return false;
  }
  T.main_rec[T.np] = rec;
  for (int32_t c = 0; c < T.chunks; ++c) {
    uint32_t* d = T.desc.data() + (size_t)c * 64;
    uint32_t fl = 0;
    for (int j = 0; j < kEvChunk; ++j) {
      const uint32_t f = d[j * kEvDescDw + 1];
      if (((f & kEvFar0) && !(f & kEvSync0)) || ((f & kEvFar1) && !(f & kEvSync1))) fl |= kEvChunkFar;
      if (d[j * kEvDescDw + 6] != 0xFFFF0000u) fl |= kEvChunkEntry;
      if (f & kEvSecond) fl |= kEvChunkSecond;
      if (f & kEvEntrySync) fl |= kEvChunkEntrySync;
      if (f & (0xFFFF0000u | kEvSync0 | kEvSync1 | kEvPinned | kEvFar1)) fl |= kEvChunkRare;
      if ((f & kEvFar0) && d[j * kEvDescDw + 4] >> 16 != 0xFFFFu) fl |= kEvChunkRare;
    }
    for (int b = kEvChunkUse, j = 3; j > 0; --j)
      for (int i = j - 1; i >= 0; --i, ++b)
        for (int k = 0; k < 4; ++k)
          if (kEvChunk * c + j < n && first[kEvChunk * c + j].d[k] == kEvChunk * c + i) fl |= 1u << b;
    d[15] = fl;
  }
  T.nrec = rec;
  T.ops.insert(T.ops.end(), 8, EvOps{0.0, 0, 0.0, 0.0});
  for (int32_t k = 0; k < T.tiles; ++k) T.tile_rec.push_back(T.main_rec[kEvChunk * (ev_first_chunk(n, k) + 1)]);
  return true;
}

}  // namespace ckm

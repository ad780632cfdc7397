// Event path (see ckm_events.h): the closure kernel, which decides R and the
// FREE terms of every (candidate, stage, node), the simulate kernel, which
// runs the U recurrence on them, and the gather of the best candidate's R.
//
// Decisions are bits: with 32 stages to a word and a candidate to a lane, one
// instruction decides a node for 32 x 64 (stage, candidate) pairs, and every
// access to memory or LDS is one word (or four) per lane at a wave-uniform
// address. The sums are binary64 per (candidate, stage); a word's bit j, taken
// alone in the low half of a binary64, is 2^(j - 1074), so that one AND and
// one FMA make a masked update of an accumulator that counts in units of
// 2^(j - 1074).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ckm_events.h"
#include "ckm_internal.h"

namespace ckm {
namespace {

template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

constexpr int kBufWord3 = 0x00020000;   // raw byte-addressed buffer: reads past its end give 0

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// ---------------------------------------------------------------------------
// Closure: one wave per (group, tile).
struct ClosureArgs {
  int32_t n, tiles, tlo, thi, g0;   // tiles tlo .. thi - 1 of the groups from g0
  int32_t npins;
  uint32_t far_bytes;               // far accumulators of one wave
  size_t s_bytes;                   // S words of one group
  size_t ev_bytes;                  // event records of one group in the chunk
  const char* stiles;               // S words, group-major
  char* events;                     // event records, group-major from group g0
  char* far;                        // far accumulators, per (group - g0, tile - tlo)
  const uint32_t* desc;             // chunks x 64 dwords
  cptr<uint32_t> extra;
  cptr<uint64_t> tile_off;          // byte offset of each tile's event records in a group
  cptr<int32_t> pins;
  const int32_t* best_k;            // not NULL: only the group of this candidate (none when negative)
};

// A chunk whose records are not stored yet: their release words are on their
// way from LDS, and are taken up while the next chunk is decided.
struct Pending {
  uint32_t R[4], S[4], a0[4], a1[4], a2[4], a3[4];
  uint32_t d;       // its descriptors
  bool live, second, far;
};

struct Quad {
  uint32_t x[4];
};

struct Closure {
  __amdgpu_buffer_rsrc_t rs, rn, re, rf, rd;   // S words of the tile and the next, events, far, descriptors
  uint32_t next;                    // lane offset in the next tile (after the last tile: past every buffer, reads give 0)
  const char* tile;                 // the tile's S words
  const char* far;                  // the wave's far accumulators
  uint32_t tile_bytes, far_bytes;
  lds_char* lds;                    // this lane's column
  uint32_t lane;
  int32_t b0, n, vstart;            // first stage of the tile, nodes, first node of the scan
  uint32_t pre[4], held[4];         // accumulators and S words of the next chunk's nodes

  __device__ __forceinline__ uint32_t at(uint32_t off) const { return *(lds_u32*)(lds + off); }
  __device__ __forceinline__ void put(uint32_t off, uint32_t x) const { *(lds_u32*)(lds + off) = x; }
  __device__ __forceinline__ uint32_t lds_or(uint32_t off, uint32_t x) const {
    return __hip_atomic_fetch_or((lds_u32*)(lds + off), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  __device__ __forceinline__ uint32_t load_desc(int c) const {
    return __builtin_amdgcn_raw_buffer_load_b32(rd, (int)(4u * lane), uniform(c > 0 ? 256 * c : 0), 0);
  }
  // S words of chunk c, of the tile or the next
  __device__ __forceinline__ Quad load_quad(__amdgpu_buffer_rsrc_t r, uint32_t vo, int c) const {
    const auto a = __builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, uniform(c > 0 ? kEvQuadBytes * c : 0), 0);
    return {{a[0], a[1], a[2], a[3]}};
  }
  __device__ __forceinline__ Quad load_own(int c) const { return load_quad(rs, 16u * lane, c); }
  __device__ __forceinline__ Quad load_next(int c) const { return load_quad(rn, next, c); }
  // S_{t+1} of the tile's stages: its own words shifted, the next tile's first stage on top
  __device__ __forceinline__ uint32_t s1_of(uint32_t s, uint32_t next) const {
    return __builtin_amdgcn_alignbit(next, s, 1);
  }
  __device__ __forceinline__ uint32_t load_s1(uint32_t node) const {
    const int so = (int)(kEvQuadBytes * (node >> 2)), at = (int)(4u * (node & 3u));
    return s1_of(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(16u * lane) + at, so, 0),
                 __builtin_amdgcn_raw_buffer_load_b32(rn, (int)next + at, so, 0));
  }
  __device__ __forceinline__ uint32_t load_far(uint32_t slot) const {
    return __builtin_amdgcn_raw_buffer_load_b32(rf, (int)(4u * lane), (int)(slot * kEvSlotBytes), 0);
  }
  __device__ __forceinline__ void store_far(uint32_t slot, uint32_t x) const {
    __builtin_amdgcn_raw_buffer_store_b32(x, rf, (int)(4u * lane), (int)(slot * kEvSlotBytes), 0);
  }
  // The accumulator of a far dependency: in device memory when a far user
  // above has been decided in this scan, else S_{t+1}.
  __device__ __forceinline__ uint32_t far_acc(uint32_t node, uint32_t up, uint32_t slot) const {
    return (int32_t)up <= vstart ? load_far(slot) : load_s1(node);
  }
  __device__ __forceinline__ void store_record(uint32_t so, uint32_t R, uint32_t S, uint32_t f0, uint32_t f1) const {
    const u32x4 a = {R, S, f0, f1};
    __builtin_amdgcn_raw_buffer_store_b128(a, re, (int)(16u * lane), (int)so, 0);
  }
  // The next chunk's accumulators (LDS works in order: every update so far is in them).
  __device__ __forceinline__ void read_chunk(int c) {
    const uint32_t ring = (uint32_t)((kEvChunk * c) & (kEvRing - 1)) * kEvSlotBytes;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pre[j] = at(ring + (uint32_t)j * kEvSlotBytes);
      held[j] = at(ring + (uint32_t)(kEvHeld + j) * kEvSlotBytes);
    }
  }
};

__device__ __forceinline__ uint32_t rl(uint32_t w, int lane) { return __builtin_amdgcn_readlane(w, lane); }

// Accumulators of a chunk's far slots (2 j + s), on their way to its staging
// slots; S words and accumulators of a chunk on their way into the ring.
struct FarSet {
  uint32_t x[8], next[8];   // the accumulator, or the tile's and the next tile's S words
};
struct Entry {
  Quad s, next;
  uint32_t far[4];
};

__device__ __forceinline__ bool is_far_slot(uint32_t flags, int k) {
  return k ? (flags & (kEvFar1 | kEvSync1)) == kEvFar1 : (flags & (kEvFar0 | kEvSync0)) == kEvFar0;
}
__device__ __forceinline__ void far_issue(const Closure& s, uint32_t d, int c, FarSet& f) {
  const uint32_t fl = rl(d, 15);
  if (c < 0 || !(fl & kEvChunkFar)) return;
  if (!(fl & kEvChunkRare)) {
    // S_{t+1} of the nodes' slots 0 (of any word for those that are not far)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int so = (int)rl(d, 16 * j + 11);
      f.x[2 * j] = __builtin_amdgcn_raw_buffer_load_b32(s.rs, (int)(16u * s.lane), so, 0);
      f.next[2 * j] = __builtin_amdgcn_raw_buffer_load_b32(s.rn, (int)s.next, so, 0);
    }
    return;
  }
#pragma unroll
  for (int o = 0; o < 8; ++o) {   // slots 1, then slots 0
    const int j = o & 3, k = 1 - (o >> 2), i = 2 * j + k;
    if (!is_far_slot(rl(d, 16 * j + 1), k)) continue;
    // one load from the far accumulators or the tile's S words, one (a read
    // past the buffer for the former) from the next tile's; no branch, so
    // that neither waits for the other
    const uint32_t w = rl(d, 16 * j + 4 + k);
    const bool acc = (int32_t)(w >> 16) <= s.vstart;
    const uint32_t slot = (rl(d, 16 * j + 7) >> (16 * k)) & 0xFFFFu, at = 4u * (w & 3u);
    const uint32_t so = kEvQuadBytes * ((w & 0xFFFFu) >> 2);
    const auto r = buffer(acc ? s.far : s.tile, acc ? s.far_bytes : s.tile_bytes);
    f.x[i] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)((acc ? 4u : 16u) * s.lane + (acc ? 0u : at)),
                                                  (int)(acc ? slot * kEvSlotBytes : so), 0);
    f.next[i] = __builtin_amdgcn_raw_buffer_load_b32(s.rn, (int)(acc ? 0xFFFFF000u : s.next + at), (int)so, 0);
  }
}
__device__ __forceinline__ void far_stage(const Closure& s, uint32_t d, int c, FarSet& f) {
  const uint32_t fl = rl(d, 15);
  if (c < 0 || !(fl & kEvChunkFar)) return;
  if (!(fl & kEvChunkRare)) {
    const uint32_t stage = (uint32_t)(kEvStage + 2 * ((kEvChunk * c) & 7)) * kEvSlotBytes;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      asm volatile("" : "+v"(f.x[2 * j]), "+v"(f.next[2 * j]));
      s.put(stage + (uint32_t)(2 * j) * kEvSlotBytes, s.s1_of(f.x[2 * j], f.next[2 * j]));
    }
    return;
  }
#pragma unroll
  for (int o = 0; o < 8; ++o) {   // slots 1, then slots 0
    const int j = o & 3, k = 1 - (o >> 2), i = 2 * j + k;
    if (!is_far_slot(rl(d, 16 * j + 1), k)) continue;
    const bool acc = (int32_t)(rl(d, 16 * j + 4 + k) >> 16) <= s.vstart;
    // used here and not before, as in finish()
    asm volatile("" : "+v"(f.x[i]), "+v"(f.next[i]));
    s.put(rl(d, 16 * j + 2 * k), acc ? f.x[i] : s.s1_of(f.x[i], f.next[i]));
  }
}
__device__ __forceinline__ void entry_issue(const Closure& s, uint32_t d, int e, Entry& x) {
  x.s = s.load_own(e);
  x.next = s.load_next(e);
  if (e < 0 || !(rl(d, 15) & kEvChunkEntry)) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) x.far[j] = s.load_far(rl(d, 16 * j + 6) & 0xFFFFu);
}
__device__ __forceinline__ void entry_write(const Closure& s, uint32_t d, int e, Entry& x) {
  if (e < 0) return;
  // used here and not before, as in finish()
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(x.s.x[j]), "+v"(x.next.x[j]), "+v"(x.far[j]));
  const uint32_t ring = (uint32_t)((kEvChunk * e) & (kEvRing - 1)) * kEvSlotBytes;
  uint32_t a[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = s.s1_of(x.s.x[j], x.next.x[j]);
  if (rl(d, 15) & kEvChunkEntry) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w = rl(d, 16 * j + 6);
      uint32_t far = x.far[j];
      if (__builtin_expect((rl(d, 16 * j + 1) & kEvEntrySync) != 0u, 0)) far = s.load_far(w & 0xFFFFu);
      a[j] = (int32_t)(w >> 16) <= s.vstart ? far : a[j];
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    s.put(ring + (uint32_t)j * kEvSlotBytes, a[j]);
    s.put(ring + (uint32_t)(kEvHeld + j) * kEvSlotBytes, x.s.x[j]);
  }
}

// Stores a chunk's records and the accumulators of its far dependencies.
__device__ __forceinline__ void finish(const Closure& s, Pending& p) {
  if (!p.live) return;
  p.live = false;
  const int vo = (int)(16u * s.lane);
  // the release words are used here and not before (the compiler would wait
  // for them as soon as they are asked for)
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(p.a0[j]), "+v"(p.a1[j]));
  if (!p.second) {
    const int so = (int)rl(p.d, 3);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32x4 w = {p.R[j], p.S[j], p.R[j] & ~p.a0[j], p.R[j] & ~p.a1[j]};
      __builtin_amdgcn_raw_buffer_store_b128(w, s.re, vo + j * kEvRecBytes, so, 0);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int so = (int)rl(p.d, 16 * j + 3);
      const u32x4 w = {p.R[j], p.S[j], p.R[j] & ~p.a0[j], p.R[j] & ~p.a1[j]};
      __builtin_amdgcn_raw_buffer_store_b128(w, s.re, vo, so, 0);
      if (rl(p.d, 16 * j + 1) & kEvSecond) {
        asm volatile("" : "+v"(p.a2[j]), "+v"(p.a3[j]));
        const u32x4 w2 = {0u, 0u, p.R[j] & ~p.a2[j], p.R[j] & ~p.a3[j]};
        __builtin_amdgcn_raw_buffer_store_b128(w2, s.re, vo + kEvRecBytes, so, 0);
      }
    }
  }
  if (p.far) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_buffer_store_b32(p.a0[j] | p.R[j], s.rf, (int)(4u * s.lane), (int)rl(p.d, 16 * j + 12), 0);
  }
}

// Node 4c + J in the general form: its word R, then its dependencies' release
// words and accumulators. Every access waits for the one before.
template <int J>
__device__ __forceinline__ void any_node(const ClosureArgs& a, const Closure& s, int c, uint32_t d) {
  const uint32_t f = rl(d, 16 * J + 1), so = rl(d, 16 * J + 3);
  const uint32_t ring = (uint32_t)((kEvChunk * c + J) & (kEvRing - 1)) * kEvSlotBytes;
  const uint32_t S0 = s.at(ring + kEvHeld * kEvSlotBytes);
  uint32_t R = s.at((f & kEvPinned) ? rl(d, 16 * J + 10) : ring) & ~S0;
  const int v = kEvChunk * c + J, b = v - s.b0;
  // stages below v compute nothing here, stage v computes it (4a)
  if (b >= 0) R = b >= kEvTile ? 0u : (R & (~0u << b)) | (v < s.n ? 1u << b : 0u);
  const uint32_t first = rl(d, 16 * J + 9);
  const uint32_t so2 = so + ((f & kEvSecond) ? 2u : 1u) * kEvRecBytes;
  for (int x = (int)(f >> 16) - 1; x >= 0; --x) {
    const auto e = *(cptr<u32x8>)(a.extra + (size_t)(first + (uint32_t)x) * kEvExtraDw);
    if (e[1] & kEvFar0) s.put(e[0] & 0xFFFFu, s.far_acc(e[3] & 0xFFFFu, e[4] & 0xFFFFu, e[2] & 0xFFFFu));
    if (e[1] & kEvFar1) s.put(e[0] >> 16, s.far_acc(e[3] >> 16, e[4] >> 16, e[2] >> 16));
    const uint32_t a0 = s.lds_or(e[0] & 0xFFFFu, R), a1 = s.lds_or(e[0] >> 16, R);
    s.store_record(so2 + (uint32_t)x * kEvRecBytes, 0, 0, R & ~a0, R & ~a1);
    if (e[1] & kEvFar0) s.store_far(e[2] & 0xFFFFu, a0 | R);
    if (e[1] & kEvFar1) s.store_far(e[2] >> 16, a1 | R);
  }
  const uint32_t fs = rl(d, 16 * J + 7);
  if (f & kEvSync0) {
    const uint32_t w = rl(d, 16 * J + 4);
    s.put(rl(d, 16 * J), s.far_acc(w & 0xFFFFu, w >> 16, fs & 0xFFFFu));
  }
  if (f & kEvSync1) {
    const uint32_t w = rl(d, 16 * J + 5);
    s.put(rl(d, 16 * J + 2), s.far_acc(w & 0xFFFFu, w >> 16, fs >> 16));
  }
  const uint32_t a0 = s.lds_or(rl(d, 16 * J), R), a1 = s.lds_or(rl(d, 16 * J + 2), R);
  s.store_record(so, R, S0, R & ~a0, R & ~a1);
  if (f & kEvSecond) {
    const uint32_t o = rl(d, 16 * J + 8);
    const uint32_t a2 = s.lds_or(o & 0xFFFFu, R), a3 = s.lds_or(o >> 16, R);
    s.store_record(so + kEvRecBytes, 0, 0, R & ~a2, R & ~a3);
  }
  if (f & kEvFar0) s.store_far(fs & 0xFFFFu, a0 | R);
  if (f & kEvFar1) s.store_far(fs >> 16, a1 | R);
}

// The chunks whose descriptors are at hand.
struct Descs {
  uint32_t c0, c1, c2, c3;   // chunks c .. c - 3
  uint32_t e0, e1, e2;       // chunks c - 7 .. c - 9
};

// Decides chunk c. Most chunks, those below the tile's stages with none of the
// rare forms, are decided four nodes at once: a wave alone on its SIMD waits
// out every LDS access, so their accumulators are read together (after the
// updates of the chunk above), uses within the chunk pass through registers,
// and the records of the chunk above are stored while the updates run.
__device__ __forceinline__ void decide(const ClosureArgs& a, Closure& s, int c, uint32_t d, Pending& p, Pending& last) {
  const uint32_t flags = rl(d, 15);
  if (__builtin_expect(kEvChunk * c + 3 >= s.b0 || (flags & kEvChunkRare), 0)) {
    finish(s, last);
    any_node<3>(a, s, c, d);
    any_node<2>(a, s, c, d);
    any_node<1>(a, s, c, d);
    any_node<0>(a, s, c, d);
    s.read_chunk(c - 1);
    p.live = false;
    return;
  }
  const auto use = [&](int b) { return (uint32_t)((int32_t)(flags << (31 - kEvChunkUse - b)) >> 31); };
  p.d = d;
#pragma unroll
  for (int j = 0; j < 4; ++j) p.S[j] = s.held[j];
  p.R[3] = s.pre[3] & ~p.S[3];
  p.R[2] = (s.pre[2] | (p.R[3] & use(0))) & ~p.S[2];
  p.R[1] = (s.pre[1] | (p.R[3] & use(1)) | (p.R[2] & use(3))) & ~p.S[1];
  p.R[0] = (s.pre[0] | (p.R[3] & use(2)) | (p.R[2] & use(4)) | (p.R[1] & use(5))) & ~p.S[0];
  p.live = true;
  p.far = (flags & kEvChunkFar) != 0;
  p.second = (flags & kEvChunkSecond) != 0;
  if (!p.second) {
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      p.a0[j] = s.lds_or(rl(d, 16 * j), p.R[j]);
      p.a1[j] = s.lds_or(rl(d, 16 * j + 2), p.R[j]);
    }
  } else {
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      p.a0[j] = s.lds_or(rl(d, 16 * j), p.R[j]);
      p.a1[j] = s.lds_or(rl(d, 16 * j + 2), p.R[j]);
      // absent second records update the slot that is all ones
      const uint32_t o = rl(d, 16 * j + 8);
      p.a2[j] = s.lds_or(o & 0xFFFFu, p.R[j]);
      p.a3[j] = s.lds_or(o >> 16, p.R[j]);
    }
  }
  s.read_chunk(c - 1);
  finish(s, last);
}

// Chunk c, then the loads that come due: f and x hold the far accumulators of
// chunk c - 1 and the ring entry of chunk c - 7, and take those of chunks
// c - 3 and c - 9.
__device__ __forceinline__ void closure_chunk(const ClosureArgs& a, Closure& s, int c, Descs& d, FarSet& f, Entry& x,
                                              Pending& p, Pending& last) {
  const uint32_t c4 = s.load_desc(c - 4), e3 = s.load_desc(c - 10);
  decide(a, s, c, d.c0, p, last);
  far_stage(s, d.c1, c - 1, f);
  far_issue(s, d.c3, c - 3, f);
  if (__builtin_expect(c >= kEvNear + 1 && (rl(d.e0, 15) & kEvChunkEntrySync), 0)) finish(s, p);
  entry_write(s, d.e0, c - 7, x);
  entry_issue(s, d.e2, c - 9, x);
  d = {d.c1, d.c2, d.c3, c4, d.e1, d.e2, e3};
}

__global__ void __launch_bounds__(kWave) ckm_closure_kernel(ClosureArgs a) {
  __shared__ uint32_t lds[kEvSlots * kWave];
  const int lane = threadIdx.x;
  const int tile = a.thi - 1 - (int)blockIdx.y;   // the longest scans start first
  const int slot = blockIdx.x;                    // of the event and far arrays
  int group = a.g0 + slot;
  if (a.best_k) {
    const int bk = uniform(a.best_k[0]);
    if (bk < 0) return;
    group = bk / kWave;
  }
  Closure s;
  s.lane = lane;
  s.lds = (lds_char*)&lds[lane];
  s.b0 = kEvTile * tile;
  s.n = a.n;
  const char* st = a.stiles + (size_t)group * a.s_bytes + stile_off(tile);
  s.tile = st;
  s.tile_bytes = stile_bytes(tile);
  s.rs = buffer(st, s.tile_bytes);
  s.rn = buffer(tile + 1 < a.tiles ? st + stile_bytes(tile) : st, stile_bytes(tile));   // as many quads are read
  s.next = tile + 1 < a.tiles ? 16u * lane : 0xFFFFF000u;
  const uint64_t eo = a.tile_off[tile];
  s.re = buffer(a.events + (size_t)slot * a.ev_bytes + (eo - a.tile_off[a.tlo]), (uint32_t)(a.tile_off[tile + 1] - eo));
  s.far = a.far + ((size_t)slot * (a.thi - a.tlo) + (tile - a.tlo)) * a.far_bytes;
  s.far_bytes = a.far_bytes;
  s.rf = buffer(s.far, a.far_bytes);
  const int cT = ev_first_chunk(a.n, tile);
  s.rd = buffer(a.desc, (uint32_t)(cT + 1) * 256u);
  s.vstart = 4 * cT + 3;

  // the slots as they are before anything is decided: S_{t+1} everywhere
  Descs d = {s.load_desc(cT),     s.load_desc(cT - 1), s.load_desc(cT - 2), s.load_desc(cT - 3),
             s.load_desc(cT - 7), s.load_desc(cT - 8), s.load_desc(cT - 9)};
  s.put(kEvNone * kEvSlotBytes, ~0u);
  for (int p = 0; p < a.npins; ++p)
    if (a.pins[p] <= s.vstart) s.put((uint32_t)(kEvPin + p) * kEvSlotBytes, s.load_s1((uint32_t)a.pins[p]));
  for (int c = cT; c >= 0 && c >= cT - kEvNear; --c) {
    const Quad q = s.load_own(c), nx = s.load_next(c);
    const uint32_t ring = (uint32_t)((kEvChunk * c) & (kEvRing - 1)) * kEvSlotBytes;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s.put(ring + (uint32_t)j * kEvSlotBytes, s.s1_of(q.x[j], nx.x[j]));
      s.put(ring + (uint32_t)(kEvHeld + j) * kEvSlotBytes, q.x[j]);
    }
  }
  FarSet f0 = {}, f1 = {};
  far_issue(s, d.c0, cT, f0);
  far_stage(s, d.c0, cT, f0);
  Entry x0 = {}, x1 = {};
  far_issue(s, d.c1, cT - 1, f0);
  entry_issue(s, d.e0, cT - 7, x0);
  far_issue(s, d.c2, cT - 2, f1);
  entry_issue(s, d.e1, cT - 8, x1);
  s.read_chunk(cT);
  Pending p0, p1;
  p0.live = p1.live = false;
  int c = cT;
  for (; c >= 1; c -= 2) {
    closure_chunk(a, s, c, d, f0, x0, p0, p1);
    closure_chunk(a, s, c - 1, d, f1, x1, p1, p0);
  }
  if (c == 0) {
    closure_chunk(a, s, 0, d, f0, x0, p0, p1);
    finish(s, p0);
  } else {
    finish(s, p1);
  }
}

// ---------------------------------------------------------------------------
// Simulate: the U recurrence (Section 4.4) and the cost (Section 4.3), one
// wave per (group, 8 stages of a tile, part of the tile's records). Before
// node v is computed the memory is U_{t,0} + U; computing it adds M_v (the
// peak is taken there), then the dependencies that FREE releases after it
// leave. All sums are binary64 integers below 2^53, exact in any order; stage
// j of the tile counts in units of 2^(j - 1074), so that its bit of a word is
// the unit itself (denormals are exact and run at full rate).
struct SimArgs {
  int32_t n, K, tlo, thi, g0, groups;
  double base;                      // M_in + 2 M_param
  size_t ev_bytes;                  // event records of one group in the chunk
  const char* events;               // from group g0
  cptr<char> ops;
  cptr<uint64_t> tile_off;
  int64_t* __restrict__ peak;
  int64_t* __restrict__ cost;
};

constexpr int kSub = 8;             // stages per wave
constexpr int kSubs = kEvTile / kSub;

struct SimStages {
  double U[kSub], top[kSub], U0[kSub];   // relative to the stage's start; its peak; U_{t,0}
};

// One event record (words w = R, S, F0, F1) for stages kFirst .. kFirst + 7.
template <int kFirst>
__device__ __forceinline__ void sim_record(SimStages& x, const u32x4& w, double M, double M0, double M1) {
  constexpr int b0 = (int)(1u << kFirst), b1 = (int)(2u << kFirst), b2 = (int)(4u << kFirst), b3 = (int)(8u << kFirst),
                b4 = (int)(16u << kFirst), b5 = (int)(32u << kFirst), b6 = (int)(64u << kFirst),
                b7 = (int)(128u << kFirst);
  asm("v_mov_b32 v9, 0\n\t"
      "v_mov_b32 v11, 0\n\t"
      "v_and_b32 v8, %[b0], %[S]\n\t"
      "v_and_b32 v10, %[b1], %[S]\n\t"
      "v_fma_f64 %[z0], v[8:9], %[M], %[z0]\n\t"
      "v_fma_f64 %[z1], v[10:11], %[M], %[z1]\n\t"
      "v_and_b32 v8, %[b2], %[S]\n\t"
      "v_and_b32 v10, %[b3], %[S]\n\t"
      "v_fma_f64 %[z2], v[8:9], %[M], %[z2]\n\t"
      "v_fma_f64 %[z3], v[10:11], %[M], %[z3]\n\t"
      "v_and_b32 v8, %[b4], %[S]\n\t"
      "v_and_b32 v10, %[b5], %[S]\n\t"
      "v_fma_f64 %[z4], v[8:9], %[M], %[z4]\n\t"
      "v_fma_f64 %[z5], v[10:11], %[M], %[z5]\n\t"
      "v_and_b32 v8, %[b6], %[S]\n\t"
      "v_and_b32 v10, %[b7], %[S]\n\t"
      "v_fma_f64 %[z6], v[8:9], %[M], %[z6]\n\t"
      "v_fma_f64 %[z7], v[10:11], %[M], %[z7]"
      : [z0] "+v"(x.U0[0]), [z1] "+v"(x.U0[1]), [z2] "+v"(x.U0[2]), [z3] "+v"(x.U0[3]), [z4] "+v"(x.U0[4]),
        [z5] "+v"(x.U0[5]), [z6] "+v"(x.U0[6]), [z7] "+v"(x.U0[7])
      : [S] "v"(w[1]), [M] "s"(M), [b0] "i"(b0), [b1] "i"(b1), [b2] "i"(b2), [b3] "i"(b3), [b4] "i"(b4), [b5] "i"(b5),
        [b6] "i"(b6), [b7] "i"(b7)
      : "v8", "v9", "v10", "v11");
  // pairs of stages, so that no instruction waits for the one before it
#define CKM_PAIR(i, j, bi, bj)                                                                            \
  asm("v_mov_b32 v9, 0\n\t"                                                                               \
      "v_mov_b32 v11, 0\n\t"                                                                              \
      "v_and_b32 v8, %[a], %[R]\n\t"                                                                      \
      "v_and_b32 v10, %[b], %[R]\n\t"                                                                     \
      "v_fma_f64 %[u0], v[8:9], %[M], %[u0]\n\t"                                                          \
      "v_fma_f64 %[u1], v[10:11], %[M], %[u1]\n\t"                                                        \
      "v_and_b32 v8, %[a], %[F]\n\t"                                                                      \
      "v_and_b32 v10, %[b], %[F]\n\t"                                                                     \
      "v_max_f64 %[t0], %[t0], %[u0]\n\t"                                                                 \
      "v_max_f64 %[t1], %[t1], %[u1]\n\t"                                                                 \
      "v_fma_f64 %[u0], v[8:9], -%[M0], %[u0]\n\t"                                                        \
      "v_fma_f64 %[u1], v[10:11], -%[M0], %[u1]\n\t"                                                      \
      "v_and_b32 v8, %[a], %[G]\n\t"                                                                      \
      "v_and_b32 v10, %[b], %[G]\n\t"                                                                     \
      "v_fma_f64 %[u0], v[8:9], -%[M1], %[u0]\n\t"                                                        \
      "v_fma_f64 %[u1], v[10:11], -%[M1], %[u1]"                                                          \
      : [u0] "+v"(x.U[i]), [u1] "+v"(x.U[j]), [t0] "+v"(x.top[i]), [t1] "+v"(x.top[j])                     \
      : [R] "v"(w[0]), [F] "v"(w[2]), [G] "v"(w[3]), [M] "s"(M), [M0] "s"(M0), [M1] "s"(M1), [a] "i"(bi), \
        [b] "i"(bj)                                                                                       \
      : "v8", "v9", "v10", "v11")
  CKM_PAIR(0, 1, b0, b1);
  CKM_PAIR(2, 3, b2, b3);
  CKM_PAIR(4, 5, b4, b5);
  CKM_PAIR(6, 7, b6, b7);
#undef CKM_PAIR
}

// Records r0 .. r1 - 1 (r0 a multiple of 4; reads past the tile's records give
// zeros, which change nothing), four at a time, the next four on their way.
// Every fourth record's cost is this wave's to count, over all 32 stages.
template <int kSubIdx>
__device__ __forceinline__ void sim_scan(SimStages& x, uint64_t& cost_lo, uint64_t& cost_hi, __amdgpu_buffer_rsrc_t re,
                                         cptr<char> ops, uint32_t lane, int r0, int r1) {
  u32x4 cur[4], nxt[4];
  const auto load = [&](u32x4(&w)[4], int r) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = __builtin_amdgcn_raw_buffer_load_b128(re, (int)(16u * lane) + r * kEvRecBytes + i * kEvRecBytes, 0, 0);
  };
  const auto four = [&](const u32x4(&w)[4], int r) {
    const cptr<u64x8> o = (cptr<u64x8>)(ops + (size_t)r * sizeof(EvOps));
    const u64x8 oa = o[0], ob = o[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto v = [&](int k) { return i < 2 ? oa[4 * i + k] : ob[4 * (i - 2) + k]; };
      sim_record<kSub * kSubIdx>(x, w[i], __builtin_bit_cast(double, v(0)), __builtin_bit_cast(double, v(2)),
                                 __builtin_bit_cast(double, v(3)));
      if (i == kSubIdx) {
        const uint32_t c = (uint32_t)__builtin_popcount(w[i][0]);
        cost_lo += (uint64_t)c * (uint32_t)v(1);
        cost_hi += (uint64_t)c * (uint32_t)(v(1) >> 32);
      }
    }
  };
  load(cur, r0);
  for (int r = r0; r < r1; r += 8) {
    load(nxt, r + 4);
    four(cur, r);
    if (r + 4 >= r1) break;
    load(cur, r + 8);
    four(nxt, r + 4);
  }
}

// kSegs waves share a tile's eight stages, each a part of the records; their
// results are joined in order (a part's peak counts from the memory the parts
// before it leave).
template <int kSegs>
__global__ void __launch_bounds__(kWave* kSegs) ckm_simulate_kernel(SimArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int seg = kSegs == 1 ? 0 : uniform((int)threadIdx.x / kWave);
  // the four waves that read one tile's records come 8 blocks apart: blocks
  // go to the 8 XCDs in turn, so these share an L2
  const int id = blockIdx.x, sub = (id >> 3) & (kSubs - 1), item = (id / (8 * kSubs)) * 8 + (id & 7);
  if (item >= (a.thi - a.tlo) * a.groups) return;
  const int tile = a.thi - 1 - item / a.groups;   // the longest start first
  const int slot = item % a.groups;
  const uint64_t eo = a.tile_off[tile], bytes = a.tile_off[tile + 1] - eo;
  const auto re = buffer(a.events + (size_t)slot * a.ev_bytes + (eo - a.tile_off[a.tlo]), (uint32_t)bytes);
  const int fours = ((int)(bytes / kEvRecBytes) + 3) / 4;
  const int r0 = 4 * (fours * seg / kSegs), r1 = 4 * (fours * (seg + 1) / kSegs);
  SimStages x;
#pragma unroll
  for (int j = 0; j < kSub; ++j) {
    x.U[j] = 0.0;
    x.top[j] = -INFINITY;
    x.U0[j] = 0.0;
  }
  uint64_t cost_lo = 0, cost_hi = 0;
  if (r0 < r1) {
    switch (sub) {
      case 0: sim_scan<0>(x, cost_lo, cost_hi, re, a.ops, lane, r0, r1); break;
      case 1: sim_scan<1>(x, cost_lo, cost_hi, re, a.ops, lane, r0, r1); break;
      case 2: sim_scan<2>(x, cost_lo, cost_hi, re, a.ops, lane, r0, r1); break;
      default: sim_scan<3>(x, cost_lo, cost_hi, re, a.ops, lane, r0, r1); break;
    }
  }
  const int k = (a.g0 + slot) * kWave + lane;
  const uint64_t cost = cost_lo + (cost_hi << 32);
  if (k < a.K && cost) atomicAdd(reinterpret_cast<unsigned long long*>(a.cost) + k, (unsigned long long)cost);
  if constexpr (kSegs > 1) {
    __shared__ double part[3 * kSub][kWave];
    for (int s = 1; s < kSegs; ++s) {
      __syncthreads();
      if (seg == s) {
#pragma unroll
        for (int j = 0; j < kSub; ++j) {
          part[3 * j][lane] = x.U[j];
          part[3 * j + 1][lane] = x.top[j];
          part[3 * j + 2][lane] = x.U0[j];
        }
      }
      __syncthreads();
      if (seg == 0) {
#pragma unroll
        for (int j = 0; j < kSub; ++j) {
          x.top[j] = fmax(x.top[j], x.U[j] + part[3 * j + 1][lane]);
          x.U[j] += part[3 * j][lane];
          x.U0[j] += part[3 * j + 2][lane];
        }
      }
    }
    if (seg) return;
  }
  int64_t peak = INT64_MIN;
#pragma unroll
  for (int j = 0; j < kSub; ++j) {
    const int b = kSub * sub + j;
    if (kEvTile * tile + b < a.n) {
      const int64_t p = (int64_t)(a.base + ldexp(x.U0[j] + x.top[j], 1074 - b));
      peak = p > peak ? p : peak;
    }
  }
  if (k < a.K) atomicMax(reinterpret_cast<long long*>(a.peak) + k, (long long)peak);
}

// ---------------------------------------------------------------------------
// Best candidate's R rows of a chunk's tiles from their event records: block
// per tile, lane = node.
__global__ void __launch_bounds__(256) ckm_best_events_kernel(const char* __restrict__ events, size_t ev_bytes,
                                                              int32_t one_group, int32_t tlo, int32_t n,
                                                              const uint64_t* __restrict__ tile_off,
                                                              const int32_t* __restrict__ main_rec, int32_t words64,
                                                              const int32_t* __restrict__ best_k,
                                                              uint64_t* __restrict__ R_rows) {
  const int tile = tlo + blockIdx.x;
  const int bk = best_k[0];
  const char* rec = events + (size_t)(bk < 0 || one_group ? 0 : bk / kWave) * ev_bytes + (tile_off[tile] - tile_off[tlo]) +
                    16 * (bk & (kWave - 1));
  const int lim = min(n, kEvTile * (tile + 1));   // nodes above compute nothing in these stages
  const int v = blockIdx.y * 256 + threadIdx.x;
  if (v >= kWave * words64) return;               // whole waves
  uint32_t w = 0;
  if (bk >= 0 && v < lim) w = *reinterpret_cast<const uint32_t*>(rec + (size_t)main_rec[v] * kEvRecBytes);
  for (int j = 0; j < kEvTile && kEvTile * tile + j < n; ++j) {
    const uint64_t row = __ballot((w >> j) & 1u);
    if ((threadIdx.x & (kWave - 1)) == 0) R_rows[(size_t)(kEvTile * tile + j) * words64 + v / kWave] = row;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
static ClosureArgs closure_args(const ckm_graph& g, const Layout& L, const EvChunk& ch, char* work) {
  const EventGraph& ev = g.ev;
  ClosureArgs a;
  a.n = g.n;
  a.tiles = ev.tiles;
  a.tlo = ch.tlo;
  a.thi = ch.thi;
  a.g0 = ch.g0;
  a.npins = ev.npins;
  a.far_bytes = (uint32_t)ev.nf * kEvSlotBytes;
  a.s_bytes = stiles_bytes(g.n);
  a.ev_bytes = ev.tile_off[ch.thi] - ev.tile_off[ch.tlo];
  a.stiles = work + L.rows_off;
  a.events = work + L.events_off;
  a.far = a.events + (size_t)ch.gn * a.ev_bytes;
  a.desc = ev.d_desc;
  a.extra = (cptr<uint32_t>)ev.d_extra;
  a.tile_off = (cptr<uint64_t>)ev.d_tile_off;
  a.pins = (cptr<int32_t>)ev.d_pins;
  a.best_k = nullptr;
  return a;
}

hipError_t launch_events(const ckm_graph& g, const Layout& L, int32_t K, char* work, hipStream_t stream) {
  EvChunk ch;
  for (bool more = first_event_chunk(g, L, K, ch); more; more = next_event_chunk(g, L, K, ch)) {
    const ClosureArgs c = closure_args(g, L, ch, work);
    hipLaunchKernelGGL(ckm_closure_kernel, dim3(ch.gn, ch.thi - ch.tlo), dim3(kWave), 0, stream, c);
    SimArgs s;
    s.n = g.n;
    s.K = K;
    s.tlo = ch.tlo;
    s.thi = ch.thi;
    s.g0 = ch.g0;
    s.groups = ch.gn;
    s.base = (double)g.base;
    s.ev_bytes = c.ev_bytes;
    s.events = c.events;
    s.ops = (cptr<char>)g.ev.d_ops;
    s.tile_off = c.tile_off;
    s.peak = reinterpret_cast<int64_t*>(work + L.part_peak_off);
    s.cost = reinterpret_cast<int64_t*>(work + L.part_cost_off);
    const int64_t items = (int64_t)ch.gn * (ch.thi - ch.tlo);
    const dim3 grid((unsigned)((items + 7) / 8 * 8 * kSubs));
    if (items >= 4096)
      hipLaunchKernelGGL(ckm_simulate_kernel<1>, grid, dim3(kWave), 0, stream, s);
    else if (items >= 1024)
      hipLaunchKernelGGL(ckm_simulate_kernel<2>, grid, dim3(2 * kWave), 0, stream, s);
    else if (items >= 256)
      hipLaunchKernelGGL(ckm_simulate_kernel<4>, grid, dim3(4 * kWave), 0, stream, s);
    else
      hipLaunchKernelGGL(ckm_simulate_kernel<8>, grid, dim3(8 * kWave), 0, stream, s);
  }
  return hipGetLastError();
}

hipError_t launch_best_events(const ckm_graph& g, const Layout& L, int32_t K, const int32_t* d_best_k,
                              uint64_t* d_best_R, char* work, hipStream_t stream) {
  // the event records of every group are still there when one chunk held
  // them all; else the best candidate's group is decided again
  EvChunk ch;
  bool more = first_event_chunk(g, L, K, ch);
  const bool kept = ch.tlo == 0 && ch.thi == g.ev.tiles && ch.gn == (K + kWave - 1) / kWave;
  if (!kept) more = first_event_chunk(g, L, 1, ch);
  for (; more; more = next_event_chunk(g, L, 1, ch)) {
    ClosureArgs c = closure_args(g, L, ch, work);
    if (!kept) {
      c.best_k = d_best_k;
      hipLaunchKernelGGL(ckm_closure_kernel, dim3(1, ch.thi - ch.tlo), dim3(kWave), 0, stream, c);
    }
    const int32_t words64 = L.row_words / 2;
    hipLaunchKernelGGL(ckm_best_events_kernel, dim3(ch.thi - ch.tlo, (kWave * words64 + 255) / 256), dim3(256), 0,
                       stream, c.events, c.ev_bytes, kept ? 0 : 1, ch.tlo, g.n, g.ev.d_tile_off, g.ev.d_main_rec,
                       words64, d_best_k, d_best_R);
    if (kept) break;
  }
  return hipGetLastError();
}

}  // namespace ckm

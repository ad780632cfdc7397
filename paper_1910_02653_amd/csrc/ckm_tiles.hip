// Tile path (see ckm_tiles.h): the closure kernel, which decides R of every
// (candidate, stage, node), the hub words, the simulate kernel, which runs the
// U recurrence, and the gather of the best candidate's R.
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

#include "ckm_internal.h"
#include "ckm_tiles.h"

namespace ckm {
namespace {

template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

constexpr int kBufWord3 = 0x00020000;          // raw byte-addressed buffer: reads past its end give 0
constexpr uint32_t kPastEnd = 0xFFFFF000u;     // a lane offset past the end of any tile

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t rl(uint32_t w, int lane) { return __builtin_amdgcn_readlane(w, lane); }
// S_{t+1} of a tile's stages: its own S words shifted, the next tile's first stage on top.
__device__ __forceinline__ uint32_t s1_of(uint32_t s, uint32_t next) { return __builtin_amdgcn_alignbit(next, s, 1); }

struct TileArgs {
  int32_t n, tiles, groups;
  size_t s_bytes, r_bytes;          // S and R tiles of one group
  const char* stiles;
  char* rtiles;
};
// The buffers of one (group, tile).
struct TileBufs {
  __amdgpu_buffer_rsrc_t s, next, r;
  uint32_t vo, vo_next;             // lane offsets; the next tile's is past the end after the last tile
  uint32_t r_bytes;
  __device__ __forceinline__ TileBufs(const TileArgs& a, int group, int tile, int lane) {
    const char* st = a.stiles + (size_t)group * a.s_bytes + stile_off(tile);
    const uint32_t bytes = stile_bytes(tile);
    const bool last = tile + 1 == a.tiles;
    s = buffer(st, bytes);
    next = buffer(last ? st : st + bytes, bytes);   // as many nodes of it are read
    vo = 4u * (uint32_t)lane;
    vo_next = last ? kPastEnd : vo;
    r_bytes = kRBase + bytes;
    r = buffer(a.rtiles + (size_t)group * a.r_bytes + rtile_off(tile), r_bytes);
  }
};

// ---------------------------------------------------------------------------
// Hub words, in the closure's blocks or in a launch of their own.
struct HubArgs {
  cptr<int32_t> ptr;
  cptr<HubUser> users;
  cptr<uint32_t> at;                // TileTables::hub_at (null: no hub words)
  char* buf;                        // the words of a launch's pairs, one pair after another
  int32_t item0, items;             // the pairs
  int32_t nhub;
};
__device__ __forceinline__ void tile_of(const TileArgs& t, int item, int& tile, int& group) {
  tile = t.tiles - 1 - item / t.groups;   // the longest start first
  group = item % t.groups;
}
// A pair's hub words: a word of zeros, then `words` words.
struct HubBuf {
  __amdgpu_buffer_rsrc_t buf;
  uint32_t words;
  __device__ __forceinline__ HubBuf(const TileArgs& t, const HubArgs& h, int tile, int group) {
    const auto before = [&](int T, int g) { return (uint64_t)t.groups * h.at[T + 1] + (uint64_t)g * (h.at[T] - h.at[T + 1]); };
    int tile0, group0;
    tile_of(t, h.item0, tile0, group0);
    words = h.at[tile] - h.at[tile + 1] - 1;
    buf = buffer(h.buf + (before(tile, group) - before(tile0, group0)) * kSlotBytes, node_off(1 + (int)words));
  }
};
// One wave's hub, over its users below the tile's end from the highest down. The
// bound is memory: a word read per user, and one written per step of them.
__device__ __forceinline__ void hub_words(const TileBufs& b, const HubArgs& h, __amdgpu_buffer_rsrc_t out, int hub) {
  if (hub == 0) __builtin_amdgcn_raw_buffer_store_b32(0u, out, (int)b.vo, 0, 0);
  const int e1 = h.ptr[hub + 1];
  int e0 = h.ptr[hub];
  for (int end = e1; e0 < end;) {   // users at or above the tile's end compute nothing in its stages
    const int mid = (e0 + end) / 2;
    if (h.users[mid].r < b.r_bytes)
      end = mid;
    else
      e0 = mid + 1;
  }
  uint32_t acc = 0;
  for (int e = e0; e < e1; e += 8) {
    uint32_t x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      x[k] = __builtin_amdgcn_raw_buffer_load_b32(b.r, (int)b.vo, (int)h.users[min(e + k, e1 - 1)].r, 0);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (e + k >= e1) break;
      acc |= x[k];
      const uint32_t xo = h.users[e + k].x;
      if (xo) __builtin_amdgcn_raw_buffer_store_b32(acc, out, (int)b.vo, (int)xo, 0);
    }
  }
}
__global__ void __launch_bounds__(kWave) ckm_hub_kernel(TileArgs t, HubArgs h) {
  int tile, group;
  tile_of(t, h.item0 + (int)blockIdx.x, tile, group);
  hub_words(TileBufs(t, group, tile, threadIdx.x), h, HubBuf(t, h, tile, group).buf, blockIdx.y);
}

// ---------------------------------------------------------------------------
// Closure: one block per (group, tile): a wave that decides, and kPrep waves
// that prepare the block of nodes below. The bound is the deciding wave's chain:
// per chunk of four nodes an LDS round trip (near users) and a few dependent
// bit operations, 8 (T + 1) chunks in a row for tile T. So all else is taken
// off that wave, and a launch hides the chain only by its number of blocks.
// Measured: n = 1009: 64 us with 3 or 8 groups, 69 us with 16 (its 256 chunks at
// 0.25 us); n = 4001, K = 4096 (8064 blocks): 2.82 ms.
constexpr int kPrep = 2;
constexpr int kPrepNodes = kTile / kPrep;

constexpr int kDescVecs = kTile / kChunk4 * kDescDwords / kWave;   // descriptor dwords per lane and block

struct ClosureArgs {
  TileArgs t;
  const uint32_t* desc;
  const uint32_t* far;
  cptr<uint32_t> far_more, near_more;
  HubArgs h;                        // nhub 0: the hub words, if any, are made in another launch
};

__device__ __forceinline__ uint32_t lds_get(lds_char* p, uint32_t off) { return *(const lds_u32*)(p + off); }
__device__ __forceinline__ void lds_put(lds_char* p, uint32_t off, uint32_t x) { *(lds_u32*)(p + off) = x; }
__device__ __forceinline__ uint32_t load_r(const TileBufs& b, uint32_t off) {
  // a user past the tile's last node computes nothing in its stages
  return __builtin_amdgcn_raw_buffer_load_b32(b.r, (int)b.vo, (int)(off < b.r_bytes ? off : 0u), 0);
}

// A prepare wave's S words of one block, requested one block ahead.
struct PrepIn {
  uint32_t s[kPrepNodes], next[kPrepNodes];
};
__device__ __forceinline__ void prep_load(const TileBufs& b, int v0, PrepIn& in) {
#pragma unroll
  for (int i = 0; i < kPrepNodes; ++i) {
    in.s[i] = __builtin_amdgcn_raw_buffer_load_b32(b.s, (int)b.vo, (int)node_off(v0 + i), 0);
    in.next[i] = __builtin_amdgcn_raw_buffer_load_b32(b.next, (int)b.vo_next, (int)node_off(v0 + i), 0);
  }
}
// Nodes v0 .. v0 + kPrepNodes - 1 into the prepared words of their block; far:
// their far users (a dword per lane), x: R of the first of them.
__device__ __forceinline__ void prep_store(const ClosureArgs& a, const TileBufs& b, lds_char* lds, int v0,
                                           const PrepIn& in, uint32_t far, uint32_t (&x)[kPrepNodes]) {
  lds += (uint32_t)(v0 & (kRingNodes - 1)) * kSlotBytes;
  const uint64_t some = __ballot(far != 0u);
  if (some & 0xFFFF0000u) {
    uint32_t y[kPrepNodes];
#pragma unroll
    for (int i = 0; i < kPrepNodes; ++i) y[i] = load_r(b, rl(far, 16 + i));
#pragma unroll
    for (int i = 0; i < kPrepNodes; ++i) x[i] |= y[i];
  }
#pragma unroll
  for (int i = 0; i < kPrepNodes; ++i) {
    lds_put(lds, kSlotNeed * kSlotBytes + kSlotBytes * i, s1_of(in.s[i], in.next[i]) | x[i]);
    lds_put(lds, kSlotS * kSlotBytes + kSlotBytes * i, in.s[i]);
  }
  for (uint64_t more = some >> 48; more; more &= more - 1) {
    const int i = __builtin_ctzll(more);
    const uint32_t e0 = rl(far, 32 + i), e1 = e0 + rl(far, 48 + i);
    uint32_t acc = 0;
    for (uint32_t e = e0; e < e1; e += 8) {
      uint32_t y[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) y[k] = load_r(b, a.far_more[min(e + k, e1 - 1)]);
#pragma unroll
      for (int k = 0; k < 8; ++k) acc |= y[k];
    }
    const uint32_t o = (uint32_t)(kSlotNeed + i) * kSlotBytes;
    lds_put(lds, o, lds_get(lds, o) | acc);
  }
}

// R of a chunk's nodes from what each needs (its prepared word and its near
// users' R) and its S word: uses within the chunk pass through registers. kTop:
// the tile's own block, nodes 32 T + i, 32 T + i + 1, ...: stages below node v
// compute nothing at v, stage v computes it.
template <bool kTop>
__device__ __forceinline__ void decide(const uint32_t (&need)[4], const uint32_t (&s)[4], uint32_t flags, int i,
                                       int nodes, uint32_t (&R)[4]) {
  const auto use = [&](int bit) { return (uint32_t)((int32_t)(flags << (31 - bit)) >> 31); };
  const auto settle = [&](int j, uint32_t x) {
    const uint32_t r = x & ~s[j];
    return kTop ? (r & (~0u << (i + j))) | (i + j < nodes ? 1u << (i + j) : 0u) : r;
  };
  R[3] = settle(3, need[3]);
  R[2] = settle(2, need[2] | (R[3] & use(0)));
  R[1] = settle(1, need[1] | (R[3] & use(1)) | (R[2] & use(3)));
  R[0] = settle(0, need[0] | (R[3] & use(2)) | (R[2] & use(4)) | (R[1] & use(5)));
}

// The block's chunks from the top down. blk: LDS of this lane's column, from
// the block's ring slots on; r_off: the block's R tile byte offset.
template <int kNear, bool kTop>
__device__ __forceinline__ void decide_block(const TileBufs& b, lds_char* lds, lds_char* blk, uint32_t r_off,
                                             const uint32_t (&d)[kDescVecs], int nodes) {
  uint32_t need[kTile / 4][4], s[kTile / 4][4];
#pragma unroll
  for (int c = kTile / 4 - 1; c >= 0; --c)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      need[c][j] = lds_get(blk, (uint32_t)(kSlotNeed + 4 * c + j) * kSlotBytes);
      s[c][j] = lds_get(blk, (uint32_t)(kSlotS + 4 * c + j) * kSlotBytes);
    }
#pragma unroll
  for (int c = kTile / 4 - 1; c >= 0; --c) {
    const uint32_t dc = d[c / 2];
    const int dl = kDescDwords * (c & 1);
    uint32_t u[4][kNear], R[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < kNear; ++k) u[j][k] = lds_get(lds, rl(dc, dl + 4 * j + k));
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < kNear; ++k) need[c][j] |= u[j][k];
    decide<kTop>(need[c], s[c], rl(dc, dl + 16), 4 * c, nodes, R);
#pragma unroll
    for (int j = 0; j < 4; ++j) lds_put(blk, (uint32_t)(4 * c + j) * kSlotBytes, R[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_buffer_store_b32(R[j], b.r, (int)b.vo + kSlotBytes * j, (int)(r_off + node_off(4 * c)), 0);
  }
}
// The same for any number of near users.
template <bool kTop>
__device__ __forceinline__ void decide_block_any(const ClosureArgs& a, const TileBufs& b, lds_char* lds, lds_char* blk,
                                                 uint32_t r_off, uint32_t (&d)[kDescVecs], int nodes) {
#pragma unroll 1
  for (int c = kTile / 4 - 1; c >= 0; --c) {
    const uint32_t dc = d[kDescVecs - 1];
    const int dl = kDescDwords * (c & 1);
    lds_char* ch = blk + 4 * c * kSlotBytes;
    uint32_t need[4], s[4], R[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      need[j] = lds_get(ch, (uint32_t)(kSlotNeed + j) * kSlotBytes);
      s[j] = lds_get(ch, (uint32_t)(kSlotS + j) * kSlotBytes);
#pragma unroll
      for (int k = 0; k < 4; ++k) need[j] |= lds_get(lds, rl(dc, dl + 4 * j + k));
      const uint32_t e0 = rl(dc, dl + 17 + 2 * j), e1 = e0 + rl(dc, dl + 18 + 2 * j);
      for (uint32_t e = e0; e < e1; ++e) need[j] |= lds_get(lds, a.near_more[e]);
    }
    decide<kTop>(need, s, rl(dc, dl + 16), 4 * c, nodes, R);
#pragma unroll
    for (int j = 0; j < 4; ++j) lds_put(ch, (uint32_t)j * kSlotBytes, R[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_buffer_store_b32(R[j], b.r, (int)b.vo + kSlotBytes * j, uniform((int)(r_off + node_off(4 * c))), 0);
    if (!(c & 1)) {
#pragma unroll
      for (int k = kDescVecs - 1; k > 0; --k) d[k] = d[k - 1];
    }
  }
}
template <bool kTop>
__device__ __forceinline__ void decide_block(const ClosureArgs& a, const TileBufs& b, lds_char* lds, int nb,
                                             uint32_t (&d)[kDescVecs]) {
  lds_char* blk = lds + (nb & 1) * kTile * kSlotBytes;
  const uint32_t r_off = (uint32_t)uniform((int)(kRBase + node_off(kTile * nb)));
  const int nodes = a.t.n - kTile * nb;
  const uint32_t flags = rl(d[0], 16);
  if (flags & kBlockMany)
    decide_block_any<kTop>(a, b, lds, blk, r_off, d, nodes);
  else if (flags & kBlockNear4)
    decide_block<4, kTop>(b, lds, blk, r_off, d, nodes);
  else if (flags & kBlockNear3)
    decide_block<3, kTop>(b, lds, blk, r_off, d, nodes);
  else
    decide_block<2, kTop>(b, lds, blk, r_off, d, nodes);
}

// Barrier between phases. What the deciding wave wrote, to LDS and to the R
// tile, is read by the others after it; those write LDS only, and keep their
// loads for the next block in flight.
__device__ __forceinline__ void phase_end_decide() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void phase_end_prep() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__global__ void __launch_bounds__(kWave*(1 + kPrep)) ckm_closure_kernel(ClosureArgs a) {
  __shared__ uint32_t slots[kClosureSlots * kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = uniform((int)threadIdx.x / kWave);
  const int tile = a.t.tiles - 1 - (int)blockIdx.y;   // the longest scans start first
  const TileBufs b(a.t, blockIdx.x, tile, lane);
  lds_char* lds = (lds_char*)&slots[lane];
  if (wave == 0) {
    lds_put(lds, kRingEmpty * kSlotBytes, 0u);
    for (int i = 0; i < kRingNodes; ++i) lds_put(lds, (uint32_t)i * kSlotBytes, 0u);
    __builtin_amdgcn_raw_buffer_store_b32(0u, b.r, (int)b.vo, 0, 0);   // the empty word
  }
  if (wave > 0) {
    // phase p prepares block tile - p; blocks tile - p + 2 and up are decided
    const uint32_t* fars = a.far + kWave * (wave - 1) + lane;
    int v0 = kTile * tile + kPrepNodes * (wave - 1);
    const uint32_t* descs = a.desc + (kDescVecs / kPrep) * kWave * (wave - 1) + lane;
    uint32_t far = fars[(size_t)tile * (kPrep * kWave)], d[kDescVecs / kPrep];
#pragma unroll
    for (int i = 0; i < kDescVecs / kPrep; ++i) d[i] = descs[(size_t)(tile * kDescVecs + i) * kWave];
    PrepIn in;
    prep_load(b, v0, in);
    phase_end_prep();
    for (int p = 0; p <= tile; ++p, v0 -= kTile) {
#pragma unroll
      for (int i = 0; i < kDescVecs / kPrep; ++i)
        lds_put(lds, (uint32_t)(kSlotDesc + kDescVecs * ((tile - p) & 1) + kDescVecs / kPrep * (wave - 1) + i) * kSlotBytes,
                d[i]);
      const PrepIn now = in;
      const uint32_t far_now = far;
      // loads return in order: this block's before the next one's
      uint32_t x[kPrepNodes];
#pragma unroll
      for (int i = 0; i < kPrepNodes; ++i) x[i] = load_r(b, rl(far, i));
      if (p < tile) {
        far = fars[(size_t)(tile - p - 1) * (kPrep * kWave)];
#pragma unroll
        for (int i = 0; i < kDescVecs / kPrep; ++i) d[i] = descs[(size_t)((tile - p - 1) * kDescVecs + i) * kWave];
        prep_load(b, v0 - kTile, in);
      }
      prep_store(a, b, lds, v0, now, far_now, x);
      phase_end_prep();
    }
    phase_end_prep();
  } else {
    phase_end_decide();
    // phase p decides block tile - p + 1
    for (int p = 0; p <= tile + 1; ++p) {
      if (p > 0) {
        const int nb = tile - p + 1;
        uint32_t d[kDescVecs];
#pragma unroll
        for (int i = 0; i < kDescVecs; ++i) d[i] = lds_get(lds, (uint32_t)(kSlotDesc + kDescVecs * (nb & 1) + i) * kSlotBytes);
        if (nb == tile)
          decide_block<true>(a, b, lds, nb, d);
        else
          decide_block<false>(a, b, lds, nb, d);
      }
      phase_end_decide();
    }
  }
  if (a.h.nhub) {
    const auto out = HubBuf(a.t, a.h, tile, blockIdx.x).buf;
    for (int hub = wave; hub < a.h.nhub; hub += 1 + kPrep) hub_words(b, a.h, out, hub);
  }
}

// ---------------------------------------------------------------------------
// Simulate: the U recurrence (Section 4.4) and the cost (Section 4.3), one
// wave per (group, 8 stages of a tile, part of the tile's records). Before
// node v is computed the memory is U_{t,0} + U; computing it adds M_v (the
// peak is taken there), then the dependencies that FREE releases after it
// leave. All sums are binary64 integers below 2^53, exact in any order; a
// wave's stage j counts U in units of 2^(j - 1074), so that its bit of a word
// is the unit itself (denormals are exact and run at full rate). The bound is
// vector issue (per record and stage four ANDs, four FMAs and a maximum), then
// the latency of a record's words, hidden by four waves per SIMD.
// Measured: n = 1009, K = 1024: 158 us (its VALU instructions at 39.3 T lane
// operations/s 138 us), K = 512 105 us, one group 73 us; n = 4001, K = 4096: 10.2 ms.
// One kernel for closure and simulation, a stage to a wave: 440 us and 75 ms.
struct SimArgs {
  TileArgs t;
  HubArgs h;                        // and the pairs of the launch
  int32_t K, g0;                    // g0: the first group of the pass
  double base;                      // M_in + 2 M_param
  cptr<u64x4> ops;                  // SimOps
  cptr<u32x8> refs;                 // SimRefs
  cptr<int32_t> tile_rec;
  cptr<int32_t> users;              // the graph's users lists
  int64_t* __restrict__ peak;
  int64_t* __restrict__ cost;
};

struct SimStages8 {
  double U[8], top[8], U0[8];       // relative to the stage's start; its highest value; the start
};

// One record's masked updates of eight stages, whose bits are b0 .. b7 of the
// words: U0 += S M, U += R M, the peak, U -= F M0, U -= G M1. Each takes its bit
// into the low word of a binary64 whose high word is 0. Zero sizes (absent
// dependencies, records past a node's first) change nothing and are passed by.
#define CKM_SIM_FMA(acc, i0, i1, b0, b1, W, Msz)                                     \
  "v_and_b32 v8, " b0 ", %[" W "]\n\tv_and_b32 v10, " b1 ", %[" W "]\n\t"            \
  "v_fma_f64 %[" acc i0 "], v[8:9], " Msz ", %[" acc i0 "]\n\t"                      \
  "v_fma_f64 %[" acc i1 "], v[10:11], " Msz ", %[" acc i1 "]\n\t"
#define CKM_SIM_ADD(i0, i1, b0, b1)                  \
  CKM_SIM_FMA("z", i0, i1, b0, b1, "S", "%[M]")      \
  CKM_SIM_FMA("u", i0, i1, b0, b1, "R", "%[M]")      \
  "v_max_f64 %[t" i0 "], %[t" i0 "], %[u" i0 "]\n\t" \
  "v_max_f64 %[t" i1 "], %[t" i1 "], %[u" i1 "]\n\t"
#define CKM_SIM_FREE0(i0, i1, b0, b1) CKM_SIM_FMA("u", i0, i1, b0, b1, "F", "-%[M0]")
#define CKM_SIM_FREE1(i0, i1, b0, b1) CKM_SIM_FMA("u", i0, i1, b0, b1, "G", "-%[M1]")
#define CKM_SIM_LOW(X) X("0", "1", "1", "2") X("2", "3", "4", "8") X("4", "5", "16", "32") X("6", "7", "64", "0x80")
#define CKM_SIM_HIGH(X) \
  X("0", "1", "0x100", "0x200") X("2", "3", "0x400", "0x800") X("4", "5", "0x1000", "0x2000") X("6", "7", "0x4000", "0x8000")
#define CKM_SIM_RECORD(EACH, x)                                                                                \
  asm("v_mov_b32 v9, 0\n\tv_mov_b32 v11, 0\n\t"                                                               \
      "s_cmp_eq_u64 %[M], 0\n\ts_cbranch_scc1 .Lsim_free%=\n\t" EACH(CKM_SIM_ADD)                            \
      ".Lsim_free%=:\n\t" EACH(CKM_SIM_FREE0)                                                                 \
      "s_cmp_eq_u64 %[M1], 0\n\ts_cbranch_scc1 .Lsim_done%=\n\t" EACH(CKM_SIM_FREE1) ".Lsim_done%=:"         \
      : [u0] "+v"(x.U[0]), [u1] "+v"(x.U[1]), [u2] "+v"(x.U[2]), [u3] "+v"(x.U[3]), [u4] "+v"(x.U[4]),         \
        [u5] "+v"(x.U[5]), [u6] "+v"(x.U[6]), [u7] "+v"(x.U[7]), [t0] "+v"(x.top[0]), [t1] "+v"(x.top[1]),     \
        [t2] "+v"(x.top[2]), [t3] "+v"(x.top[3]), [t4] "+v"(x.top[4]), [t5] "+v"(x.top[5]),                    \
        [t6] "+v"(x.top[6]), [t7] "+v"(x.top[7]), [z0] "+v"(x.U0[0]), [z1] "+v"(x.U0[1]), [z2] "+v"(x.U0[2]),  \
        [z3] "+v"(x.U0[3]), [z4] "+v"(x.U0[4]), [z5] "+v"(x.U0[5]), [z6] "+v"(x.U0[6]), [z7] "+v"(x.U0[7])     \
      : [R] "v"(R), [S] "v"(S), [F] "v"(F), [G] "v"(G), [M] "s"(M), [M0] "s"(M0), [M1] "s"(M1)                 \
      : "v8", "v9", "v10", "v11", "scc")

template <int kSub>
__device__ __forceinline__ void sim_record(SimStages8 (&x)[kSub / 8], uint32_t R, uint32_t S, uint32_t F, uint32_t G,
                                           double M, double M0, double M1) {
  CKM_SIM_RECORD(CKM_SIM_LOW, x[0]);
  if constexpr (kSub > 8) CKM_SIM_RECORD(CKM_SIM_HIGH, x[1]);
}

// The words of a record: requested a record ahead.
struct SimIn {
  uint32_t R, S, s0, n0, s1, n1, u[2][4];
};

// kSub stages per wave; kSegs waves share the tile's records, and each part
// then counts from the memory that the parts before it leave.
template <int kSub, int kSegs>
__global__ void __launch_bounds__(kWave* kSegs) ckm_simulate_kernel(SimArgs a) {
  constexpr int kSubs = kTile / kSub;
  const int lane = threadIdx.x & (kWave - 1);
  const int seg = kSegs == 1 ? 0 : uniform((int)threadIdx.x / kWave);
  // blocks go to the 8 XCDs in turn; those that read one tile come 8 apart and
  // share an L2
  const int id = blockIdx.x, sub = (id >> 3) % kSubs, item = (id / (8 * kSubs)) * 8 + (id & 7);
  if (item >= a.h.items) return;
  int tile, group;
  tile_of(a.t, a.h.item0 + item, tile, group);
  if (kTile * tile + kSub * sub >= a.t.n) return;   // no stages
  TileBufs b(a.t, group, tile, lane);
  __amdgpu_buffer_rsrc_t hubs = b.r;
  uint32_t hub_words = 0;
  if (a.h.at) {
    const HubBuf h(a.t, a.h, tile, group);
    hubs = h.buf;
    hub_words = h.words;
  }
  if (sub != kSubs - 1) b.vo_next = kPastEnd;   // only the last stages reach into the next tile
  const int recs = a.tile_rec[tile];
  const int r0 = (int)((int64_t)recs * seg / kSegs), r1 = (int)((int64_t)recs * (seg + 1) / kSegs);
  const uint32_t sh = (uint32_t)(kSub * sub);
  // whole words: loads of a byte or half per lane take the cache as many cycles
  // as eight words
  const auto word_s = [&](uint32_t off) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(b.s, (int)b.vo, (int)off, 0); };
  const auto word_n = [&](uint32_t off) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(b.next, (int)b.vo_next, (int)off, 0); };

  SimStages8 x[kSub / 8];
#pragma unroll
  for (int h = 0; h < kSub / 8; ++h)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      x[h].U[j] = 0.0;
      x[h].top[j] = 0.0;   // no stage's peak is below its start
      x[h].U0[j] = 0.0;
    }
  uint64_t cost_lo = 0, cost_hi = 0;
  SimIn in;
  const auto load_words = [&](const u32x8& f) {
    const auto half = [&](int k) { return k % 2 ? f[k / 2] >> 16 : f[k / 2] & 0xFFFFu; };
    const auto slot = [&](int k) { return half(k) * (uint32_t)kSlotBytes; };
    // the record read past a tile's last belongs to the next tile's first node:
    // its words are in the memory after the tile's, and are not used
    in.R = __builtin_amdgcn_raw_buffer_load_b32(b.r, (int)b.vo, (int)(slot(0) + kRBase), 0);
    in.S = word_s(slot(0));
    in.s0 = word_s(slot(1));
    in.n0 = word_n(slot(1));
    in.s1 = word_s(slot(2));
    in.n1 = word_n(slot(2));
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int k = 0; k < 4; ++k) in.u[d][k] = k < 2 ? load_r(b, slot(4 + 4 * d + k)) : 0u;
    const uint32_t more = f[1] >> 16;
    if (more) {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        if (more & kMoreThird << d) in.u[d][2] = load_r(b, slot(6 + 4 * d));
        if (more & kMoreFourth << d) in.u[d][3] = load_r(b, slot(7 + 4 * d));
        if (more & kMoreHub << d) {
          const uint32_t h = half(7 + 4 * d);   // a word that the tile does not make covers nothing in it
          in.u[d][3] = __builtin_amdgcn_raw_buffer_load_b32(hubs, (int)b.vo, (int)(h <= hub_words ? h * kSlotBytes : 0u), 0);
        }
        if (more & kMoreList << d) {
          const uint32_t e1 = f[6 + d] + half(6 + 4 * d);
          for (uint32_t e = f[6 + d]; e < e1; e += 4) {
            uint32_t y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) y[k] = load_r(b, kRBase + node_off(a.users[min(e + k, e1 - 1)]));
#pragma unroll
            for (int k = 0; k < 4; ++k) in.u[d][2] |= y[k];
          }
        }
      }
    }
  };
  if (r0 < r1) {
    u32x8 f = a.refs[r0];
    load_words(f);
    f = a.refs[r0 + 1];
    for (int r = r0; r < r1; ++r) {
      const u32x8 ahead = a.refs[r + 2];
      const u64x4 now = a.ops[r];
      uint32_t R = in.R >> sh, S = in.S >> sh,
               F = (in.R & ~(s1_of(in.s0, in.n0) | in.u[0][0] | in.u[0][1] | in.u[0][2] | in.u[0][3])) >> sh,
               G = (in.R & ~(s1_of(in.s1, in.n1) | in.u[1][0] | in.u[1][1] | in.u[1][2] | in.u[1][3])) >> sh;
      asm volatile("" : "+v"(R), "+v"(S), "+v"(F), "+v"(G));   // before the next loads
      load_words(f);   // past the part's end they are not used
      f = ahead;
      const uint32_t c = (uint32_t)__builtin_popcount(R & ((1u << kSub) - 1u));
      cost_lo += (uint64_t)c * (uint32_t)now[3];
      cost_hi += (uint64_t)c * (uint32_t)(now[3] >> 32);
      sim_record<kSub>(x, R, S, F, G, __builtin_bit_cast(double, (uint64_t)now[0]),
                       __builtin_bit_cast(double, (uint64_t)now[1]), __builtin_bit_cast(double, (uint64_t)now[2]));
    }
  }
  const int k = (a.g0 + group) * kWave + lane;
  const uint64_t cost = cost_lo + (cost_hi << 32);
  if (k < a.K && cost) atomicAdd(reinterpret_cast<unsigned long long*>(a.cost) + k, (unsigned long long)cost);
  // the parts' sums meet in LDS, eight stages at a time; each wave joins some
  // of the stages
  __shared__ double cell[kSegs][16][kWave];
  constexpr int kMine = 8 / kSegs;
  double peak = 0.0;   // above the base
#pragma unroll
  for (int h = 0; h < kSub / 8; ++h) {
    if (h) __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      cell[seg][j][lane] = x[h].U[j];
      cell[seg][8 + j][lane] = x[h].top[j];
    }
    __syncthreads();
    double top[kMine], U0[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int j = kMine * seg + i;
      double before = 0.0;
      top[i] = 0.0;
#pragma unroll
      for (int s = 0; s < kSegs; ++s) {
        top[i] = fmax(top[i], before + cell[s][8 + j][lane]);
        before += cell[s][j][lane];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) cell[seg][j][lane] = x[h].U0[j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int j = kMine * seg + i, bit = 8 * h + j;
      U0[i] = 0.0;
#pragma unroll
      for (int s = 0; s < kSegs; ++s) U0[i] += cell[s][j][lane];
      if (kTile * tile + kSub * sub + bit < a.t.n) peak = fmax(peak, ldexp(U0[i] + top[i], 1074 - bit));
    }
  }
  if (k < a.K) atomicMax(reinterpret_cast<long long*>(a.peak) + k, (long long)(a.base + peak));
}

}  // namespace

// ---------------------------------------------------------------------------
template <int kSub, int kSegs>
static void launch_simulate(const SimArgs& s, hipStream_t stream) {
  const int64_t items = ((int64_t)s.h.items + 7) / 8 * 8;
  hipLaunchKernelGGL((ckm_simulate_kernel<kSub, kSegs>), dim3((unsigned)(items * (kTile / kSub))), dim3(kWave * kSegs),
                     0, stream, s);
}

// (group, tile) pairs from which the chip is full with fewer waves per pair:
// with few, eight stages a wave and eight parts a tile shorten each wave's run
// over the records; from kSimWide on sixteen stages read each word once for
// twice the stages; from kSimFull on four parts leave half the sums to join.
// Measured, whole call, 8 stages and 8 parts / 16 and 8 / 16 and 4:
// n = 1009: 256 pairs (K = 512) 227 / 236 / 267 us; 288 242 / 249; 320 260 / 261;
// 352 275 / 271; 512 357 / 323 / 345; 704 - / 418 / 424; 768 - / 447 / 445; 1024 - / 562 / 547.
// n = 747: 264 pairs 242 / 244 / 280; 288 250 / 251; 312 263 / 258; 384 296 / 274 / 295;
// 672 - / 381 / 383; 768 - / 415 / 409. n = 337: 264 pairs 95 / 96; 308 104 / 103; 352 112 / 106.
// On graphs of up to kSimFewTiles tiles, whose waves have few records, four parts are
// enough from kSimFew pairs on. Measured, 8 and 8 / 8 and 4 / 16 and 8: n = 101: 128 pairs
// 35.8 / 37.1 us; 192 44.9 / 43.6; 256 48.8 / 45.9 / 46.9; n = 169: 192 pairs 55.0 / 55.0; 288
// 68.5 / 65.9 / 67.1; 384 78 / 74 / 72;
// n = 337: 176 pairs 78.3 / 81.4.
constexpr int64_t kSimWide = 304, kSimFull = 736, kSimFew = 176;
constexpr int32_t kSimFewTiles = 6;

// Rounds of eight users (all hubs together) up to which the closure's waves make
// the hub words after their last block: a launch costs more than a few rounds.
// Measured, whole call, in the closure / in a launch: 3 rounds (n = 61, K = 64) 30.6 /
// 32.4 us; 9 (n = 401) 95.4 / 96.3, K = 3000 208 / 210; 20 (n = 747) 161.8 / 160.3, K = 3000
// 545 / 552; 42 (n = 1601) 359 / 356; 97 (n = 150, six users per node) 93 / 78.
constexpr int32_t kHubInline = 12;

hipError_t launch_tiles(const ckm_graph& g, const Layout& L, int32_t K, int32_t g0, int32_t groups, char* work,
                        hipStream_t stream) {
  ClosureArgs c;
  c.t.n = g.n;
  c.t.tiles = (g.n + kTile - 1) / kTile;
  c.t.groups = groups;
  c.t.s_bytes = stile_off(c.t.tiles);
  c.t.r_bytes = rtile_off(c.t.tiles);
  c.t.stiles = work + L.rows_off;
  c.t.rtiles = work + L.rrows_off;
  c.desc = g.tile.d_desc;
  c.far = g.tile.d_far;
  c.far_more = (cptr<uint32_t>)g.tile.d_far_more;
  c.near_more = (cptr<uint32_t>)g.tile.d_near_more;
  SimArgs s;
  s.t = c.t;
  s.K = K;
  s.g0 = g0;
  s.base = (double)g.base;
  s.ops = (cptr<u64x4>)g.tile.d_ops;
  s.refs = (cptr<u32x8>)g.tile.d_refs;
  s.tile_rec = (cptr<int32_t>)g.tile.d_tile_rec;
  s.users = (cptr<int32_t>)g.d_user_idx;
  s.peak = reinterpret_cast<int64_t*>(work + L.part_peak_off);
  s.cost = reinterpret_cast<int64_t*>(work + L.part_cost_off);
  const int32_t pairs = groups * c.t.tiles;
  HubArgs h = {};
  if (g.tile.nhub) {
    h.ptr = (cptr<int32_t>)g.tile.d_hub_ptr;
    h.users = (cptr<HubUser>)g.tile.d_hub;
    h.at = (cptr<uint32_t>)g.tile.d_hub_at;
    h.buf = work + L.hub_off;
    h.nhub = g.tile.nhub;
  }
  s.h = c.h = h;
  const bool inlined = g.tile.hub_rounds <= kHubInline && (size_t)groups * 256 * (h.nhub ? g.tile.hub_at[0] : 0) <= L.hub_bytes;
  if (!inlined) c.h.nhub = 0;
  hipLaunchKernelGGL(ckm_closure_kernel, dim3(groups, c.t.tiles), dim3(kWave * (1 + kPrep)), 0, stream, c);
  // the simulation in one launch, or as many as the room for hub words asks for
  for (; s.h.item0 < pairs; s.h.item0 += s.h.items) {
    s.h.items = pairs - s.h.item0;
    if (!inlined) {
      size_t room = L.hub_bytes;   // holds the largest pair at least
      int32_t i = s.h.item0, fit = 1;
      for (; i < pairs && fit; i += fit) {
        const size_t bytes = hub_pair_bytes(g.tile, c.t.tiles - 1 - i / groups);
        fit = (int32_t)std::min<size_t>(groups - i % groups, room / bytes);
        room -= fit * bytes;
      }
      s.h.items = i - s.h.item0;
      hipLaunchKernelGGL(ckm_hub_kernel, dim3(s.h.items, h.nhub), dim3(kWave), 0, stream, s.t, s.h);
    }
    if (s.h.items >= kSimFull)
      launch_simulate<16, 4>(s, stream);
    else if (s.h.items >= kSimWide)
      launch_simulate<16, 8>(s, stream);
    else if (s.h.items >= kSimFew && c.t.tiles <= kSimFewTiles)
      launch_simulate<8, 4>(s, stream);
    else
      launch_simulate<8, 8>(s, stream);
  }
  return hipGetLastError();
}

}  // namespace ckm

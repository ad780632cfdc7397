// Event path (see ckm_events.h): the closure kernel, which decides R and the
// FREE terms of every (candidate, stage, node), the simulate kernel, which
// runs the U recurrence on them, and the gather of the best candidate's R.
//
// The two halves of the work want different layouts. Decisions are bits:
// with 64 candidates to a word and a stage to a lane, one instruction decides
// a node for 64 x 64 (candidate, stage) pairs. The sums are binary64 per
// (candidate, stage): with a candidate to a lane, a word is an execution mask
// and a masked update costs one vector instruction (and a scalar move). The
// words go from the one layout to the other through memory: the closure
// writes them by vector stores, lane = stage, and the simulate kernel, launched
// after it, reads them by scalar loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "ckm_events.h"
#include "ckm_internal.h"

namespace ckm {
namespace {

template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint64_t u64x8 __attribute__((ext_vector_type(8)));
typedef double f64x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) uint64_t lds_u64;

constexpr int kBufWord3 = 0x00020000;         // raw byte-addressed buffer
constexpr uint32_t kOutside = 0xC0000000u;    // past any buffer here: loads give 0, stores are dropped

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ uint64_t word(uint32_t lo, uint32_t hi) { return (uint64_t)lo | (uint64_t)hi << 32; }

// ---------------------------------------------------------------------------
// Closure: one wave per (group, tile of 64 stages), lane = stage.
struct ClosureArgs {
  int32_t n, pairs, tlo, thi, g0;   // tiles tlo .. thi - 1 of the groups from g0
  uint32_t row0;                    // the tiles' first event record in a group
  uint32_t s_bytes;                 // bytes of one group's mask rows
  uint32_t ev_bytes;                // bytes of one group's event records in the chunk
  uint32_t far_bytes;               // bytes of one wave's far accumulators
  int32_t npins;
  const uint64_t* srows;            // mask rows, group-major
  char* events;                     // event records, group-major from group g0
  char* far;                        // far accumulators, per (group - g0, tile)
  const uint32_t* desc;             // chunks x 64 dwords
  cptr<uint32_t> extra;
  cptr<uint32_t> row_off;
  cptr<int32_t> tile_chunk;
  cptr<int32_t> pins;
  const int32_t* best_k;            // not NULL: only the group of this candidate (none when negative)
};

// A record whose release words are still on their way from LDS: they are
// taken up, and the record stored, one node later.
struct Pending {
  uint64_t R, S, a0, a1, a2, a3;
  uint32_t vo, vo2;                 // per-lane byte offset of the row (kOutside: not stored)
  uint32_t so;                      // byte offset of the record in the row
  uint32_t flags, fs;               // descriptor words 1 and 2
};

struct Closure {
  __amdgpu_buffer_rsrc_t rs, re, rf, rd;   // S rows, events, far accumulators, descriptors
  lds_char* lds;                    // this lane's column
  uint32_t lane, r0, r1, row;       // byte offsets: S rows t and t + 1, event row t
  int32_t t, vstart;
  uint32_t len;                     // records of the lane's row (0: no such stage)
  uint64_t pre, Rprev;
  Pending p;

  __device__ __forceinline__ uint64_t at(uint32_t off) const { return *(lds_u64*)(lds + off); }
  __device__ __forceinline__ void put(uint32_t off, uint64_t x) const { *(lds_u64*)(lds + off) = x; }
  __device__ __forceinline__ uint64_t lds_or(uint32_t off, uint64_t x) const {
    return __hip_atomic_fetch_or((lds_u64*)(lds + off), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  __device__ __forceinline__ uint32_t load_desc(int c) const {
    return __builtin_amdgcn_raw_buffer_load_b32(rd, (int)(4u * lane), c > 0 ? 256 * c : 0, 0);
  }
  // S row words of the four nodes of chunk c
  __device__ __forceinline__ void load_s(uint32_t r, int c, uint64_t (&x)[4]) const {
    const auto a = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)r, 32 * c, 0);
    const auto b = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)r + 16, 32 * c, 0);
    x[0] = word(a[0], a[1]);
    x[1] = word(a[2], a[3]);
    x[2] = word(b[0], b[1]);
    x[3] = word(b[2], b[3]);
  }
  __device__ __forceinline__ uint64_t load_s1(uint32_t node) const {
    const auto a = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)r1, (int)(8u * node), 0);
    return word(a[0], a[1]);
  }
  __device__ __forceinline__ uint64_t load_far(uint32_t slot) const {
    const auto a = __builtin_amdgcn_raw_buffer_load_b64(rf, (int)(8u * lane), (int)(slot * kEvSlotBytes), 0);
    return word(a[0], a[1]);
  }
  __device__ __forceinline__ void store_far(uint32_t slot, uint64_t x) const {
    const u32x2 d = {(uint32_t)x, (uint32_t)(x >> 32)};
    __builtin_amdgcn_raw_buffer_store_b64(d, rf, (int)(8u * lane), (int)(slot * kEvSlotBytes), 0);
  }
  // The accumulator of a far dependency: in device memory when a far user
  // above has been decided in this scan, else S_{t+1}.
  __device__ __forceinline__ uint64_t far_acc(uint32_t node, uint32_t up, uint32_t slot) const {
    return (int32_t)up <= vstart ? load_far(slot) : load_s1(node);
  }
  __device__ __forceinline__ void store_record(uint32_t vo, uint32_t so, uint64_t R, uint64_t S, uint64_t f0,
                                               uint64_t f1) const {
    const u32x4 a = {(uint32_t)R, (uint32_t)(R >> 32), (uint32_t)S, (uint32_t)(S >> 32)};
    const u32x4 b = {(uint32_t)f0, (uint32_t)(f0 >> 32), (uint32_t)f1, (uint32_t)(f1 >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(a, re, (int)vo, (int)so, 0);
    __builtin_amdgcn_raw_buffer_store_b128(b, re, (int)vo + 16, (int)so, 0);
  }
  // Stores the pending record (its release words, and the accumulators of far
  // dependencies).
  __device__ __forceinline__ void finish() {
    store_record(p.vo, p.so, p.R, p.S, p.R & ~p.a0, p.R & ~p.a1);
    if (p.flags & (kEvSecond | kEvFar0 | kEvFar1)) {
      if (p.flags & kEvSecond) store_record(p.vo2, p.so + kEvRecBytes, 0, 0, p.R & ~p.a2, p.R & ~p.a3);
      if (p.flags & kEvFar0) store_far(p.fs & 0xFFFFu, p.a0 | p.R);
      if (p.flags & kEvFar1) store_far(p.fs >> 16, p.a1 | p.R);
    }
  }
  __device__ __forceinline__ void nothing_pending() {
    p.vo = p.vo2 = kOutside;
    p.flags = 0;
  }
};

__device__ __forceinline__ uint32_t rl(uint32_t w, int lane) { return __builtin_amdgcn_readlane(w, lane); }

// The accumulators of chunk c's far slots (descriptors d), for its staging
// slots: x[2 j + s].
__device__ __forceinline__ void far_issue(const Closure& s, uint32_t d, uint64_t (&x)[8]) {
  if (!(rl(d, 15) & kEvChunkFar)) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t f = rl(d, 16 * j + 1);
    if ((f & (kEvFar0 | kEvSync0)) == kEvFar0) {
      const uint32_t w = rl(d, 16 * j + 4);
      x[2 * j] = s.far_acc(w & 0xFFFFu, w >> 16, rl(d, 16 * j + 2) & 0xFFFFu);
    }
    if ((f & (kEvFar1 | kEvSync1)) == kEvFar1) {
      const uint32_t w = rl(d, 16 * j + 5);
      x[2 * j + 1] = s.far_acc(w & 0xFFFFu, w >> 16, rl(d, 16 * j + 2) >> 16);
    }
  }
}
__device__ __forceinline__ void far_stage(const Closure& s, uint32_t d, const uint64_t (&x)[8]) {
  if (!(rl(d, 15) & kEvChunkFar)) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t f = rl(d, 16 * j + 1), o = rl(d, 16 * j);
    if ((f & (kEvFar0 | kEvSync0)) == kEvFar0) s.put(o & 0xFFFFu, x[2 * j]);
    if ((f & (kEvFar1 | kEvSync1)) == kEvFar1) s.put(o >> 16, x[2 * j + 1]);
  }
}

// Node 4c + J: its word R, then its dependencies' release words and
// accumulators. d: the chunk's descriptors; dn: the next chunk's. kTop: the
// node may be at or above the stage of some lane.
template <bool kTop, int J>
__device__ __forceinline__ void closure_node(const ClosureArgs& a, Closure& s, int c, uint32_t d, uint32_t dn,
                                             uint64_t S0, int32_t& rho) {
  const int v = 4 * c + J;
  const uint32_t f = rl(d, 16 * J + 1);
  const uint64_t fwd = (f & kEvOwnFwd) ? ~0ull : 0ull;
  uint64_t R = (s.pre | (s.Rprev & fwd)) & ~S0;
  if (kTop) {
    R = v == s.t ? ~0ull : v > s.t ? 0ull : R;
    S0 = v > s.t ? 0ull : S0;
    if (v >= a.n) R = 0ull;
  }
  const uint32_t more = f >> 16;
  const int32_t second = (f & kEvSecond) ? 1 : 0;
  rho -= 1 + second + (int32_t)more;
  if (__builtin_expect((f & (0xFFFF0000u | kEvSync0 | kEvSync1)) != 0u, 0)) {
    // records beyond the second, and far slots too close to the user above:
    // their accumulators are loaded here, after every store before
    s.finish();
    s.nothing_pending();
    const uint32_t first = rl(d, 16 * J + 3);
    for (int x = (int)more - 1; x >= 0; --x) {
      const auto e = *(cptr<u32x8>)(a.extra + (size_t)(first + (uint32_t)x) * kEvExtraDw);
      if (e[1] & kEvFar0) s.put(e[0] & 0xFFFFu, s.far_acc(e[3] & 0xFFFFu, e[4] & 0xFFFFu, e[2] & 0xFFFFu));
      if (e[1] & kEvFar1) s.put(e[0] >> 16, s.far_acc(e[3] >> 16, e[4] >> 16, e[2] >> 16));
      const uint64_t a0 = s.lds_or(e[0] & 0xFFFFu, R), a1 = s.lds_or(e[0] >> 16, R);
      const int32_t at = rho + 1 + second + x;
      const uint32_t vo = !kTop || (uint32_t)at < s.len ? s.row : kOutside;
      s.store_record(vo, (uint32_t)at * kEvRecBytes, 0, 0, R & ~a0, R & ~a1);
      if (e[1] & kEvFar0) s.store_far(e[2] & 0xFFFFu, a0 | R);
      if (e[1] & kEvFar1) s.store_far(e[2] >> 16, a1 | R);
    }
    if (f & kEvSync0) {
      const uint32_t w = rl(d, 16 * J + 4);
      s.put(rl(d, 16 * J) & 0xFFFFu, s.far_acc(w & 0xFFFFu, w >> 16, rl(d, 16 * J + 2) & 0xFFFFu));
    }
    if (f & kEvSync1) {
      const uint32_t w = rl(d, 16 * J + 5);
      s.put(rl(d, 16 * J) >> 16, s.far_acc(w & 0xFFFFu, w >> 16, rl(d, 16 * J + 2) >> 16));
    }
  }
  // the next node's accumulator, read before this node's updates (LDS works
  // in order): kEvOwnFwd says when they touch it
  s.pre = s.at(J > 0 ? rl(d, 16 * (J - 1) + 7) : rl(dn, 16 * 3 + 7));
  const uint32_t o = rl(d, 16 * J);
  const uint64_t a0 = s.lds_or(o & 0xFFFFu, R), a1 = s.lds_or(o >> 16, R);
  uint64_t a2 = 0, a3 = 0;
  if (f & kEvSecond) {
    const uint32_t o2 = rl(d, 16 * J + 8);
    a2 = s.lds_or(o2 & 0xFFFFu, R);
    a3 = s.lds_or(o2 >> 16, R);
  }
  s.finish();
  s.p.R = R;
  s.p.S = S0;
  s.p.a0 = a0;
  s.p.a1 = a1;
  s.p.a2 = a2;
  s.p.a3 = a3;
  s.p.vo = s.p.vo2 = s.row;
  if (kTop) {
    if ((uint32_t)rho >= s.len) s.p.vo = kOutside;
    if ((uint32_t)rho + 1 >= s.len) s.p.vo2 = kOutside;
  }
  s.p.so = (uint32_t)rho * kEvRecBytes;
  s.p.flags = f;
  s.p.fs = rl(d, 16 * J + 2);
  s.Rprev = R;
}

// Chunk c (descriptors d, S words s0); loads for the next chunk (descriptors
// dn) and for the ring entry of chunk c - 7 (descriptors de).
template <bool kTop>
__device__ __forceinline__ void closure_chunk(const ClosureArgs& a, Closure& s, int c, uint32_t& d, uint32_t& dn,
                                              uint32_t& de, uint64_t (&s0)[4]) {
  const int e = c - (kEvNear + 1);
  uint64_t s0n[4], ent[4], fx[8];
  s.load_s(s.r0, c > 0 ? c - 1 : 0, s0n);
  s.load_s(s.r1, e > 0 ? e : 0, ent);
  const uint32_t dnn = s.load_desc(c - 2), den = s.load_desc(e - 1);
  s.finish();   // its far accumulators are stored before the loads below
  s.nothing_pending();
  if (c > 0) far_issue(s, dn, fx);
  const bool entry = e >= 0 && (rl(de, 15) & kEvChunkEntry);
  if (entry) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w = rl(de, 16 * j + 6);
      if ((int32_t)(w >> 16) <= s.vstart) ent[j] = s.load_far(w & 0xFFFFu);
    }
  }
  int32_t rho = (int32_t)rl(d, kEvDescDw + 15);
  closure_node<kTop, 3>(a, s, c, d, dn, s0[3], rho);
  closure_node<kTop, 2>(a, s, c, d, dn, s0[2], rho);
  closure_node<kTop, 1>(a, s, c, d, dn, s0[1], rho);
  closure_node<kTop, 0>(a, s, c, d, dn, s0[0], rho);
  if (c > 0) far_stage(s, dn, fx);
  if (e >= 0) {
    if (entry) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (rl(de, 16 * j + 1) & kEvEntrySync) {
          s.finish();
          s.nothing_pending();
          const uint32_t w = rl(de, 16 * j + 6);
          if ((int32_t)(w >> 16) <= s.vstart) ent[j] = s.load_far(w & 0xFFFFu);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) s.put((uint32_t)((4 * e + j) & (kEvRing - 1)) * kEvSlotBytes, ent[j]);
  }
  d = dn;
  dn = dnn;
  de = den;
#pragma unroll
  for (int j = 0; j < 4; ++j) s0[j] = s0n[j];
}

__global__ void __launch_bounds__(kWave) ckm_closure_kernel(ClosureArgs a) {
  __shared__ uint64_t lds[kEvSlots * kWave];
  const int lane = threadIdx.x;
  const int tile = a.thi - 1 - (int)blockIdx.y;   // the longest scans start first
  int slot = blockIdx.x;                            // of the event and far arrays
  int group = a.g0 + slot;
  if (a.best_k) {
    const int bk = __builtin_amdgcn_readfirstlane(a.best_k[0]);
    if (bk < 0) return;
    group = bk / kWave;
  }
  Closure s;
  s.lane = lane;
  s.lds = (lds_char*)&lds[lane];
  s.t = kWave * tile + lane;
  s.rs = buffer(reinterpret_cast<const char*>(a.srows) + (size_t)group * a.s_bytes, a.s_bytes);
  s.re = buffer(a.events + (size_t)slot * a.ev_bytes, a.ev_bytes);
  s.rf = buffer(a.far + ((size_t)slot * (a.thi - a.tlo) + (tile - a.tlo)) * a.far_bytes, a.far_bytes);
  const int cT = a.tile_chunk[tile];
  s.rd = buffer(a.desc, (uint32_t)(cT + 1) * 256u);
  s.vstart = 4 * cT + 3;
  s.r0 = (uint32_t)(mrow_off(min(s.t, a.n)) * 8);
  s.r1 = (uint32_t)(mrow_off(min(s.t + 1, a.n)) * 8);
  const bool stage = s.t < 2 * a.pairs;
  s.row = stage ? (a.row_off[stage ? s.t : 0] - a.row0) * (uint32_t)kEvRecBytes : kOutside;
  s.len = stage ? a.row_off[(stage ? s.t : 0) + 1] - a.row_off[stage ? s.t : 0] : 0u;
  s.Rprev = 0;
  s.p.R = s.p.S = s.p.a0 = s.p.a1 = s.p.a2 = s.p.a3 = 0;
  s.p.so = s.p.fs = 0;
  s.nothing_pending();

  // the slots as they are before anything is decided: S_{t+1} everywhere
  uint32_t d = s.load_desc(cT), dn = s.load_desc(cT - 1), de = s.load_desc(cT - kEvNear - 1);
  s.put(kEvNone * kEvSlotBytes, ~0ull);
  for (int p = 0; p < a.npins; ++p) s.put((uint32_t)(kEvPin + p) * kEvSlotBytes, s.load_s1((uint32_t)a.pins[p]));
  for (int c = cT; c >= 0 && c >= cT - kEvNear; --c) {
    uint64_t x[4];
    s.load_s(s.r1, c, x);
#pragma unroll
    for (int j = 0; j < 4; ++j) s.put((uint32_t)((4 * c + j) & (kEvRing - 1)) * kEvSlotBytes, x[j]);
  }
  {
    uint64_t fx[8];
    far_issue(s, d, fx);
    far_stage(s, d, fx);
  }
  s.pre = s.at(rl(d, 16 * 3 + 7));
  uint64_t s0[4];
  s.load_s(s.r0, cT, s0);

  int c = cT;
  for (; c >= 16 * tile; --c) closure_chunk<true>(a, s, c, d, dn, de, s0);
  for (; c >= 0; --c) closure_chunk<false>(a, s, c, d, dn, de, s0);
  s.finish();
}

// ---------------------------------------------------------------------------
// Simulate: the U recurrence (Section 4.4) and the cost (Section 4.3) of the
// two stages of a pair, lane = candidate. Before node v is computed the
// memory is U; computing it adds M_v (the peak is taken there), then the
// dependencies that FREE releases after it leave. All sums are binary64
// integers below 2^53, exact in any order.
struct SimArgs {
  int32_t n, K, phi, g0;            // pairs below phi, from the top
  uint32_t row0;                    // as in ClosureArgs
  double base;                      // M_in + 2 M_param
  uint64_t ev_bytes;                // bytes of one group's event records in the chunk
  cptr<char> events;                // from group g0
  cptr<char> ops;
  cptr<uint32_t> row_off;
  int64_t* __restrict__ peak;
  int64_t* __restrict__ cost;
};

struct SimStage {
  double U, top, cost, U0;          // relative to the memory at the stage's start; its peak; cost; U_{t,0}
};

// One event record of both stages: words R, S, F0, F1 each, and the record's
// M_v, C_v and the sizes of its two dependencies. Each masked update is a
// scalar move into the execution mask and one vector instruction; the mask is
// full again at the end.
__device__ __forceinline__ void sim_record(SimStage& x, SimStage& y, uint64_t Rx, uint64_t Sx, uint64_t Fx0,
                                           uint64_t Fx1, uint64_t Ry, uint64_t Sy, uint64_t Fy0, uint64_t Fy1,
                                           double M, double C, double M0, double M1) {
  asm("s_mov_b64 exec, %[Sx]\n\t"
      "v_add_f64 %[Zx], %[Zx], %[M]\n\t"
      "s_mov_b64 exec, %[Sy]\n\t"
      "v_add_f64 %[Zy], %[Zy], %[M]\n\t"
      "s_mov_b64 exec, %[Rx]\n\t"
      "v_add_f64 %[Ux], %[Ux], %[M]\n\t"
      "v_add_f64 %[Cx], %[Cx], %[C]\n\t"
      "v_max_f64 %[Tx], %[Tx], %[Ux]\n\t"
      "s_mov_b64 exec, %[Ry]\n\t"
      "v_add_f64 %[Uy], %[Uy], %[M]\n\t"
      "v_add_f64 %[Cy], %[Cy], %[C]\n\t"
      "v_max_f64 %[Ty], %[Ty], %[Uy]\n\t"
      "s_mov_b64 exec, %[Fx0]\n\t"
      "v_add_f64 %[Ux], %[Ux], -%[M0]\n\t"
      "s_mov_b64 exec, %[Fy0]\n\t"
      "v_add_f64 %[Uy], %[Uy], -%[M0]\n\t"
      "s_mov_b64 exec, %[Fx1]\n\t"
      "v_add_f64 %[Ux], %[Ux], -%[M1]\n\t"
      "s_mov_b64 exec, %[Fy1]\n\t"
      "v_add_f64 %[Uy], %[Uy], -%[M1]\n\t"
      "s_mov_b64 exec, -1"
      : [Ux] "+v"(x.U), [Uy] "+v"(y.U), [Tx] "+v"(x.top), [Ty] "+v"(y.top), [Cx] "+v"(x.cost), [Cy] "+v"(y.cost),
        [Zx] "+v"(x.U0), [Zy] "+v"(y.U0)
      : [Rx] "s"(Rx), [Ry] "s"(Ry), [Sx] "s"(Sx), [Sy] "s"(Sy), [Fx0] "s"(Fx0), [Fy0] "s"(Fy0), [Fx1] "s"(Fx1),
        [Fy1] "s"(Fy1), [M] "s"(M), [C] "s"(C), [M0] "s"(M0), [M1] "s"(M1));
}

template <typename T>
__device__ __forceinline__ T sload(cptr<char> p, uint32_t off) {
  return *(cptr<T>)(p + off);
}

// kSegs waves share a pair, each a part of its records; their results are
// joined in order (a part's peak counts from the memory the parts before it
// leave).
template <int kSegs>
__global__ void __launch_bounds__(kWave* kSegs) ckm_simulate_kernel(SimArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int seg = kSegs == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int pair = a.phi - 1 - (int)blockIdx.y;   // the longest rows start first
  const uint32_t o0 = a.row_off[2 * pair] - a.row0, o1 = a.row_off[2 * pair + 1] - a.row0;
  const uint32_t two = (o1 - o0) / 2;               // records in twos
  const uint32_t b0 = two * (uint32_t)seg / kSegs, b1 = two * (uint32_t)(seg + 1) / kSegs;
  const cptr<char> ev = a.events + (uint64_t)blockIdx.x * a.ev_bytes;
  const cptr<char> px = ev + (uint64_t)o0 * kEvRecBytes, py = ev + (uint64_t)o1 * kEvRecBytes;
  SimStage x{0.0, -INFINITY, 0.0, 0.0}, y{0.0, -INFINITY, 0.0, 0.0};
  for (uint32_t b = b0; b < b1; ++b) {
    const uint32_t off = b * 64u;
    const u64x8 ex = sload<u64x8>(px, off), ey = sload<u64x8>(py, off);
    const f64x8 op = sload<f64x8>(a.ops, off);
    sim_record(x, y, ex[0], ex[1], ex[2], ex[3], ey[0], ey[1], ey[2], ey[3], op[0], op[1], op[2], op[3]);
    sim_record(x, y, ex[4], ex[5], ex[6], ex[7], ey[4], ey[5], ey[6], ey[7], op[4], op[5], op[6], op[7]);
  }
  if constexpr (kSegs > 1) {
    __shared__ double part[kSegs][8][kWave];
    double(*q)[kWave] = part[seg];
    q[0][lane] = x.U; q[1][lane] = x.top; q[2][lane] = x.cost; q[3][lane] = x.U0;
    q[4][lane] = y.U; q[5][lane] = y.top; q[6][lane] = y.cost; q[7][lane] = y.U0;
    __syncthreads();
    if (seg) return;
    for (int k = 1; k < kSegs; ++k) {
      x.top = fmax(x.top, x.U + part[k][1][lane]);
      x.U += part[k][0][lane];
      x.cost += part[k][2][lane];
      x.U0 += part[k][3][lane];
      y.top = fmax(y.top, y.U + part[k][5][lane]);
      y.U += part[k][4][lane];
      y.cost += part[k][6][lane];
      y.U0 += part[k][7][lane];
    }
  }
  int64_t peak = (int64_t)(a.base + x.U0 + x.top), cost = (int64_t)x.cost;
  if (2 * pair + 1 < a.n) {
    const int64_t p2 = (int64_t)(a.base + y.U0 + y.top);
    peak = p2 > peak ? p2 : peak;
    cost += (int64_t)y.cost;
  }
  const int k = (a.g0 + (int)blockIdx.x) * kWave + lane;
  if (k < a.K) {
    atomicMax(reinterpret_cast<long long*>(a.peak) + k, (long long)peak);
    atomicAdd(reinterpret_cast<unsigned long long*>(a.cost) + k, (unsigned long long)cost);
  }
}

// ---------------------------------------------------------------------------
// Best candidate's R rows t0 .. from the event records of a chunk: block per
// row, lane = node.
__global__ void __launch_bounds__(256) ckm_best_events_kernel(const char* __restrict__ events, size_t ev_bytes,
                                                              int32_t one_group, int32_t t0, uint32_t row0,
                                                              const uint32_t* __restrict__ row_off,
                                                              const int32_t* __restrict__ main_rec, int32_t words64,
                                                              const int32_t* __restrict__ best_k,
                                                              uint64_t* __restrict__ R_rows) {
  const int t = t0 + blockIdx.x;
  const int bk = best_k[0];
  const char* row = events + (size_t)(bk < 0 || one_group ? 0 : bk / kWave) * ev_bytes +
                    (size_t)(row_off[t] - row0) * kEvRecBytes;
  for (int v = threadIdx.x; v < kWave * words64; v += 256) {
    bool r = false;
    if (bk >= 0 && v <= t)
      r = (*reinterpret_cast<const uint64_t*>(row + (size_t)main_rec[v] * kEvRecBytes) >> (bk & (kWave - 1))) & 1;
    const uint64_t w = __ballot(r);
    if ((threadIdx.x & (kWave - 1)) == 0) R_rows[(size_t)t * words64 + v / kWave] = w;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
static ClosureArgs closure_args(const ckm_graph& g, const Layout& L, const EvChunk& ch, char* work) {
  const EventGraph& ev = g.ev;
  ClosureArgs a;
  a.n = g.n;
  a.pairs = ev.pairs;
  a.tlo = ch.tlo;
  a.thi = ch.thi;
  a.g0 = ch.g0;
  a.row0 = (uint32_t)ev.tile_row[ch.tlo];
  a.s_bytes = (uint32_t)(mask_rows_words(g.n) * sizeof(uint64_t));
  a.ev_bytes = (uint32_t)((ev.tile_row[ch.thi] - ev.tile_row[ch.tlo]) * kEvRecBytes);
  a.far_bytes = (uint32_t)ev.nf * kEvSlotBytes;
  a.npins = ev.npins;
  a.srows = reinterpret_cast<const uint64_t*>(work + L.rows_off);
  a.events = work + L.events_off;
  a.far = a.events + (size_t)ch.gn * a.ev_bytes;
  a.desc = ev.d_desc;
  a.extra = (cptr<uint32_t>)ev.d_extra;
  a.row_off = (cptr<uint32_t>)ev.d_row_off;
  a.tile_chunk = (cptr<int32_t>)ev.d_tile_chunk;
  a.pins = (cptr<int32_t>)ev.d_pins;
  a.best_k = nullptr;
  return a;
}

hipError_t launch_events(const ckm_graph& g, const Layout& L, int32_t K, char* work, hipStream_t stream) {
  for (const EvChunk& ch : event_chunks(g, L, K)) {
    const ClosureArgs c = closure_args(g, L, ch, work);
    hipLaunchKernelGGL(ckm_closure_kernel, dim3(ch.gn, ch.thi - ch.tlo), dim3(kWave), 0, stream, c);
    SimArgs s;
    s.n = g.n;
    s.K = K;
    s.phi = std::min(32 * ch.thi, g.ev.pairs);
    s.g0 = ch.g0;
    s.row0 = c.row0;
    s.base = (double)g.base;
    s.ev_bytes = c.ev_bytes;
    s.events = (cptr<char>)c.events;
    s.ops = (cptr<char>)g.ev.d_ops;
    s.row_off = c.row_off;
    s.peak = reinterpret_cast<int64_t*>(work + L.part_peak_off);
    s.cost = reinterpret_cast<int64_t*>(work + L.part_cost_off);
    const dim3 grid(ch.gn, s.phi - 32 * ch.tlo);
    const int64_t waves = (int64_t)grid.x * grid.y;
    if (waves >= 8192)
      hipLaunchKernelGGL(ckm_simulate_kernel<1>, grid, dim3(kWave), 0, stream, s);
    else if (waves >= 2048)
      hipLaunchKernelGGL(ckm_simulate_kernel<2>, grid, dim3(2 * kWave), 0, stream, s);
    else if (waves >= 1024)
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
  std::vector<EvChunk> chunks = event_chunks(g, L, K);
  const bool kept = chunks.size() == 1;
  if (!kept) chunks = event_chunks(g, L, 1);
  for (const EvChunk& ch : chunks) {
    ClosureArgs c = closure_args(g, L, ch, work);
    if (!kept) {
      c.best_k = d_best_k;
      hipLaunchKernelGGL(ckm_closure_kernel, dim3(1, ch.thi - ch.tlo), dim3(kWave), 0, stream, c);
    }
    const int32_t t0 = kWave * ch.tlo, t1 = std::min(kWave * ch.thi, g.n);
    hipLaunchKernelGGL(ckm_best_events_kernel, dim3(t1 - t0), dim3(256), 0, stream, c.events, (size_t)c.ev_bytes,
                       kept ? 0 : 1, t0, c.row0, g.ev.d_row_off, g.ev.d_main_rec, L.row_words / 2, d_best_k,
                       d_best_R);
  }
  return hipGetLastError();
}

}  // namespace ckm

// Event path: the static tables that the closure and simulate kernels of a
// graph read, and the host code that builds them.
//
// The evaluate stage of the event path runs in two kernels. The closure
// kernel makes, for every group of 64 candidates and every stage, one
// 32-byte event record per graph record: the words R (computed), S (held at
// the stage's start), F0 and F1 (released after it), bit j of each being
// candidate j. The simulate kernel runs the U recurrence over the records of
// a stage, in increasing order. A graph record is a node with its first two
// dependencies; a node with more dependencies has further records of two
// dependencies each right after it (R = S = 0 there).
//
// The closure scans nodes downwards with one accumulator per node i,
//   acc_i = S_{t+1}[i] | OR of R_t[u] over the users u of i decided so far,
// so that R_t[i] = acc_i & ~S_t[i] when the scan reaches i (Algorithm 2,
// constraints 1b and 1c), and FREE(t, i, v) = R_t[v] & ~acc_i just before
// user v is added to it (eq. collectable). The tables lay the accumulators
// out in LDS slots of one 64-bit word per lane:
//   ring     32 slots, node i in slot i mod 32: the nodes of the current
//            4-node chunk and the six below it
//   staging  two slots per node, by node mod 8: accumulators of dependencies
//            more than six chunks below their user (far); they live in
//            device memory (far slot, one word per lane) between far users,
//            and enter the ring seven chunks ahead of their node
//   pins     nodes whose far users come so close together that the load
//            issued for one would miss the store of the one before: these
//            keep an LDS slot through the whole scan
//   extra    two slots for far dependencies in records beyond the second
//   none     all ones: the slot of an absent dependency (it frees nothing)
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace ckm {

constexpr int kEvRecBytes = 32;             // event record: R, S, F0, F1
constexpr int kEvChunk = 4;                  // nodes per chunk
constexpr int kEvNear = 6;                   // chunks below the current one resident in the ring
constexpr int kEvDescDw = 16;                // dwords per node descriptor
constexpr int kEvSlotBytes = 512;            // one 64-bit word per lane
constexpr int kEvRing = 32, kEvStage = kEvRing, kEvPin = kEvStage + 16, kEvPins = 12, kEvXtra = kEvPin + kEvPins,
              kEvNone = kEvXtra + 2, kEvSlots = kEvNone + 1;

// Node descriptor dwords (lane l of a chunk's load holds dword l; node 4c + j
// at 16 j):
//   0 LDS byte offsets of slots 0, 1 (low, high half)
//   1 flags | number of records beyond the second << 16
//   2 far slots of slots 0, 1
//   3 index of the first record beyond the second (EvExtra)
//   4, 5 slot 0, 1 when far: dependency | next higher far user << 16
//   6 the node's own far slot | its lowest far user << 16 (0xFFFF: none)
//   7 LDS byte offset of the node's accumulator
//   8 LDS byte offsets of slots 2, 3 (second record)
//   15 j = 0: chunk flags; j = 1: first record of the next chunk
constexpr uint32_t kEvOwnFwd = 1u;       // node v + 1 has v among its first four slots
constexpr uint32_t kEvFar0 = 2u, kEvFar1 = 4u;     // slot 0 / 1 is far
constexpr uint32_t kEvSync0 = 8u, kEvSync1 = 16u;  // ... and is loaded when used (too close to the user above)
constexpr uint32_t kEvSecond = 32u;      // has a second record
constexpr uint32_t kEvEntrySync = 64u;   // ring entry loaded at the end of its chunk (a far user seven chunks above)
constexpr uint32_t kEvChunkFar = 1u, kEvChunkEntry = 2u;   // some slot is far (not sync) | some node has a far user

// A record beyond a node's second, 8 dwords: LDS byte offsets, flags
// (kEvFar0, kEvFar1), far slots, dependencies, next higher far users.
constexpr int kEvExtraDw = 8;

struct EventTables {
  int32_t n = 0, np = 0, chunks = 0;   // nodes, padded to whole chunks with at least three empty ones
  int32_t nrec = 0;                    // records (padded nodes have one each), a multiple of 4 with padding
  int32_t nf = 0;                      // far slots
  int32_t pairs = 0, tiles = 0;        // stage pairs, tiles of 64 stages
  std::vector<uint32_t> desc;          // chunks * 64 dwords
  std::vector<uint32_t> extra;
  std::vector<double> ops;             // nrec x (M_v, C_v, M of slot 0, M of slot 1)
  std::vector<uint32_t> row_off;       // first event record of stage t, 0 .. 2 pairs; both stages of a pair have
                                       // as many: the records of the pair's last node and all before, rounded up to 4
  std::vector<int32_t> main_rec;       // first record of node v, 0 .. np
  std::vector<int32_t> tile_chunk;     // chunk in which the scan of a tile's stages starts
  std::vector<int32_t> pins;           // nodes with a slot of their own, at most kEvPins
};

// False when the event records of one tile's 64 stages would take more than
// max_tile_bytes for a group, or a group's 2^32 records (very dense graphs).
bool build_events(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                  const int32_t* user_ptr, const int32_t* user_idx, uint64_t max_tile_bytes, EventTables& T);

}  // namespace ckm

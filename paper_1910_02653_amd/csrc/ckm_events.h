// Event path: the static tables that the closure and simulate kernels of a
// graph read, and the host code that builds them.
//
// The evaluate stage of the event path runs in two kernels over tiles of 32
// stages, with a candidate to a lane and a stage to a bit. The closure kernel
// makes, for every group of 64 candidates and every tile, one event record
// per graph record: per lane the words R (computed), S (held at the stage's
// start), F0 and F1 (released after it), bit j being stage 32 T + j. The
// simulate kernel runs the U recurrence over a tile's records, in increasing
// order. A graph record is a node with its first two dependencies; a node
// with more has further records of two dependencies each right after it
// (R = S = 0 there).
//
// The closure scans nodes downwards with one accumulator per node i,
//   acc_i = S_{t+1}[i] | OR of R_t[u] over the users u of i decided so far,
// so that R_t[i] = acc_i & ~S_t[i] when the scan reaches i (Algorithm 2,
// constraints 1b and 1c), and FREE(t, i, v) = R_t[v] & ~acc_i just before
// user v is added to it (eq. collectable). The tables lay the accumulators
// out in LDS slots of one 32-bit word per lane:
//   ring     32 slots, node i in slot i mod 32: the nodes of the current
//            4-node chunk and the six chunks below it
//   staging  two slots per node, by node mod 8: accumulators of dependencies
//            more than six chunks below their user (far); they live in
//            device memory (far slot, one word per lane) between far users,
//            and enter the ring seven chunks ahead of their node
//   pins     nodes whose far users come so close together that the load
//            issued for one would miss the store of the one before: these
//            keep an LDS slot through the whole scan
//   extra    two slots for far dependencies in records beyond the second
//   none     all ones: the slot of an absent dependency (it frees nothing)
// and, beside the ring, the words S_t of its nodes.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace ckm {

constexpr int kEvTile = 32;                  // stages per tile
constexpr int kEvChunk = 4;                  // nodes per chunk
constexpr int kEvNear = 6;                   // chunks below the current one resident in the ring
constexpr int kEvAhead = 2;                  // chunks between a load from device memory and its use
constexpr int kEvDescDw = 16;                // dwords per node descriptor
constexpr int kEvRecBytes = 1024;            // event record of a group: R, S, F0, F1 per lane
constexpr int kEvSlotBytes = 256;            // one 32-bit word per lane
constexpr int kEvQuadBytes = 1024;           // S words of four nodes, 16 bytes per lane
constexpr int kEvRing = 32, kEvStage = kEvRing, kEvPin = kEvStage + 16, kEvPins = 16, kEvXtra = kEvPin + kEvPins,
              kEvNone = kEvXtra + 2, kEvHeld = 96, kEvSlots = kEvHeld + kEvRing;
static_assert(kEvNone < kEvHeld, "LDS slots");

// Node descriptor dwords (lane l of a chunk's load holds dword l; node 4c + j
// at 16 j):
//   0 LDS byte offset of slot 0
//   1 flags | number of records beyond the second << 16
//   2 LDS byte offset of slot 1
//   3 byte offset of the node's first event record in a tile
//   4, 5 slot 0, 1 when far: dependency | next higher far user << 16
//   6 the node's own far slot | its lowest far user << 16 (0xFFFF: none)
//   7 far slots of slots 0, 1 (low, high half)
//   8 LDS byte offsets of slots 2, 3 (second record)
//   9 index of the first record beyond the second
//   10 LDS byte offset of the node's pin (kEvPinned)
//   11 byte offset in a tile's S words of slot 0's dependency when far (else 0)
//   12 byte offset of slot 0's far accumulator when far, else that of a spare
//   15 (j = 0 only) chunk flags
constexpr uint32_t kEvFar0 = 2u, kEvFar1 = 4u;     // slot 0 / 1 is far
constexpr uint32_t kEvSync0 = 8u, kEvSync1 = 16u;  // ... and is loaded when used (too close to the user above)
constexpr uint32_t kEvSecond = 32u;      // has a second record
constexpr uint32_t kEvEntrySync = 64u;   // ring entry loaded when written (a far user just above the ring)
constexpr uint32_t kEvPinned = 128u;     // the node's accumulator is in a pin
// Chunk flags: some slot is far (not sync); some node has a far user; some node
// has a second record; a node needs one of the rare forms (records beyond the
// second, a sync slot, a pin, a far slot 1, a far dependency with a far user
// above); a node has kEvEntrySync; bits 8 ..: node 4c + j uses node 4c + i, for (j, i) = (3, 2), (3, 1),
// (3, 0), (2, 1), (2, 0), (1, 0).
constexpr uint32_t kEvChunkFar = 1u, kEvChunkEntry = 2u, kEvChunkSecond = 4u, kEvChunkRare = 8u,
                   kEvChunkEntrySync = 16u;
constexpr int kEvChunkUse = 8;

// A record beyond a node's second, 8 dwords: LDS byte offsets, flags
// (kEvFar0, kEvFar1), far slots, dependencies, next higher far users.
constexpr int kEvExtraDw = 8;

struct EvOps {          // a record's operands
  double M;             // M_v (0 past a node's first record)
  uint64_t C;           // C_v
  double M0, M1;        // sizes of its two dependencies
};

struct EventTables {
  int32_t n = 0, np = 0, chunks = 0;   // nodes, padded to whole chunks
  int32_t nrec = 0;                    // records
  int32_t nf = 0;                      // far slots, the spare among them
  int32_t tiles = 0;
  std::vector<uint32_t> desc;          // chunks * 64 dwords
  std::vector<uint32_t> extra;
  std::vector<EvOps> ops;              // nrec, and a few empty ones for reads ahead
  std::vector<int32_t> main_rec;       // first record of node v, 0 .. np
  std::vector<int32_t> tile_rec;       // records of a tile's scan: those of nodes 0 .. its last chunk's end
  std::vector<int32_t> pins;           // nodes with a slot of their own, at most kEvPins
};

// The chunk in which the scan of tile T starts: that of its last stage's node.
constexpr int32_t ev_first_chunk(int32_t n, int32_t T) {
  return (kEvTile * T + kEvTile < n ? kEvTile * T + kEvTile - 1 : n - 1) / kEvChunk;
}

// False when one tile's event records would take more than max_tile_bytes for
// a group (very dense graphs).
bool build_events(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                  const int32_t* user_ptr, const int32_t* user_idx, uint64_t max_tile_bytes, EventTables& T);

}  // namespace ckm

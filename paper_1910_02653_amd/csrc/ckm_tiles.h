// Tile path: the static tables that the closure and simulate kernels of a
// graph read, and the host code that builds them.
//
// The path works on tiles of 32 stages, with a candidate to a lane and a stage
// to a bit: one 32-bit word per (group of 64 candidates, tile, node, lane), bit
// j being stage 32 T + j. The closure kernel decides R (Algorithm 2,
// constraints 1b, 1c, 4a) by blocks of 32 nodes, from the tile's last down:
//   R[v] = (S_{t+1}[v] | OR of R[u] over the users u of v) & ~S_t[v].
// Users two or more blocks up (far users) are ORed in while the block above is
// being decided; those in the block and the next one (near users) are read
// from LDS, four nodes (a chunk) at a time. The simulate kernel runs the U
// recurrence over the nodes in increasing order, and makes each FREE word
// (eq. collectable) where it is needed:
//   F(i, v) = R[v] & ~(S_{t+1}[i] | OR of R[u] over the users u > v of i).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace ckm {

constexpr int kTile = 32;                    // stages per tile, nodes per block
constexpr int kChunk4 = 4;                   // nodes per chunk
constexpr int kSlotBytes = 256;              // one word per lane (in LDS and in the tiles)
// LDS slots of the closure kernel: R of the last two blocks (node v in slot
// v mod 64), a slot of zeros, and what is prepared of two blocks.
constexpr int kRingNodes = 64;
constexpr int kRingEmpty = kRingNodes;
constexpr int kSlotNeed = kRingEmpty + 1;    // S_{t+1} | far users, [block parity][32]
constexpr int kSlotS = kSlotNeed + 64;       // S_t, likewise
constexpr int kSlotDesc = kSlotS + 64;       // chunk descriptors, [block parity][4]
constexpr int kClosureSlots = kSlotDesc + 8;

// Chunk descriptor, 32 dwords (lane 32 (c mod 2) + l of a load of two chunks
// holds dword l):
//   4 j + k       LDS byte offset of near user k < 4 of node 4c + j (the slot
//                 of zeros when absent); users in the chunk are not among them
//   16            flags of the block, and bits 0 .. 5: node 4c + j uses node 4c + i, for (j, i) =
//                 (3, 2), (3, 1), (3, 0), (2, 1), (2, 0), (1, 0)
//   17 + 2 j, +1  first and count of node 4c + j's near users beyond the four
constexpr int kDescDwords = 32;
constexpr uint32_t kBlockNear3 = 1u << 8;    // some node of the block has a third near user
constexpr uint32_t kBlockNear4 = 1u << 9;    // ... a fourth
constexpr uint32_t kBlockMany = 1u << 10;    // ... a fifth

// Far users of half a block (16 nodes), 64 dwords: node i's first two users' R
// tile byte offsets at i and 16 + i (0, the tile's empty word, when absent),
// first and count of the rest at 32 + i and 48 + i.
constexpr int kFarNodes = 16, kFarDwords = 64;

// A simulation record: a node with its first two dependencies; a node with more
// has further records of two dependencies each right after it.
struct SimOps {
  double M;            // M_v (0 past a node's first record)
  double M0, M1;       // sizes of the dependencies (0 when absent)
  double pad;
};
// Its words, as offsets in slots (node_off / 256): S tile slots of the node and
// the dependencies, R tile slots of the dependencies' users above v (0 when
// absent).
struct SimRefs {
  uint16_t v, s[2];
  uint16_t u[2][4];
  uint16_t more;       // u[.][2] present
  uint64_t C;          // C_v (0 past a node's first record)
};
constexpr int32_t kMaxSlots = 65536;         // of an R tile, for the tile path

// Nodes with more than kHubUsers users: for each user with three or more above
// it, the OR of those above (a hub word) is made once, after the closure, and
// stands in for them.
constexpr int kHubUsers = 5;
struct HubUser {
  uint32_t r;          // R tile byte offset of the user
  uint32_t x;          // R tile byte offset of the hub word of the users above it (0: none)
};

struct TileTables {
  int32_t n = 0, tiles = 0, nrec = 0, nhub = 0;
  uint32_t rbase = 0;                   // R tile byte offset of node 0: after the empty word and the hub words
  std::vector<uint32_t> desc;           // tiles * 8 chunks * kDescDwords
  std::vector<uint32_t> near_more;      // LDS byte offsets
  std::vector<uint32_t> far;            // tiles * 2 * kFarDwords
  std::vector<uint32_t> far_more;       // R tile byte offsets
  std::vector<SimOps> ops;              // nrec
  std::vector<SimRefs> refs;            // nrec
  std::vector<int32_t> tile_rec;        // records of the nodes below each tile's end
  std::vector<int32_t> hub_ptr;         // nhub + 1
  std::vector<HubUser> hub;             // users in decreasing order
};

// S tile byte offset of node v's words (R tiles: + rbase).
constexpr uint32_t node_off(int32_t v) { return (uint32_t)v * (uint32_t)kSlotBytes; }
// False when the graph does not take the tile path (an R tile with its hub words
// has more than kMaxSlots slots).
bool build_tiles(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                 const int32_t* user_ptr, const int32_t* user_idx, TileTables& T);

}  // namespace ckm

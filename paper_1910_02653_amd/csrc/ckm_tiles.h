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
  uint64_t C;          // C_v (0 past a node's first record)
};
// Its words, as slots of kSlotBytes: of the S tile for the node and the
// dependencies, of the R tile for the dependencies' users above v (0, the empty
// word, when absent), of the tile's hub words for the rest of them.
struct SimRefs {
  uint16_t v, s[2];
  uint16_t more;       // kMore* << dependency
  uint16_t u[2][4];    // three users, or two and the count of the list; the hub word or a fourth user
  uint32_t list[2];    // kMoreList: where the users past the second are in the graph's users
};
constexpr uint32_t kMoreThird = 1, kMoreHub = 4, kMoreList = 16, kMoreFourth = 64;

// Hub words. A node with more than kHubUsers users has a word for its highest
// `step` users, one for its highest 2 step, and so on: the OR of their R, made
// after the closure. A dependency with three or more users above v takes one of
// them and the less than `step` users below those that it covers; with two or
// less it takes these (so that step 1 needs no word of one or two users).
// step is the smallest with at most kHubWordsPerNode words per node, or 4, the
// largest whose users fit in a record; if a tile would have more than kMaxHubWords
// then, it is as large as that needs, and the users past the second come in a
// list. So a tile's hub words are a few per node, or at most a quarter of the
// edges, and never above 16 MB, whatever the graph. (A word per user, without
// these bounds, took 75 times the S rows at n = 300 and all edges.) With few users
// a word each is read faster, with many the words written cost more: step 1 / 4,
// n = 300, 12 dependencies per node, K = 64 205 / 215 us; four blocks of 64 nodes, all
// pairs of a block an edge, n = 513, K = 512 1.57 / 1.48 ms; n = 300, all edges 2.69 / 2.41.
constexpr int kHubUsers = 5;
constexpr int kHubWordsPerNode = 4;
constexpr int kHubStep = 4;
constexpr int64_t kMaxHubWords = 65535;      // slot 0 is a word of zeros
struct HubUser {
  uint32_t r;          // R tile byte offset of the user
  uint32_t x;          // byte offset among the hub words of the word that it completes (0: none)
};

struct TileTables {
  int32_t n = 0, tiles = 0, nrec = 0, nhub = 0, step = 1;
  std::vector<uint32_t> desc;           // tiles * 8 chunks * kDescDwords
  std::vector<uint32_t> near_more;      // LDS byte offsets
  std::vector<uint32_t> far;            // tiles * 2 * kFarDwords
  std::vector<uint32_t> far_more;       // R tile byte offsets
  std::vector<SimOps> ops;              // nrec
  std::vector<SimRefs> refs;            // nrec
  std::vector<int32_t> tile_rec;        // records of the nodes below each tile's end
  std::vector<int32_t> hub_ptr;         // nhub + 1
  std::vector<HubUser> hub;             // users in decreasing order
  // Hub words are numbered from 1 in the order of the lowest user that each
  // covers, and a tile makes those that cover a node of it. hub_at[T]: slots
  // of a group's tiles T and up (each with a word of zeros, slot 0); empty
  // without hub words.
  std::vector<uint32_t> hub_at;         // tiles + 1
};

// S tile byte offset of node v's words; R tiles have an empty word before them.
constexpr uint32_t node_off(int32_t v) { return (uint32_t)v * (uint32_t)kSlotBytes; }
constexpr uint32_t kRBase = kSlotBytes;
void build_tiles(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr, const int32_t* dep_idx,
                 const int32_t* user_ptr, const int32_t* user_idx, TileTables& T,
                 int64_t max_hub_words = kMaxHubWords);

}  // namespace ckm

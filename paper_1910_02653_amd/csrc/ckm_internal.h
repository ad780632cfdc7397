// Internal declarations shared by the host glue and the HIP kernels of libckm.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <vector>

#include "ckm.h"

namespace ckm {
struct SyncCache;  // buffers and stream of the synchronous entry points (ckm_host.cpp)

// The tile path's tables on the device (TileTables, ckm_tiles.h); on is false
// for wide graphs, which do not take it.
struct TileGraph {
  bool on = false;
  int32_t nhub = 0, hub_rounds = 0;   // hub_rounds: users of all hubs, in rounds of eight
  std::vector<uint32_t> hub_at;  // slots of hub words of a group in the tiles above each (TileTables)
  const uint32_t* d_desc = nullptr;
  const uint32_t* d_near_more = nullptr;
  const uint32_t* d_far = nullptr;
  const uint32_t* d_far_more = nullptr;
  const void* d_ops = nullptr;
  const void* d_refs = nullptr;
  const int32_t* d_tile_rec = nullptr;
  const int32_t* d_hub_ptr = nullptr;
  const void* d_hub = nullptr;
  const uint32_t* d_hub_at = nullptr;
};
}

// Graph on the device. Node arrays hold sizes and costs as int64. Users
// rows are sorted ascending; for the dep entry e = (i -> v) in v's deps row,
// dep_upos[e] is the index in user_idx of the first user of i that is
// greater than v. The evaluate kernels sum sizes and costs in binary64 when
// every sum they form stays below 2^53 (exact there), and in int64 otherwise
// (`wide`); the node records carry the values in the chosen form.
struct ckm_graph {
  int32_t n = 0;
  int32_t num_edges = 0;
  int device = 0;
  int64_t base = 0;           // M_in + 2 M_param (eq. U_init constant overhead)
  bool wide = false;          // sums reach 2^53: int64 arithmetic in the evaluate kernels
  int32_t eval_waves = 1;     // resident evaluate waves per CU for this n (work plan sizing)
  void* d_mem = nullptr;      // one allocation holding every array below
  const int64_t* d_M = nullptr;
  const int64_t* d_C = nullptr;
  const int32_t* d_user_ptr = nullptr;
  const int32_t* d_user_idx = nullptr;
  const int32_t* d_dep_ptr = nullptr;
  const int32_t* d_dep_idx = nullptr;
  const int32_t* d_dep_upos = nullptr;
  const void* d_recs = nullptr;  // n node records of ckm::kNodeRecBytes (see ckm_kernels.hip)
  ckm::TileGraph tile;           // the tile path's tables
  const void* d_mrecs = nullptr; // mask-path node data when the graph fits it, else NULL
  ckm::SyncCache* sync = nullptr;  // reused by the synchronous calls; freed with the graph
};

namespace ckm {

constexpr int kWave = 64;
constexpr int kNodeRecBytes = 256;
constexpr int kMaxNodesWords = CKM_MAX_NODES / 32;

// Where the evaluate kernel's S rows come from.
enum : int {
  kSrcRound = 0,      // randomized rounding of S* (deterministic candidate 0 under CKM_F_DET0)
  kSrcUser = 1,       // the caller's integral S matrices
  kSrcThreshold = 2,  // threshold rounding [clamp(S*) > p_k], one threshold per candidate
  kSrcRows = 3,       // randomized rounding done beforehand into the work buffer's row array
};

// The row arrays (S rows streamed by the evaluate kernel, R rows it keeps; S and
// R tiles on the tile path) are used when the S rows fit in this many bytes
// (about K * n^2 / 16 bytes each; 4.1 GB at n = 4001, K = 4096); larger
// problems, or work buffers sized without them, make the S rows in the evaluate
// kernel and recompute the best candidate's R.
constexpr size_t kRowsMaxBytes = (size_t)8 << 30;
// A buffer that does not hold the tiles of all groups is used in passes over them
// on graphs of at least kPassTiles tiles when a pass has kPassPairs (group, tile)
// pairs, which fill the chip. Measured, passes / the scan without row arrays:
// n = 129, K = 65,536 in 2 passes 494 / 787 us, in 8 (640 pairs each) 626; K = 4096
// in 2 (160 pairs) 86 / 74; n = 1009, K = 4096 in 4 (512 pairs) 1249 / 2773;
// n = 33, K = 65,536 in 2 (1024 pairs) 129 / 105.
constexpr int32_t kPassTiles = 3, kPassPairs = 512;
// Room asked for hub words, at most: when all (group, tile) pairs have more, hub
// words and simulation run in several launches, each over the pairs that fit (64
// at least). Measured, in the launches that the room leads to:
// n = 2049, 65,568 edges, K = 512 (520 pairs): 17.2 ms in eight, 8.2 in one;
// n = 801, 40,008 edges, K = 512 (208 pairs): 4.0 ms in two, 3.5 in one.
constexpr size_t kHubMaxBytes = (size_t)1 << 30;

// Host-side builder of the per-node records the evaluate kernel reads
// (layout documented with NodeRec in ckm_kernels.hip). Writes n records.
// M, C: int64 sizes and costs; wide: store them as int64 (else as binary64).
void build_node_records(int32_t n, const int64_t* M, const int64_t* C, bool wide, const int32_t* dep_ptr,
                        const int32_t* dep_idx, const int32_t* user_ptr, const int32_t* user_idx,
                        void* out);

// Mask path (ckm_kernels.hip): bytes and builder of a graph's node data (false
// when it does not fit), 64-bit words of a group's mask rows, and when it is used.
int32_t mask_records_bytes(int32_t n);
bool build_mask_records(int32_t n, const int64_t* M, const int64_t* C, const int32_t* dep_ptr,
                        const int32_t* dep_idx, const int32_t* user_ptr, const int32_t* user_idx, void* out);
size_t mask_rows_words(int32_t n);
bool use_masks(const ckm_graph& g, int32_t K);

// The tile path's S and R words (ckm_tiles.h): for one candidate group, tile T
// of 32 stages holds a word per lane of 32 (T + 1) nodes, one tile after another. An R tile has a word before them.
__host__ __device__ __forceinline__ uint32_t stile_bytes(int T) { return 8192u * (uint32_t)(T + 1); }
__host__ __device__ __forceinline__ size_t stile_off(int T) { return (size_t)4096 * T * (T + 1); }
__host__ __device__ __forceinline__ size_t rtile_off(int T) { return stile_off(T) + (size_t)256 * T; }

// Hub words of a (group, tile) pair: a word of zeros and the tile's.
inline size_t hub_pair_bytes(const TileGraph& t, int T) { return (size_t)256 * (t.hub_at[T] - t.hub_at[T + 1]); }

// Work-buffer layout for (n, K). Offsets are bytes from the buffer start,
// each 256-byte aligned.
struct Layout {
  int32_t n = 0, K = 0;
  int32_t ldq = 0;        // q / det row stride in elements: round_up(n + 8, 64)
  int32_t det_words = 0;  // ldq / 32
  int32_t row_words = 0;  // 32-bit words per output bit row: 2 * ceil(n / 64)
  int32_t max_splits = 0; // most work items per group of 64 candidates
  int32_t reduce_blocks = 0;
  size_t q_off = 0, det_off = 0, nan_off = 0, part_peak_off = 0, part_cost_off = 0,
         best_off = 0, srows_off = 0, thr_sorted_off = 0, thr_rank_off = 0,
         // execution plans: per-stage statement and compute counts, check
         // flags, first statement and first register, and the go flag
         plan_cnt_off = 0, plan_comp_off = 0, plan_err_off = 0, plan_pos_off = 0, plan_rbase_off = 0,
         plan_go_off = 0,
         // R transposed (n columns of ceil(n/32) words) and per-row word ranks
         plan_rt_off = 0, plan_rpre_off = 0,
         bbest_off = 0,  // per-block best of the batch multipliers
         total = 0,        // bytes every call needs
         rows_off = 0,     // S rows of every candidate (kSrcRows, or S tiles), past `total`
         rrows_off = 0,    // R rows (or R tiles) of every candidate, written by the evaluate stage
         hub_off = 0,      // the tile path's hub words, of as many (group, tile) pairs as hub_bytes hold
         hub_bytes = 0,
         total_rows = 0;   // total plus the row arrays (and the hub words) when they are used
  bool rows_on = false;    // the S rows fit kRowsMaxBytes (and, after
                           // check_work, the caller's buffer holds both)
  bool masks = false;      // the mask path: S rows as masks, R rows as the row arrays
  int32_t pass_groups = 0; // tile path: candidate groups evaluated at a time, all with
                           // rows_on; fewer where the buffer holds no more (0: none)
};

Layout make_layout(const ckm_graph& g, int32_t K);

// Records a thread-local error message (ckm_last_error) and returns st.
ckm_status set_error(ckm_status st, const char* fmt, ...);

// The static work area of ckm_round_eval_noalloc (ckm_noalloc.hip):
// noalloc_setup resolves its address on `device`, which must be current
// (graph creation calls it); noalloc_scratch returns the kept address, or
// NULL when the device was never set up.
hipError_t noalloc_setup(int device);
void* noalloc_scratch(int device);

// How the stages of one group of 64 candidates are cut into work items (one
// wave each). Items are numbered in dispatch order, most expensive first, so
// the cheap ones fill the end of the launch.
//   kind 0: `items` ranges of about equal sum of stage lengths, top first.
//   kind 1: stages T0 .. n-1 in R1 items of P consecutive stages (top
//           first), then stages 0 .. T0-1 in R2 ranges of about equal sum of
//           stage lengths (top first).
struct Plan {
  int32_t items = 1, kind = 0, P = 0, T0 = 0, R1 = 0, R2 = 0;
};
Plan plan_auto(int32_t n, int32_t K, int32_t max_items, int32_t waves_per_cu);
Plan plan_stages(int32_t n, int32_t max_items);
Plan plan_splits(int32_t n, int32_t splits);

// Resident evaluate waves per CU for a graph of n nodes (the runtime's
// occupancy figure for the kernel variant and LDS size n and wide select).
int32_t eval_waves_per_cu(int32_t n, bool wide);

// ckm_round_eval_async.
ckm_status round_eval(const ckm_graph* g, const double* d_s_frac, int64_t ld, int32_t K, uint64_t seed,
                      int64_t budget, uint32_t flags, int64_t* d_peak, int64_t* d_cost, uint8_t* d_feasible,
                      int32_t* d_best_k, uint64_t* d_best_S, uint64_t* d_best_R, int32_t* d_status, void* d_work,
                      size_t work_bytes, void* stream);

// Kernel launchers (defined in ckm_kernels.hip). They only enqueue work.
hipError_t launch_quantize(const ckm_graph& g, const Layout& L, const double* d_s, int64_t ld,
                           char* work, hipStream_t stream);
// Randomized path: every candidate's S rows rounded once into the work
// buffer's row array (nothing when L.rows_on is false).
hipError_t launch_round_rows(const ckm_graph& g, const Layout& L, int32_t K, uint64_t seed, uint32_t flags,
                             char* work, hipStream_t stream);
// Threshold family: ranks of the K thresholds, their sorted copy, and the
// keys of S* in place of the quantized thresholds q.
hipError_t launch_threshold_keys(const ckm_graph& g, const Layout& L, const double* d_s, int64_t ld,
                                 const double* d_p, int32_t K, char* work, hipStream_t stream);
// Execution plan of (S, R) (bit rows of row_words 32-bit words): counts,
// checks and prefix sums, then the statements when d_P is not null.
hipError_t launch_plan(const ckm_graph& g, const Layout& L, const uint64_t* d_S, const uint64_t* d_R,
                       uint32_t flags, int32_t* d_P, int64_t capacity, int64_t* d_count, int64_t* d_mem,
                       int32_t* d_status, char* work, hipStream_t stream);
// Largest batch multiplier per candidate from the totals of the last
// evaluate, and the best one.
hipError_t launch_max_batch(const ckm_graph& g, const Layout& L, int32_t K, int64_t budget, int64_t cost_cap,
                            int64_t* d_batch, int32_t* d_best_k, int64_t* d_best_batch, int32_t* d_status,
                            char* work, hipStream_t stream);
// src: one of kSrcRound, kSrcUser, kSrcThreshold (kSrcRound streams the row
// array when L.rows_on, rounding it first unless flags has CKM_F_ROUNDED).
// s_user: for kSrcUser, K
// caller-supplied S matrices ([K][n][row_words] 32-bit words).
hipError_t launch_evaluate(const ckm_graph& g, const Layout& L, int32_t K, uint64_t seed,
                           uint32_t flags, const Plan& plan, int src, const uint64_t* s_user, char* work,
                           hipStream_t stream);
// Tile path (ckm_tiles.hip): the evaluate of candidate groups g0 .. g0 + groups - 1
// on their S tiles.
hipError_t launch_tiles(const ckm_graph& g, const Layout& L, int32_t K, int32_t g0, int32_t groups, char* work,
                        hipStream_t stream);
hipError_t launch_select(const ckm_graph& g, const Layout& L, int32_t K, uint64_t seed,
                         int64_t budget, uint32_t flags, int64_t* d_peak,
                         int64_t* d_cost, uint8_t* d_feasible, int32_t* d_best_k,
                         uint64_t* d_best_S, uint64_t* d_best_R, int32_t* d_status, int src,
                         const uint64_t* s_user, char* work, hipStream_t stream);

}  // namespace ckm

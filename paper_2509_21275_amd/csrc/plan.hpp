// Host-side planning for chunk attention: descriptor checks and the tile schedules that
// the kernels walk.  Pure C++ (no HIP), so it can be exercised without a GPU.
//
// A chunk {C, S} (paper section 3.1) arrives as a segment table; the schedule turns it into
// independent work items.  Only tiles that contain at least one unmasked (query, key) pair
// are ever scheduled: the causal mask and the block-diagonal structure of a packed chunk
// are exploited by construction, not by testing tiles on the device.
#pragma once
#include <cstdint>
#include <vector>

#include "../../include/chunk_attn.h"

#ifdef __HIPCC__
#define CHUNK_ATTN_HD __host__ __device__
#else
#define CHUNK_ATTN_HD
#endif

namespace chunk_attn {

// A tile (64 or 32 rows) of a tensor, for the pre-pass of the backward: rows [src_row0, src_row0 + valid_rows).
struct TileJob {
  int32_t src_row0, valid_rows;
  int32_t image;  // index of the tile (per head)
  int32_t pad;
};

// Forward work item: a tile of consecutive query rows of one segment.
struct FwdItem {
  int32_t q_row0;    // first query row (global)
  int32_t q_rows;    // valid rows in the tile (>= 1)
  int32_t kv_row0;   // first key row of the segment (global)
  int32_t n0;        // keys visible to the tile's first row: C + i0 + 1; row r sees n0 + r
  int32_t pad;
  // head_dim 96 and 128, whose walks over the keys may be cut into pieces (choose_key_split; 64 and 256: one piece each):
  int32_t keys;      // keys of the item's own range: it sees min(n0 + r, keys) of them
  int32_t pieces;    // a whole item: the number of its pieces (1: not cut)
  int32_t part;      // a piece: its slot among the partial results, -1 if it is the whole item.  A whole item: its first slot
};

// Work item of the dQ kernel: a tile of consecutive query rows of one segment (as in the forward).
struct DqItem {
  int32_t q_row0;    // first query row (global)
  int32_t q_rows;    // valid rows in the tile (>= 1)
  int32_t kv_row0;   // first key row of the segment (global)
  int32_t n0;        // keys visible to the tile's first row
  int32_t pieces;    // a whole item that was cut: the number of its pieces
  int32_t q_slot0;   // slot of the tile's first row in the padded per-row arrays (LSE, D)
  int32_t keys;      // head_dim 96 and 128: keys of the item's own range, as in FwdItem
  int32_t part;      // head_dim 96 and 128: slot among the partial results, -1 if the item is not a piece (whole items that
                     // were cut: the first slot)
};

// Work item of the dK/dV kernel: up to 256 consecutive key rows of one segment and the 32-row query tiles
// (aligned to the segment's first query) that contain at least one query seeing them.
struct DkvItem {
  int32_t kv_row0;    // first key row of the tile (global)
  int32_t kv_rows;    // valid key rows
  int32_t j0;         // index of the tile's first key inside the segment
  int32_t ctx;        // context length C of the segment
  int32_t q_row_seg;  // first query row of the segment (global)
  int32_t q_len;      // queries in the segment
  int32_t qt_first;   // first 32-row query tile (inside the segment) that sees a key of this tile
  int32_t n_qt;       // number of 32-row query tiles of the segment
  int32_t q_tile0;    // index of the segment's first 64-row tile in the padded per-row arrays (LSE, D)
  int32_t reverse;    // 1: the kernel walks the query tiles from the segment's last one down to qt_first (plan_dkv)
  int32_t pieces;     // a whole item that was cut: the number of its pieces
  int32_t part;       // slot among the partial results, -1 if the item is not a piece of a cut walk (a piece walks the query tiles
                      // qt_first .. n_qt - 1 of its own).  A whole item that was cut: its first slot
};

// Work item of the one-pass backward kernel (head_dim 128): a DkvItem plus what the kernel needs to add its share of dQ
// into the float32 dQ tiles in a fixed order.  All key blocks of one (segment, key/value head) form a chain, in
// order of their first key; a block adds to a dQ tile after its predecessor in the chain has (every query tile a block
// sees is also seen by its predecessor, so the first block of a chain initialises every tile).
struct FusedItem {
  int32_t kv_row0, kv_rows, j0, ctx, q_row_seg, q_len, qt_first, n_qt, q_tile0;  // as in DkvItem
  int32_t kvh;        // key/value head
  int32_t pred;       // item index of the predecessor in the chain, -1 for the chain's first block
  int32_t delta_qt;   // qt_first - predecessor's qt_first (>= 0)
  int32_t dq_tile0;   // index of the segment's first 32-row query tile in the dQ tile array (per head)
  int32_t buf;        // which dQ tile array the block's sub-chain adds into
  int32_t pad1, pad2;
};
// A 32-row tile of dQ for the conversion to bf16 rows.
struct DqTileJob {
  int32_t q_row0, valid_rows;  // first query row (global) and rows in the tile
  int32_t tile;                // index of the tile in a dQ tile array (per head)
  int32_t qt;                  // index of the tile inside its segment
  int32_t ctx, n_blocks;       // context length and number of key blocks of the segment
  int32_t pad0, pad1;
};
struct FusedPlan {
  std::vector<FusedItem> items;
  std::vector<int32_t> order;   // workgroup b runs item order[b] (-1: nothing); b % 8 is the XCD the chain is pinned to
  std::vector<DqTileJob> tiles;
  int64_t total_qt32 = 0;       // 32-row query tiles of all segments
  int num_bufs = 1;
};
// Sub-chains per (segment, key/value head): the blocks of a chain are dealt round robin to `num_bufs` sub-chains, each
// adding into a dQ tile array of its own (summed by the conversion), which shortens the wait along a chain.
int fused_num_bufs(const chunk_attn_desc* d, int keys);
FusedPlan plan_fused(const chunk_attn_desc* d, int keys, int num_xcd, int num_bufs);

int validate(const chunk_attn_desc* d);
int64_t pair_count(const chunk_attn_desc* d);

// Tiles of `tile_rows` query rows per segment, most work first.
std::vector<FwdItem> plan_fwd(const chunk_attn_desc* d, int tile_rows);
std::vector<DqItem> plan_dq(const chunk_attn_desc* d, int tile_rows);

// ---- cutting the walks of query-stationary items over the keys ----
// A work item walks all keys its rows see, one 32-key stage after the other.  A chunk with few query rows and many keys
// has fewer items than the chip has compute units, or so few that they do not divide evenly; its walks are then cut into
// pieces that run on different compute units, write float32 partial results and are put together afterwards.
constexpr int kStageKeys = 32;
constexpr int kMinPieceStages = 8;  // below that a piece's start and end cost more than its walk
// First of `n` units of piece k of `pieces` (unsigned 32-bit: fewer than 2^26 units, as 2^31 rows make, and at most 17 pieces;
// a 64-bit division takes several times as long, on the host and even more on the device).
CHUNK_ATTN_HD inline int share_begin(int n, int pieces, int k) { return (int)((unsigned)n * (unsigned)k / (unsigned)pieces); }
// First stage of piece k of a walk of `stages` stages cut into `pieces`.  Even: the kernels take steps two at a time.
CHUNK_ATTN_HD inline int piece_begin(int stages, int pieces, int k) { return share_begin(stages, pieces, k) & ~1; }
// Pieces of a walk whose first row sees n0 keys, for a cut into pieces of about `target` stages (0: none are cut).  The
// last piece begins with a key that every row sees (the rows of a piece need one to begin with).
CHUNK_ATTN_HD inline int piece_count(int stages, int n0, int target) {
  if (target <= 0) return 1;
  int n = (stages + target - 1) / target;
  if (n > stages / kMinPieceStages) n = stages / kMinPieceStages;
  while (n > 1 && piece_begin(stages, n, n - 1) * kStageKeys >= n0) --n;
  return n < 1 ? 1 : n;
}
CHUNK_ATTN_HD inline int walk_stages(int n0, int q_rows) { return (n0 + q_rows - 1 + kStageKeys - 1) / kStageKeys; }
// Items of a chunk and the stages they walk together.
struct Walks {
  int64_t items = 0, stages = 0;
  int64_t longest = 0;  // stages of the longest walk
  int64_t largest = 0;  // items of the sequence that has most
};
Walks count_walks(const chunk_attn_desc* d, int tile_rows);
struct KeySplit {
  int target = 0;      // argument of piece_count; 0: nothing is cut
  int64_t pieces = 0;  // items to run (pieces and whole items)
  int64_t parts = 0;   // pieces among them that write a partial result
};
// Query heads that a workgroup of the forward takes whose waves divide the keys of 32 rows (8 waves: 1, 2 or 4 heads, and as many of them per
// head as are left), where that ends sooner by the estimate of plan.cpp than the head dimension's other kernel, whose walks are `other`, each
// run for `inner` (key/value head, head split) pairs, on the software-pipelined kernel or not, cut as `split` says; 0 where it does not.
constexpr int kSharedWaves = 8, kMaxSharedItems = 104;  // (as many items as kernel arguments have room for)
int choose_shared_heads(const chunk_attn_desc* d, const Walks& other, int inner, bool pipelined, const KeySplit& split);
// Blocks of the small chunks' backward: tiles of 32 rows of a segment's queries, or of its keys, and the steps of their walks, longest first.
struct ShareBlock {
  int32_t seg, tile;
  int64_t steps;  // 32-key stages, or (32-query tile, head) pairs
};
constexpr int kMaxShareSegs = 64, kMaxShareItems = 640;
std::vector<ShareBlock> share_blocks(const chunk_attn_desc* d, bool keys);
// Whether the kernel arguments have room for a chunk's blocks and its block counts stay in 32 bits.
bool shared_backward_fits(const chunk_attn_desc* d);
// Waves per workgroup (4, or 8 at head_dim 64) of the backward whose waves divide the walks of 32-row blocks, where it ends sooner by the
// estimate of plan.cpp than the head dimension's other kernels, whose walks are `dq` (each run for `inner` pairs) and `dkv` (for each
// key/value head), cut as the splits say; 0 where it does not.  For chunks that fit.  (`head_dim`: that of the tensors; d's is 128 for 96.)
int choose_shared_waves(const chunk_attn_desc* d, int head_dim, const Walks& dq, int inner, const Walks& dkv, const KeySplit& dq_split, const KeySplit& dkv_split);
// The same for the key-stationary items (`keys` keys each) of one key/value head; a stage is a 32-row query tile of one head.
Walks count_dkv_walks(const chunk_attn_desc* d, int keys);
// The cut that ends first by the estimate of plan.cpp, given that each item is run for `inner` (key/value head, head
// split) pairs on `cus` compute units; at most `max_parts` partial results.
KeySplit choose_key_split(const chunk_attn_desc* d, int tile_rows, int inner, int cus, int64_t max_parts);
// The same for the walks of key-stationary items (`keys` keys each) over the query tiles, `group` steps per tile; `target` is
// in tiles (tile_piece_count).
inline int tile_piece_count(int tiles, int target) { return target > 0 ? (tiles + target - 1) / target : 1; }
KeySplit choose_tile_split(const chunk_attn_desc* d, int keys, int cus, int64_t max_parts);
// Both kinds of item of a backward that runs them in one launch, on the same compute units: chooses the pieces of the kinds that are cut by
// themselves (`dq` and `dkv` as they come) anew, or none, with all blocks counted and room for `max_parts` partial results of blocks of either kind.
// (Each kind by itself has room for fewer, and its pieces may crowd out the other kind's blocks.)
void refine_bwd_split(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus, int64_t max_parts, KeySplit* dq, KeySplit* dkv);
// Whether the dK/dV blocks of head_dim 96 and 128, none of them cut, end sooner as kTallKeys keys each (dkv_tall_blocks) than as `keys` each.
constexpr int kTallKeys = 256;
bool tall_pays(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus);
// Whether head_dim 256 runs the pipelined dQ blocks (dq_wide_blocks) by themselves, which start and end more slowly than bwd_dq_kernel's: from walks of 5.5 stages on
// average on.  Backward, bwd_dq_kernel / wide (heads, mean walk): 64 sequences of 70, 8/8 (3) 100 / 105 us; of 170 (5) 190 / 197; of 220 (5.5)
// 283 / 277; four of 256, 8/8 (6) 50 / 49; 148 queries on 595 keys, 8/2 (17) 76 / 72; 32/8 heads: eight sequences of 220 (4) 107 / 111, 64 of 220 (4) 639 / 652,
// 64 of 256 (4.5) 776 / 760; 1024 causal tokens (16.5) 144 / 135; 909 on 5603 keys (161) 638 / 598.
inline bool dq_wide_pays(const Walks& w) { return 2 * w.stages >= 11 * w.items; }
// Whether the forward of head_dim 256 ends sooner with blocks of twice `tile_rows` query rows, 64 per wave (fwd_tall_kernel), than of `tile_rows` (fwd_wide_kernel).
bool fwd_tall_pays(const chunk_attn_desc* d, int tile_rows, int inner, int cus);
// Whether a chunk of head_dim 64 whose dQ and dK/dV are both pipelined runs them in one launch, with dK/dV blocks of kTallKeys keys, rather than in two: where several query heads
// share a key/value head, from 8 steps per walk (`w`, of blocks of 128 keys) on.  One launch to two, geometric mean (chunks): one query head 1.01 (43; 0.94 - 1.05), two 0.97 (260; 1.02 at most),
// three 0.95 (50), four and more 0.93 (141; 1.01 at most); walks of 9 to 30 steps 0.92 - 0.99 (26).  Two launches -> one: 8192 queries on 16384 keys, 32/8 heads, backward, 2998 -> 2718
// us, 8192 causal tokens 1129 -> 1005; what stays: 16317 queries on 16594 keys, 16/16, 1749 (one launch: 1822).
inline bool narrow_tall_pays(int group, const Walks& w) { return group > 1 && w.stages >= 8 * w.items; }
// Whether head_dim 256 runs its pipelined dK/dV blocks, of kWideKeys keys, rather than those of bwd_dkv_kernel, of `keys` (by estimates of both).
constexpr int kWideKeys = 128;
bool wide_pays(const chunk_attn_desc* d, int tile_rows, int inner, int keys, int cus);
// The key-stationary items to run for such a cut, longest walk first, of equal ones those that walk the same tiles side by
// side; `cut` receives the whole items that were cut.
std::vector<DkvItem> cut_items(const std::vector<DkvItem>& wholes, int target, std::vector<DkvItem>* cut);
// The items to run for a cut: pieces of one item are consecutive.  In `wholes`, items that were cut get the number of their
// pieces and their first slot.
std::vector<FwdItem> cut_items(std::vector<FwdItem>& wholes, int target);
// The same for the dQ items; `cut` receives the whole items that were cut.
std::vector<DqItem> cut_items(const std::vector<DqItem>& wholes, int target, std::vector<DqItem>* cut);
// `keys` consecutive key rows per item.  `side_by_side` = 0: every item walks its query tiles upwards.  > 0: the number
// of items of one key/value head that run at the same time; the items of a sequence are then ordered, and given a walk
// direction each, so that those items read the same query rows at about the same time (see plan.cpp).
std::vector<DkvItem> plan_dkv(const chunk_attn_desc* d, int keys, int side_by_side = 0);
// `width`-row tiles of every segment's query range, in segment order, and the number of such tiles of its key (kv) or query range.
std::vector<TileJob> query_tile_jobs(const chunk_attn_desc* d, int width);
int64_t count_tiles(const chunk_attn_desc* d, bool kv, int width);
// Key-row ranges [begin, end) not covered by any segment (to be zero-filled when not accumulating).
std::vector<std::pair<int32_t, int32_t>> uncovered_kv_ranges(const chunk_attn_desc* d);

}  // namespace chunk_attn

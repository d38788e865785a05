// Kernel parameter blocks and launchers (internal to the library).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.hpp"
#include "plan.hpp"

#ifndef DKV_KEYS
#define DKV_KEYS 128
#endif

namespace chunk_attn {

struct FwdParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* o;
  float* lse;
  const FwdItem* items;     // null: in the kernel arguments (FwdArgs)
  const FwdItem* wholes;    // what fwd_merge_kernel goes through: items before cutting (those that were not cut are passed over); or null
  float* parts;             // partial results of the pieces, kPartFloats per (slot, inner index)
  int32_t num_q_heads, num_kv_heads, group;  // group = Hq / Hkv
  int32_t heads_per_wg;                      // query heads of one group handled by one workgroup (a power of two)
  int32_t head_splits;                       // group / heads_per_wg
  int32_t total_q;
  float scale_log2;                          // softmax scale * log2(e)
  float ref_limit;                           // log2 growth of the row maximum past the first tile's with which a block is taken again
  int32_t* taken;                            // 8 block-queue counters of the pipelined forward, zero before the launch (not read
                                             // if there are no more blocks than workgroups)
  unsigned long long* clock_log;             // null, or where the pipelined forward's workgroups log their clocks
};

// Kernel arguments with room for a short list of items behind the parameters: a small chunk's schedule then needs no place in device
// memory and no launch or copy to get there.  (3.6 KB in all; 4 KB are documented for a launch.)
constexpr int kInlineItems = 104;
static_assert(kInlineItems >= kMaxSharedItems);
constexpr size_t kInlineBlob = 3584;  // bytes of a schedule that travels as a kernel argument on its way to device memory
struct FwdArgs {
  FwdParams p;
  int32_t num_blocks;
  FwdItem items[kInlineItems];
};
struct FwdMergeArgs {
  FwdParams p;
  FwdItem wholes[kInlineItems];
};

// rows of query tile per forward work item for a given head layout
// Shape of a query-stationary workgroup (forward and dQ kernels): `waves` waves of 32 query rows each, spread
// over as many query heads of one group as divide both (so that the key/value tiles they stream are shared).
// forward: 4 waves; in the pipelined kernel each wave owns two 32-row query blocks
// head dimensions that always run the software-pipelined kernels (64 does from a size on, pipe_pays)
constexpr bool pipelined(int head_dim) { return head_dim == 96 || head_dim == 128; }
inline int fwd_waves(int) { return 4; }
inline int heads_per_wg(int group, int waves) {
  int h = 1;
  while (h * 2 <= waves && group % (h * 2) == 0) h *= 2;
  return h;
}
// key rows per work item of the dK/dV kernel (32 per pair of waves); head_dim 256 leaves room for two pairs only
inline int dkv_keys(int head_dim) { return head_dim > 128 ? 64 : DKV_KEYS; }
inline int tile_rows(int group, int waves) { return 32 * (waves / heads_per_wg(group, waves)); }

// Workgroups launched by a kernel whose workgroups claim their blocks themselves (device_common.hpp): one (`per_cu`) per CU of the
// current device, and never more than there are blocks.
inline int persistent_grid(int64_t blocks, int per_cu = 1) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    cus = 256;
  return (int)std::max<int64_t>(1, std::min<int64_t>(blocks, (int64_t)cus * per_cu));
}
constexpr int kBlockQueues = 8;  // counters per kernel that claims its blocks
constexpr int kCus = 256;        // compute units of an MI355X (plans that must not depend on where they are made)
// A partial result of one block (256 rows of head_dim 96 or 128, or fewer) in the order in which the kernels hold it: [8 units of 32
// rows][up to 16 accumulator quarters][64 lanes][4] float32; for the forward then [8 units][32 rows] {reference maximum, sum}.
constexpr int kPartRowFloats = 8 * 16 * 64 * 4;
constexpr int kPartFloats = kPartRowFloats + 8 * 32 * 2;
// (a partial result of a dK/dV block has the same size: of 128 keys, units 0 .. 3 are dV, 4 .. 7 dK of 32 keys each; of 64 keys, head_dim
// 256, two units of dV and two of dK, twice as large; head_dim 64 fills half of each unit)
constexpr int part_unit_floats(int head_dim) { return head_dim > 128 ? 2 * 4096 : 4096; }

// Whether a query-stationary kernel of head_dim 64 runs as the pipelined one: its workgroups start and end more slowly than
// the other kernel's, which has three of them on a CU, and it puts twice the rows on a block.  So it needs two blocks per CU,
// walks of 100 stages on average (64 from four blocks per CU on and 45 from eight: more blocks even out better), and no walk
// that alone takes longer than the 512 workgroups' even share of all (but for a tenth).  Between three and four blocks per CU
// the second round is nearly as long as with four, and the other kernel's smaller blocks fill the chip better.
// Measured forward, other -> pipelined, 32/8 heads unless noted (blocks, mean and longest walk): 8192 queries on 16384 keys
// (1024, 384, 512) 906 -> 859 us; four sequences of 4096 (2048, 65, 128) 390 -> 377; ten of 3000 (3760, 47) 473 -> 450; eight
// of 2048 (2048, 34) 203 -> 210; 16 of 1024 (2048, 18) 128 -> 148; 4096 queries on 8192 keys (512, 193, 256) 243 -> 253; 5000
// on 6000 (632, 110, 188) 180 -> 190; 64/8: 2048 on 16384 (512, 480, 512) 568 -> 526, 3000 on 19000 (752, 548, 594) 956 -> 822,
// 3600 on 13000 (900, 350, 406) 713 -> 777; 8/8: three sequences of 6000 (576, 98, 188) 158 -> 194, four of 4096 (512, 68,
// 128) 120 -> 137.  dQ is less sensitive: the same rule serves it.
inline bool pipe_pays(const Walks& w, int inner) {
  const int64_t blocks = w.items * inner, mean = blocks >= 8 * kCus ? 45 : blocks >= 4 * kCus ? 64 : 100;
  if (blocks < 2 * kCus || (blocks > 3 * kCus && blocks < 4 * kCus)) return false;
  return w.stages >= mean * w.items && 10 * w.stages * inner >= 9 * 2 * kCus * w.longest;
}

// Events armed by chunk_attn_profile_events for the calling thread (null when disarmed).
struct ProfileEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
ProfileEvents& profile_events();

// Pointers of one backward call (device memory, caller-owned).
struct BwdArgs {
  const __bf16 *q, *k, *v, *o, *d_o;
  const float* lse;
  __bf16 *dq, *dk, *dv;
  bool accumulate;
  bool dkv_f32;  // dk / dv are fp32 arrays
  char* workspace;
};

// Host-side plan of one backward call and the layout of its workspace:
// [dQ items | dQ items that were cut | dK/dV items | dK/dV items that were cut | 64-row query-tile jobs | block-queue counters | items of the
// one-pass backward, if it runs] (one uploaded blob), then the LSE and D arrays padded to 64-row tiles.
struct BwdPlan {
  KeySplit split;                // head_dim 96 and 128: how the dQ walks are cut
  std::vector<DqItem> dq_items;  // with the pieces of walks that are cut
  std::vector<DqItem> dq_cut;    // the whole items that were cut
  KeySplit dkv_split;            // the same for the dK/dV walks
  std::vector<DkvItem> dkv_cut;
  std::vector<DkvItem> dkv_items;
  std::vector<TileJob> qjobs;
  int64_t q_tiles = 0;
  size_t n_dq_cut = 0, n_dkv_cut = 0;
  size_t dq_items_off = 0, dq_cut_off = 0, dkv_items_off = 0, dkv_cut_off = 0, qjobs_off = 0, queues_off = 0, upload_bytes = 0, blob_bytes = 0;
  size_t lse2p_off = 0, dsp_off = 0, dq_parts_off = 0, total = 0;
  // (head_dim 96 and 128 always; dQ: 64 where pipe_pays; dK/dV: 64 where dkv_pipe_pays, 256 where wide_pays)
  bool dq_pipe = false, dkv_pipe = false;  // the pipelined kernels run
  bool dq_wide = false;                    // head_dim 256: bwd_dq_wide_kernel runs
  int dq_waves = 0;                        // 32-row units of a dQ workgroup
  bool dq_first = false;                   // both kinds in one launch: the dQ blocks start before the dK/dV blocks
  bool dkv_tall = false;                   // head_dim 64, 96 and 128: the dK/dV blocks are those of dkv_tall_blocks
  bool dkv_in_step = false;                // head_dim 96 and 128: long dK/dV walks start in groups (dkv_pipe_blocks, dkv_tall_blocks)
  int share_waves = 0;                     // > 0: launch_bwd_share runs instead, with so many waves per workgroup
  bool in_turn = false;                    // head_dim 96 and 128: a launch per kind, whose partial results take the same place
  // one-pass backward (head_dim 128): its items and workgroup order travel at the end of the blob; then the per-wave
  // progress counters and the status word (cleared by a kernel on every call) and the float32 dQ tiles
  bool fused = false;
  FusedPlan fplan;
  int64_t qt32_tiles = 0;
  size_t fitems_off = 0, forder_off = 0, q32jobs_off = 0, fprog_off = 0, fprog_bytes = 0, fdq_off = 0;
};
constexpr size_t kFusedSinkBytes = 64 * 16384;  // scratch dQ tiles of the one-pass backward, behind its status word
constexpr int kNumXcd = 8;  // XCDs of an MI355X: workgroup b runs on XCD b % 8

// keys per dK/dV block of a plan that runs no kernel of the small chunks
int dkv_block_keys(const BwdPlan& plan, int head_dim);
// 0: the library's choice, 1: the two-kernel backward, 2: the one-pass backward (head_dim 128 only)
int bwd_mode();
// Device memory the caller has set aside for the clock logs of the pipelined kernels (null: none), and the section
// of kernel `which` in it (0 forward, 1 dQ, 2 dK/dV), kClockLogEntries values of 8 bytes each.
constexpr size_t kClockLogEntries = 4 * 1024;
unsigned long long* clock_log(int which);
hipError_t launch_bwd_fused(const chunk_attn_desc* d, const BwdArgs& a, const BwdPlan& plan, const float* lse2p, const float* dsp,
                            hipStream_t stream);
// Fills the offsets (and, if with_plan, the schedules) for a validated descriptor.  kCutInPlace: only where the partial results of each kind fit
// the room that head_dim 96 and 128 keep for dQ tiles anyway (workspaces of that size may be known to callers); kCutNone: no walk is cut.
enum Cut { kCutNone, kCutInPlace, kCutFine };
// share_dim: not 0: the kernel of the small chunks may run (share_waves > 0), at this head_dim (d's is 128 for 96); it needs no schedule; the sizes are the other kernels' either way.
void bwd_layout(const chunk_attn_desc* d, BwdPlan& plan, bool with_plan, Cut cut = kCutFine, int share_dim = 0);
// The host image of the blob at the start of the workspace.
std::vector<char> bwd_blob(const BwdPlan& plan);
// Zeroes the rows of dK and dV that no segment covers, unless the call accumulates.
hipError_t zero_uncovered(const chunk_attn_desc* d, const BwdArgs& a, hipStream_t stream);
// The backward of a small chunk in one launch that needs no workspace, `waves` waves per workgroup (choose_shared_waves).
hipError_t launch_bwd_share(const chunk_attn_desc* d, const BwdArgs& a, int waves, hipStream_t stream);
// Enqueues the backward kernels.  A blob of more than kInlineBlob bytes must already be on its way to the workspace on `stream`.
hipError_t launch_bwd(const chunk_attn_desc* d, const BwdArgs& a, const BwdPlan& plan, const std::vector<char>& blob, hipStream_t stream);

// The lists of one forward call: `num_blocks` blocks (items x inner); the host copies of the items and of the cut ones among the whole
// items are read only where the kernel arguments carry them.
struct FwdLists {
  int num_blocks = 0, num_items = 0;
  int num_wholes = 0;  // 0: nothing is cut
  const FwdItem *items = nullptr, *wholes = nullptr;
};
// workgroups of the pipelined forward on a CU
constexpr int fwd_per_cu(int head_dim) { return head_dim == 64 ? 2 : 1; }
// kFwdPipe: the pipelined kernel (and the launch that puts cut walks together); kFwdShare: fwd_share_kernel (head_dim 64, 96 and 128); kFwdPlain: fwd_kernel
// at head_dim 64, fwd_wide_kernel at 256; kFwdTall: fwd_tall_kernel (256).
enum FwdKind { kFwdPlain, kFwdPipe, kFwdShare, kFwdTall };
hipError_t launch_fwd(const FwdParams& p, int head_dim, FwdKind kind, const FwdLists& lists, hipStream_t stream);

}  // namespace chunk_attn

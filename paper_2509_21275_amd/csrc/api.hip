// C ABI of the chunk-attention library (include/chunk_attn.h): argument checks, workspace carving,
// schedule upload and kernel launches.  No device memory is allocated here; the only memory the
// library owns is a small ring of pinned host buffers through which tile schedules are uploaded
// (released by chunk_attn_shutdown).
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>

#include "kernels.hpp"

using namespace chunk_attn;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

thread_local std::string g_last_hip_error;

int hip_fail(hipError_t e, const char* what) {
  g_last_hip_error = std::string(what) + ": " + hipGetErrorString(e);
  return CHUNK_ATTN_HIP_ERROR;
}

// Schedules reach the device as kernel arguments where they are small (the forward's items with the forward itself, the backward's
// blob with its pre-pass, a forward blob with a launch of its own), else through pinned staging buffers.
struct InlineBlob {
  uint4 data[kInlineBlob / 16];
};
__global__ __launch_bounds__(256) void upload_inline_kernel(InlineBlob blob, uint4* dst, int n16) {
  if ((int)threadIdx.x < n16) dst[threadIdx.x] = blob.data[threadIdx.x];
}
static_assert(kInlineBlob <= 256 * 16, "one workgroup copies it");
__global__ __launch_bounds__(256) void upload_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int n16) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

// Pinned staging buffers for the schedule uploads.  A buffer is reused only after the copy that read it has
// completed; while the GPU is still busy with earlier calls the pool grows (up to kMaxBytes) instead of making the
// caller wait, so that the host can plan and enqueue ahead of the GPU.  Buffers come in power-of-two sizes and are
// never freed on the way (freeing pinned memory waits for the device): a buffer that is too small is simply skipped.
struct StagingRing {
  static constexpr size_t kMaxBytes = (size_t)256 << 20;
  static constexpr size_t kMinSlot = (size_t)256 << 10;
  struct Slot {
    void* host = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;
    bool in_flight = false;
  };
  std::vector<Slot> slots;
  size_t next = 0, total = 0;
  std::mutex mu;

  // Copies `bytes` (a multiple of 16) from src into pinned memory and enqueues the upload to `dst` on `stream`: a small kernel that reads
  // the pinned memory, which takes 3 us where the runtime's copy takes 4 (by a kernel, and 5 until the next one starts) to 20
  // (by a copy engine, from 16 KB on).
  hipError_t upload(void* dst, const void* src, size_t bytes, hipStream_t stream) {
    std::lock_guard<std::mutex> lock(mu);
    hipError_t e;
    size_t want = kMinSlot;
    while (want < bytes) want *= 2;
    // a completed buffer that is large enough, oldest first (copies on one stream complete in order, so after a few
    // pending ones the rest are pending too)
    Slot* s = nullptr;
    int pending_seen = 0;
    for (size_t i = 0; i < slots.size() && !s && pending_seen < 4; ++i) {
      const size_t idx = (next + i) % slots.size();
      Slot& c = slots[idx];
      if (c.cap < bytes) continue;
      if (c.in_flight) {
        e = hipEventQuery(c.ev);
        if (e == hipSuccess) c.in_flight = false;
        else if (e != hipErrorNotReady) return e;
        else ++pending_seen;
      }
      if (!c.in_flight) {
        s = &c;
        next = (idx + 1) % slots.size();
      }
    }
    if (!s && total + want <= kMaxBytes) {  // grow
      Slot n;
      if ((e = hipHostMalloc(&n.host, want, hipHostMallocPortable | hipHostMallocMapped)) != hipSuccess) return e;
      n.cap = want;
      if ((e = hipEventCreateWithFlags(&n.ev, hipEventDisableTiming)) != hipSuccess) return e;
      total += want;
      slots.push_back(n);
      s = &slots.back();
    }
    if (!s) {  // the pool is at its limit: wait for the oldest buffer that is large enough
      for (size_t i = 0; i < slots.size() && !s; ++i) {
        Slot& c = slots[(next + i) % slots.size()];
        if (c.cap >= bytes) s = &c;
      }
      if (s) {
        if (s->in_flight && (e = hipEventSynchronize(s->ev)) != hipSuccess) return e;
        s->in_flight = false;
      } else {  // none is: replace the oldest one (this waits for the device)
        s = &slots[next % slots.size()];
        if (s->in_flight && (e = hipEventSynchronize(s->ev)) != hipSuccess) return e;
        s->in_flight = false;
        if ((e = hipHostFree(s->host)) != hipSuccess) return e;
        total -= s->cap;
        s->host = nullptr;
        s->cap = 0;
        if ((e = hipHostMalloc(&s->host, want, hipHostMallocPortable | hipHostMallocMapped)) != hipSuccess) return e;
        s->cap = want;
        total += want;
      }
    }
    std::memcpy(s->host, src, bytes);
    void* from = nullptr;
    if ((e = hipHostGetDevicePointer(&from, s->host, 0)) != hipSuccess) return e;
    const int n16 = (int)(bytes / 16);
    hipLaunchKernelGGL(upload_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, stream, static_cast<const uint4*>(from),
                       static_cast<uint4*>(dst), n16);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipEventRecord(s->ev, stream)) != hipSuccess) return e;
    s->in_flight = true;
    return hipSuccess;
  }

  // Waits for the uploads still reading the buffers and frees them all; the ring starts again from nothing.
  hipError_t release() {
    std::lock_guard<std::mutex> lock(mu);
    hipError_t first = hipSuccess;
    for (Slot& c : slots) {
      hipError_t e = hipSuccess;
      if (c.in_flight) e = hipEventSynchronize(c.ev);
      if (e == hipSuccess && c.ev) e = hipEventDestroy(c.ev);
      if (e == hipSuccess && c.host) e = hipHostFree(c.host);
      if (e != hipSuccess && first == hipSuccess) first = e;
    }
    slots.clear();
    next = total = 0;
    return first;
  }
};
StagingRing g_ring;

hipError_t upload_schedule(void* dst, const std::vector<char>& blob, hipStream_t stream) {
  if (blob.size() > kInlineBlob) return g_ring.upload(dst, blob.data(), blob.size(), stream);
  InlineBlob a;
  std::memcpy(a.data, blob.data(), blob.size());
  hipLaunchKernelGGL(upload_inline_kernel, dim3(1), dim3(256), 0, stream, a, static_cast<uint4*>(dst), (int)(blob.size() / 16));
  return hipGetLastError();
}

// log2 growth of a row's maximum past the first key tile's at which the pipelined forward takes the row's block again with
// the true maximum: bf16 probabilities and fp32 sums hold 2^60 with room to spare
std::atomic<float> g_fwd_rescale_limit{60.0f};

std::atomic<int> g_bwd_mode{0};
std::atomic<unsigned long long*> g_clock_log{nullptr};

inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + b_bytes && y < x + a_bytes;
}
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// ---- head_dim 96 ----
// The kernels have instantiations of their own for it.  Workspaces are laid out and sized as for head_dim 128 plus padded
// copies of the operands, which the one-pass backward (head_dim 128 only, chunk_attn_test_set_bwd_mode) still runs on: a
// head of 96 is a head of 128 whose last 32 columns are zero.  Zero columns of Q and K add nothing to a score, zero columns
// of V and dO give zero columns of O, dV and (through dS K, dS^T Q) of dQ and dK, and D_i = <dO_i, O_i> is unchanged,
// so every result is the 96-wide one exactly, with the softmax scale the caller gave.
constexpr int kNarrowDim = 96, kPaddedDim = 128;

inline bool is_narrow(const chunk_attn_desc* d) { return d->head_dim == kNarrowDim; }
inline chunk_attn_desc widened(const chunk_attn_desc* d) {
  chunk_attn_desc w = *d;
  if (is_narrow(d)) w.head_dim = kPaddedDim;
  return w;
}
inline size_t padded_bytes(int64_t rows, int heads, size_t elem) { return align_up((size_t)rows * heads * kPaddedDim * elem); }

// Forward workspace: [work items | whole items that were cut | block-queue counters (zero)] (uploaded as one blob, unless
// the kernel arguments carry the items) then, for 96 and 128, the partial results of items whose walks are cut.
struct FwdLayout {
  int tile_rows;
  bool pipe;       // the pipelined kernel runs (head_dim 96 and 128, and 64 from a number of blocks on), unless
  int share;       // > 0: fwd_share_kernel runs, its workgroups taking so many heads each
  bool tall;       // head_dim 256: fwd_tall_kernel runs
  KeySplit split;  // pipelined kernel: how the walks are cut
  size_t n_items, n_wholes, wholes_off, queues_off, blob_bytes, parts_off, total;
  int64_t blocks;
  std::vector<FwdItem> items, cut;  // what runs, and the whole items that were cut
};

// Scratch memory of the forward that allocates nothing (chunk_attn_fwd_static), below.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;

// The lists of a layout whose sizes are known.
void fill_fwd_lists(const chunk_attn_desc* d, FwdLayout& L) {
  if (L.share > 0) {
    L.items = plan_fwd(d, 32);
    return;
  }
  std::vector<FwdItem> wholes = plan_fwd(d, L.tile_rows);
  L.items = cut_items(wholes, L.split.target);
  for (const FwdItem& w : wholes)
    if (w.part >= 0) L.cut.push_back(w);
}

// `may_cut`: false: no walk is cut whatever the chunk.  Partial results take the room of a transposed copy of V, or up to the
// static forward's scratch memory where that is smaller.  The cut is a function of the chunk alone, so that both entry points give the same
// bits; a workspace too small for it, which older sizes may be, runs uncut.
void layout_fwd(const chunk_attn_desc* desc, FwdLayout& L, bool with_plan, bool may_cut = true) {
  const chunk_attn_desc wide = widened(desc), *d = &wide;
  const int group = d->num_q_heads / d->num_kv_heads;
  const int inner = d->num_kv_heads * (group / heads_per_wg(group, fwd_waves(d->head_dim)));
  L.tile_rows = 2 * tile_rows(group, fwd_waves(d->head_dim));  // two 32-row blocks per wave
  Walks walks = count_walks(d, L.tile_rows);
  const bool pipe = L.pipe = pipelined(d->head_dim) || (d->head_dim == 64 && pipe_pays(walks, inner));
  if (!pipe) {
    L.tile_rows /= 2;
    walks = count_walks(d, L.tile_rows);
  }
  L.n_wholes = (size_t)walks.items;
  // (as much as a transposed copy of V takes, which no kernel makes any more: the sizes stay what callers know)
  const size_t room = align_up((size_t)count_tiles(d, true, 64) * d->num_kv_heads * d->head_dim * 64 * sizeof(__bf16));
  const size_t part_bytes = (size_t)inner * kPartFloats * sizeof(float);
  // the fixed part of a layout with n items to run: [items | whole items, if any was cut | the block-queue counters (zero)]
  auto place = [&](size_t n_items) {
    L.n_items = n_items;
    L.wholes_off = n_items * sizeof(FwdItem);
    L.queues_off = L.wholes_off + (n_items == L.n_wholes ? 0 : L.n_wholes * sizeof(FwdItem));
    L.blob_bytes = L.queues_off + kBlockQueues * sizeof(int32_t);
    L.parts_off = align_up(L.blob_bytes);
  };
  L.split = KeySplit{};
  place(L.n_wholes);
  const size_t uncut_total = L.parts_off + room;
  // (not 64: with the two blocks per CU that pipe_pays asks for its walks are even enough; cut, 3032 queries on 51484 keys,
  // 64/64 heads, took 2587 us instead of 2443)
  if (pipelined(d->head_dim) && may_cut) {
    const size_t limit = std::max(uncut_total, kStaticScratchBytes);
    L.split = choose_key_split(d, L.tile_rows, inner, kCus, (int64_t)((limit - L.parts_off) / part_bytes));
    if (L.split.target > 0) {
      place((size_t)L.split.pieces);
      if (L.parts_off + align_up((size_t)L.split.parts * part_bytes) > limit) {  // (the longer item list takes room, too)
        L.split = KeySplit{};
        place(L.n_wholes);
      }
    }
  }
  L.blocks = (int64_t)L.n_items * inner;
  L.total = std::max(uncut_total, L.parts_off + align_up((size_t)L.split.parts * part_bytes));
  if (is_narrow(desc))  // (as much as with padded copies of Q, K, V and O)
    L.total = std::max(L.total, uncut_total + 2 * padded_bytes(d->total_q, d->num_q_heads, 2) + 2 * padded_bytes(d->total_kv, d->num_kv_heads, 2));
  L.tall = d->head_dim == 256 && fwd_tall_pays(d, L.tile_rows, inner, kCus);
  if (L.tall) {  // (the size stays that of the other kernel's items, of which there are more)
    L.tile_rows *= 2;
    L.n_wholes = (size_t)count_walks(d, L.tile_rows).items;
    place(L.n_wholes);
    L.blocks = (int64_t)L.n_items * inner;
  }
  // (the layout of the workspace stays the other kernel's, so that its size does)
  L.share = may_cut && bwd_mode() == 0 ? choose_shared_heads(desc, walks, inner, pipe, L.split) : 0;
  if (L.share > 0) {
    L.n_items = (size_t)count_walks(d, 32).items;
    L.blocks = (int64_t)L.n_items * (d->num_q_heads / L.share);
  }
  if (with_plan) fill_fwd_lists(desc, L);
}

// ---- the forward that allocates nothing (chunk_attn_fwd_static) ----
// Its scratch memory is this array instead of a caller's workspace: every GPU the library runs on holds its own copy, at
// its own address, until the process ends.  Host code never uses the array's name as an address: static_scratch() asks
// the runtime for the device address once per device and hands that out.
constexpr int kStaticMaxSegments = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};  // per device

hipError_t static_scratch(char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if ((e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    g_scratch_ptr[dev] = ptr;
  }
  *out = static_cast<char*>(g_scratch_ptr[dev]);
  return hipSuccess;
}

// The forward's schedule made on the device from a segment table passed by value: work items in segment order (their
// order does not change any result) and the pieces of those that are cut, and the block-queue counters cleared.
// (Short lists of items travel as kernel arguments of the forward itself instead: fwd_inline.)
struct StaticSegs {
  chunk_attn_seg seg[kStaticMaxSegments];
};
__global__ __launch_bounds__(256) void plan_fwd_static_kernel(StaticSegs segs, int n_seg, int tile_rows, FwdItem* wholes,
                                                              int n_wholes, FwdItem* items, int target, int32_t* queues) {
  __shared__ int item0[kStaticMaxSegments + 1];
  __shared__ int wave_items[4], wave_parts[4];
  if (threadIdx.x == 0) {
    int ni = 0;
    for (int t = 0; t < n_seg; ++t) {
      item0[t] = ni;
      ni += (segs.seg[t].q_len + tile_rows - 1) / tile_rows;
    }
    item0[n_seg] = ni;
  }
  __syncthreads();
  // 256 whole items at a time; `items_before` and `parts_before` count the pieces of the items before them
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int items_before = 0, parts_before = 0;
  for (int x0 = 0; x0 < n_wholes; x0 += 256) {
    const int x = x0 + threadIdx.x;
    FwdItem it{};
    int stages = 0, n = 0;
    if (x < n_wholes) {
      int t = 0;
      while (t + 1 < n_seg && item0[t + 1] <= x) ++t;
      const chunk_attn_seg s = segs.seg[t];
      const int i0 = (x - item0[t]) * tile_rows;
      it.q_row0 = s.q_start + i0;
      it.q_rows = min(tile_rows, s.q_len - i0);
      it.kv_row0 = s.kv_start;
      it.n0 = s.kv_len - s.q_len + i0 + 1;
      it.keys = s.kv_len;
      if (target <= 0) {  // nothing is cut: no pieces to number
        it.part = -1;
        items[x] = it;
      } else {
        stages = walk_stages(it.n0, it.q_rows);
        n = piece_count(stages, it.n0, target);
      }
    }
    if (target <= 0) continue;
    int item = n, part = n > 1 ? n : 0;  // inclusive sums over the items up to this one
    for (int o = 1; o < 64; o *= 2) {
      const int a = __shfl_up(item, o), b = __shfl_up(part, o);
      if (lane >= o) {
        item += a;
        part += b;
      }
    }
    if (lane == 63) {
      wave_items[wave] = item;
      wave_parts[wave] = part;
    }
    __syncthreads();
    item += items_before - n;
    part += parts_before - (n > 1 ? n : 0);
    for (int w = 0; w < 4; ++w) {
      if (w < wave) {
        item += wave_items[w];
        part += wave_parts[w];
      }
      items_before += wave_items[w];
      parts_before += wave_parts[w];
    }
    __syncthreads();
    for (int k = 0; k < n; ++k) {
      const int b = piece_begin(stages, n, k) * kStageKeys;
      FwdItem p = it;
      p.kv_row0 += b;
      p.n0 -= b;
      p.keys = (k + 1 < n ? piece_begin(stages, n, k + 1) * kStageKeys : it.keys) - b;
      p.part = n > 1 ? part + k : -1;
      items[item + k] = p;
    }
    if (x < n_wholes) {
      it.pieces = n;
      it.part = n > 1 ? part : -1;
      wholes[x] = it;
    }
  }
  if (threadIdx.x < kBlockQueues) queues[threadIdx.x] = 0;
}

// dst[row][0 .. out_chunks) = src[row][0 .. in_chunks) followed by zero chunks
__global__ __launch_bounds__(256) void pad_rows_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n_out,
                                                       int in_chunks, int out_chunks) {
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n_out; x += (int64_t)gridDim.x * 256) {
    const int64_t row = x / out_chunks;
    const int c = (int)(x - row * out_chunks);
    dst[x] = c < in_chunks ? src[row * in_chunks + c] : make_uint4(0, 0, 0, 0);
  }
}
// dst[row][0 .. in_chunks) = src[row][0 .. in_chunks) of rows that are out_chunks wide
__global__ __launch_bounds__(256) void unpad_rows_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int64_t n_in,
                                                         int in_chunks, int out_chunks) {
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n_in; x += (int64_t)gridDim.x * 256) {
    const int64_t row = x / in_chunks;
    const int c = (int)(x - row * in_chunks);
    dst[x] = src[row * out_chunks + c];
  }
}
inline int copy_grid(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 256 * 16); }
// rows = tensor rows * heads; elem = bytes per element
hipError_t pad_rows(const void* src, void* dst, int64_t rows, size_t elem, hipStream_t stream) {
  const int in_chunks = kNarrowDim * (int)elem / 16, out_chunks = kPaddedDim * (int)elem / 16;
  const int64_t n = rows * out_chunks;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(pad_rows_kernel, dim3(copy_grid(n)), dim3(256), 0, stream, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), n, in_chunks, out_chunks);
  return hipGetLastError();
}
hipError_t unpad_rows(const void* src, void* dst, int64_t rows, size_t elem, hipStream_t stream) {
  const int in_chunks = kNarrowDim * (int)elem / 16, out_chunks = kPaddedDim * (int)elem / 16;
  const int64_t n = rows * in_chunks;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(unpad_rows_kernel, dim3(copy_grid(n)), dim3(256), 0, stream, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), n, in_chunks, out_chunks);
  return hipGetLastError();
}

// Padded copies at the head of a backward workspace, the widened call's own workspace behind them.
struct NarrowBwdLayout {
  size_t q_off, k_off, v_off, o_off, do_off, dq_off, dk_off, dv_off, inner_off, total;
};
// dk / dv copies are sized for float32, whichever entry point is called later
NarrowBwdLayout narrow_bwd_layout(const chunk_attn_desc* d, size_t inner_bytes) {
  const size_t qb = padded_bytes(d->total_q, d->num_q_heads, 2), kb = padded_bytes(d->total_kv, d->num_kv_heads, 2);
  const size_t gb = padded_bytes(d->total_kv, d->num_kv_heads, 4);
  NarrowBwdLayout N;
  N.q_off = 0;
  N.k_off = qb;
  N.v_off = N.k_off + kb;
  N.o_off = N.v_off + kb;
  N.do_off = N.o_off + qb;
  N.dq_off = N.do_off + qb;
  N.dk_off = N.dq_off + qb;
  N.dv_off = N.dk_off + gb;
  N.inner_off = N.dv_off + gb;
  N.total = N.inner_off + inner_bytes;
  return N;
}

// Whether the forward's kernel arguments carry its items: there is room for them, and no block is claimed through a counter in device
// memory, which would have to be cleared first.  Saves the launch that
// would bring them, 3 us and as much of host time.  Forward and backward of 557 causal tokens, 32/8 heads, without any upload by the
// runtime, with workgroups that find their block without a counter, and without the forward's second launch: 92 -> 73 us; 439
// tokens, 8/2 heads, 87 -> 68; the static forward of 1501 + 203 keys next to 611 short rows 41 -> 30 us.
bool fwd_inline(const FwdLayout& L, int head_dim) {
  if (L.share > 0) return true;
  const bool claims = L.pipe || head_dim == 256;
  return L.n_items <= (size_t)kInlineItems && (!claims || L.blocks <= persistent_grid(L.blocks, fwd_per_cu(head_dim)));
}

// Parameters and lists of a forward whose scratch memory is `ws`.
FwdParams fwd_params(const chunk_attn_desc* desc, const FwdLayout& L, char* ws, bool items_inline, const void* q, const void* k, const void* v,
                     void* o, float* lse) {
  FwdParams p;
  p.q = static_cast<const __bf16*>(q);
  p.k = static_cast<const __bf16*>(k);
  p.v = static_cast<const __bf16*>(v);
  p.o = static_cast<__bf16*>(o);
  p.lse = lse;
  p.items = items_inline ? nullptr : reinterpret_cast<const FwdItem*>(ws);
  p.wholes = items_inline ? nullptr : reinterpret_cast<const FwdItem*>(ws + L.wholes_off);
  p.parts = reinterpret_cast<float*>(ws + L.parts_off);
  p.num_q_heads = desc->num_q_heads;
  p.num_kv_heads = desc->num_kv_heads;
  p.group = desc->num_q_heads / desc->num_kv_heads;
  p.heads_per_wg = L.share > 0 ? L.share : heads_per_wg(p.group, fwd_waves(desc->head_dim));
  p.head_splits = p.group / p.heads_per_wg;
  p.total_q = desc->total_q;
  p.scale_log2 = desc->softmax_scale * 1.4426950408889634f;
  p.taken = reinterpret_cast<int32_t*>(ws + L.queues_off);
  p.clock_log = clock_log(0);
  p.ref_limit = g_fwd_rescale_limit.load();
  return p;
}
FwdKind fwd_kind(const FwdLayout& L) { return L.share > 0 ? kFwdShare : L.tall ? kFwdTall : L.pipe ? kFwdPipe : kFwdPlain; }
FwdLists fwd_lists(const FwdLayout& L) {
  FwdLists l;
  l.num_blocks = (int)L.blocks;
  l.num_items = (int)L.n_items;
  l.num_wholes = (int)L.cut.size();
  l.items = L.items.data();
  l.wholes = L.cut.data();
  return l;
}
}  // namespace

namespace chunk_attn {
int bwd_mode() { return g_bwd_mode.load(); }
unsigned long long* clock_log(int which) {
  unsigned long long* base = g_clock_log.load();
  return base ? base + (size_t)which * kClockLogEntries : nullptr;
}
ProfileEvents& profile_events() {
  static thread_local ProfileEvents ev;
  return ev;
}
}  // namespace chunk_attn

extern "C" {

int chunk_attn_profile_events(void* start_event, void* stop_event) {
  profile_events().start = static_cast<hipEvent_t>(start_event);
  profile_events().stop = static_cast<hipEvent_t>(stop_event);
  return CHUNK_ATTN_OK;
}

int chunk_attn_validate(const chunk_attn_desc* desc) { return validate(desc); }

int chunk_attn_shutdown(void) {
  const hipError_t e = g_ring.release();
  return e == hipSuccess ? CHUNK_ATTN_OK : hip_fail(e, "releasing the staging buffers");
}

int chunk_attn_test_set_bwd_mode(int mode) {
  if (mode < 0 || mode > 2) return CHUNK_ATTN_INVALID_ARG;
  g_bwd_mode.store(mode);
  return CHUNK_ATTN_OK;
}

int chunk_attn_measure_set_clock_log(void* device_buffer, size_t bytes) {
  if (device_buffer == nullptr) {
    g_clock_log.store(nullptr);
    return CHUNK_ATTN_OK;
  }
  if ((reinterpret_cast<uintptr_t>(device_buffer) & 7) != 0) return CHUNK_ATTN_INVALID_ARG;
  if (bytes < 3 * kClockLogEntries * sizeof(unsigned long long)) return CHUNK_ATTN_WORKSPACE_TOO_SMALL;
  g_clock_log.store(static_cast<unsigned long long*>(device_buffer));
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_bwd_status_offset(const chunk_attn_desc* desc, size_t* offset) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!offset) return CHUNK_ATTN_INVALID_ARG;
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  bwd_layout(&w, P, false);
  *offset = P.fprog_off + P.fprog_bytes - kFusedSinkBytes - 256;
  if (is_narrow(desc)) *offset += narrow_bwd_layout(desc, P.total).inner_off;
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_routes(const chunk_attn_desc* desc, int32_t* routes) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!routes) return CHUNK_ATTN_INVALID_ARG;
  FwdLayout L;
  layout_fwd(desc, L, false);
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  bwd_layout(&w, P, false, kCutFine, bwd_mode() == 0 ? desc->head_dim : 0);
  *routes = L.share > 0 ? CHUNK_ATTN_ROUTE_FWD_SHARED : (L.pipe ? CHUNK_ATTN_ROUTE_FWD_PIPELINED : 0) | (L.split.target > 0 ? CHUNK_ATTN_ROUTE_FWD_CUT : 0);
  if (P.fused || P.share_waves > 0) {
    *routes |= P.fused ? CHUNK_ATTN_ROUTE_ONE_PASS : CHUNK_ATTN_ROUTE_BWD_SHARED;
    return CHUNK_ATTN_OK;
  }
  *routes |= (P.dq_pipe ? CHUNK_ATTN_ROUTE_DQ_PIPELINED : 0) | (P.split.target > 0 ? CHUNK_ATTN_ROUTE_DQ_CUT : 0) |
             (P.dkv_pipe ? CHUNK_ATTN_ROUTE_DKV_PIPELINED : 0) | (P.dkv_split.target > 0 ? CHUNK_ATTN_ROUTE_DKV_CUT : 0);
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_dkv_keys(const chunk_attn_desc* desc, int32_t* keys) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!keys) return CHUNK_ATTN_INVALID_ARG;
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  bwd_layout(&w, P, false, kCutFine, bwd_mode() == 0 ? desc->head_dim : 0);
  *keys = P.share_waves > 0 ? 32 : dkv_block_keys(P, w.head_dim);
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_dkv_in_step(const chunk_attn_desc* desc, int32_t* in_step) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!in_step) return CHUNK_ATTN_INVALID_ARG;
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  bwd_layout(&w, P, true, kCutFine, bwd_mode() == 0 ? desc->head_dim : 0);
  *in_step = P.dkv_in_step ? 1 : 0;
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_fwd_rows(const chunk_attn_desc* desc, int32_t* rows) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!rows) return CHUNK_ATTN_INVALID_ARG;
  FwdLayout L;
  layout_fwd(desc, L, false);
  *rows = L.share > 0 ? 32 : L.pipe || L.tall ? 64 : 32;
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_shared_heads(const chunk_attn_desc* desc, int32_t* heads) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!heads) return CHUNK_ATTN_INVALID_ARG;
  FwdLayout L;
  layout_fwd(desc, L, false);
  *heads = L.share;
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_shared_waves(const chunk_attn_desc* desc, int32_t* waves) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!waves) return CHUNK_ATTN_INVALID_ARG;
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  bwd_layout(&w, P, false, kCutFine, bwd_mode() == 0 ? desc->head_dim : 0);
  *waves = P.share_waves;
  return CHUNK_ATTN_OK;
}

int chunk_attn_test_set_fwd_rescale_limit(float log2_growth) {
  g_fwd_rescale_limit.store(log2_growth);
  return CHUNK_ATTN_OK;
}

int64_t chunk_attn_pair_count(const chunk_attn_desc* desc) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  return pair_count(desc);
}

const char* chunk_attn_strerror(int code) {
  switch (code) {
    case CHUNK_ATTN_OK: return "ok";
    case CHUNK_ATTN_INVALID_ARG: return "invalid argument (null pointer, non-positive size or bad scale)";
    case CHUNK_ATTN_UNSUPPORTED: return "unsupported shape (head_dim must be 64, 96, 128 or 256; num_kv_heads must divide num_q_heads)";
    case CHUNK_ATTN_BAD_SEGMENT: return "bad segment table";
    case CHUNK_ATTN_WORKSPACE_TOO_SMALL: return "workspace too small (see chunk_attn_workspace_bytes)";
    case CHUNK_ATTN_TOO_LARGE:
      return "chunk too large for chunk_attn_fwd_static (at most 64 segments and 16 MiB of forward scratch, see "
             "chunk_attn_workspace_bytes); use chunk_attn_fwd with a workspace";
    case CHUNK_ATTN_HIP_ERROR: {
      static thread_local std::string msg;
      msg = "HIP error: " + g_last_hip_error;
      return msg.c_str();
    }
    default: return "unknown error code";
  }
}

int chunk_attn_workspace_bytes(const chunk_attn_desc* desc, size_t* fwd_bytes, size_t* bwd_bytes) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (fwd_bytes) {
    FwdLayout L;
    layout_fwd(desc, L, false);
    *fwd_bytes = L.total;
  }
  if (bwd_bytes) {
    const chunk_attn_desc w = widened(desc);
    BwdPlan P;
    bwd_layout(&w, P, false);
    *bwd_bytes = is_narrow(desc) ? narrow_bwd_layout(desc, P.total).total : P.total;
  }
  return CHUNK_ATTN_OK;
}

int chunk_attn_fwd(const chunk_attn_desc* desc, const void* q, const void* k, const void* v, void* o, float* lse,
                   void* workspace, size_t workspace_bytes, void* stream_v) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!q || !k || !v || !o || !lse || !workspace) return CHUNK_ATTN_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0) return CHUNK_ATTN_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || (reinterpret_cast<uintptr_t>(lse) & 3) != 0)
    return CHUNK_ATTN_INVALID_ARG;  // the kernels move rows in 16-byte pieces
  FwdLayout L;
  layout_fwd(desc, L, true);
  if (workspace_bytes < L.total) {  // too small for partial results: nothing is cut
    L = FwdLayout{};
    layout_fwd(desc, L, true, false);
  }
  if (workspace_bytes < L.total) return CHUNK_ATTN_WORKSPACE_TOO_SMALL;
  if (L.blocks > 0x7fffffff) return CHUNK_ATTN_UNSUPPORTED;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  char* ws = static_cast<char*>(workspace);
  const bool items_inline = fwd_inline(L, desc->head_dim);
  hipError_t e;
  if (!items_inline) {
    std::vector<char> blob(L.blob_bytes, 0);
    std::memcpy(blob.data(), L.items.data(), L.items.size() * sizeof(FwdItem));
    std::memcpy(blob.data() + L.wholes_off, L.cut.data(), L.cut.size() * sizeof(FwdItem));
    if ((e = upload_schedule(ws, blob, stream)) != hipSuccess) return hip_fail(e, "schedule upload");
  }
  const FwdParams p = fwd_params(desc, L, ws, items_inline, q, k, v, o, lse);
  ProfileEvents pe = profile_events();
  profile_events() = ProfileEvents{};
  if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return hip_fail(e, "event record");
  e = launch_fwd(p, desc->head_dim, fwd_kind(L), fwd_lists(L), stream);
  if (e != hipSuccess) return hip_fail(e, "forward launch");
  if (pe.stop && (e = hipEventRecord(pe.stop, stream)) != hipSuccess) return hip_fail(e, "event record");
  return CHUNK_ATTN_OK;
}

int chunk_attn_fwd_static(const chunk_attn_desc* desc, const void* q, const void* k, const void* v, void* o, float* lse,
                          void* stream_v) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!q || !k || !v || !o || !lse) return CHUNK_ATTN_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || (reinterpret_cast<uintptr_t>(lse) & 3) != 0)
    return CHUNK_ATTN_INVALID_ARG;
  FwdLayout L;
  layout_fwd(desc, L, false);
  if (desc->num_segments > kStaticMaxSegments || L.total > kStaticScratchBytes || L.blocks > 0x7fffffff)
    return CHUNK_ATTN_TOO_LARGE;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  char* ws = nullptr;
  hipError_t e = static_scratch(&ws);
  if (e != hipSuccess) return hip_fail(e, "address of the static scratch buffer");
  const bool items_inline = fwd_inline(L, desc->head_dim);
  if (items_inline) fill_fwd_lists(desc, L);
  const FwdParams p = fwd_params(desc, L, ws, items_inline, q, k, v, o, lse);
  FwdLists lists = fwd_lists(L);
  if (!items_inline) {
    lists.num_wholes = L.split.target > 0 ? (int)L.n_wholes : 0;  // (with those that were not cut among them)
    StaticSegs segs;
    for (int t = 0; t < desc->num_segments; ++t) segs.seg[t] = desc->segments[t];
    hipLaunchKernelGGL(plan_fwd_static_kernel, dim3(1), dim3(256), 0, stream, segs, desc->num_segments, L.tile_rows,
                       reinterpret_cast<FwdItem*>(ws + L.wholes_off), (int)L.n_wholes, reinterpret_cast<FwdItem*>(ws),
                       L.split.target, reinterpret_cast<int32_t*>(ws + L.queues_off));
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "schedule kernel launch");
  }
  e = launch_fwd(p, desc->head_dim, fwd_kind(L), lists, stream);
  if (e != hipSuccess) return hip_fail(e, "forward launch");
  return CHUNK_ATTN_OK;
}

namespace {
int bwd_any(const chunk_attn_desc* desc, const void* q, const void* k, const void* v, const void* o, const void* d_o,
            const float* lse, void* dq, void* dk, void* dv, bool dkv_f32, int accumulate_dkv, void* workspace,
            size_t workspace_bytes, void* stream_v) {
  const int rc = validate(desc);
  if (rc != CHUNK_ATTN_OK) return rc;
  if (!q || !k || !v || !o || !d_o || !lse || !dq || !dk || !dv || !workspace) return CHUNK_ATTN_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)) != 0) return CHUNK_ATTN_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(d_o) || !aligned16(dq) || !aligned16(dk) ||
      !aligned16(dv) || (reinterpret_cast<uintptr_t>(lse) & 3) != 0)
    return CHUNK_ATTN_INVALID_ARG;  // the kernels move rows in 16-byte pieces
  const chunk_attn_desc w = widened(desc);
  BwdPlan P;
  auto needed = [&]() { return is_narrow(desc) ? narrow_bwd_layout(desc, P.total).total : P.total; };
  // Gradients may take the place of O and LSE, which the other kernels read before they write any; the small chunks' kernel reads both all along.
  const size_t q_bytes = (size_t)desc->total_q * desc->num_q_heads * desc->head_dim * 2, lse_bytes = (size_t)desc->total_q * desc->num_q_heads * 4;
  const size_t kv_bytes = (size_t)desc->total_kv * desc->num_kv_heads * desc->head_dim * (dkv_f32 ? 4 : 2);
  auto in_place_of = [&](const void* x, size_t bytes) {
    return overlap(x, bytes, dq, q_bytes) || overlap(x, bytes, dk, kv_bytes) || overlap(x, bytes, dv, kv_bytes);
  };
  const bool in_place = in_place_of(o, q_bytes) || in_place_of(lse, lse_bytes);
  bwd_layout(&w, P, true, kCutFine, bwd_mode() == 0 && !in_place ? desc->head_dim : 0);
  if (workspace_bytes < needed()) bwd_layout(&w, P, true, kCutInPlace);  // too small for all partial results: fewer pieces, or
  if (workspace_bytes < needed()) bwd_layout(&w, P, true, kCutNone);     // none
  if (workspace_bytes < needed()) return CHUNK_ATTN_WORKSPACE_TOO_SMALL;
  if (is_narrow(desc) && P.fused) {  // the one-pass backward: run as head_dim 128 on zero-padded copies
    const NarrowBwdLayout N = narrow_bwd_layout(desc, P.total);
    hipStream_t st = static_cast<hipStream_t>(stream_v);
    char* base = static_cast<char*>(workspace);
    const int64_t qr = (int64_t)desc->total_q * desc->num_q_heads, kr = (int64_t)desc->total_kv * desc->num_kv_heads;
    const size_t ge = dkv_f32 ? 4 : 2;
    hipError_t pe;
    if ((pe = pad_rows(q, base + N.q_off, qr, 2, st)) != hipSuccess || (pe = pad_rows(k, base + N.k_off, kr, 2, st)) != hipSuccess ||
        (pe = pad_rows(v, base + N.v_off, kr, 2, st)) != hipSuccess || (pe = pad_rows(o, base + N.o_off, qr, 2, st)) != hipSuccess ||
        (pe = pad_rows(d_o, base + N.do_off, qr, 2, st)) != hipSuccess)
      return hip_fail(pe, "padding launch");
    // accumulating calls add to what dk / dv hold and leave the rows outside every key range as they are
    if (accumulate_dkv && ((pe = pad_rows(dk, base + N.dk_off, kr, ge, st)) != hipSuccess ||
                           (pe = pad_rows(dv, base + N.dv_off, kr, ge, st)) != hipSuccess))
      return hip_fail(pe, "padding launch");
    const int r = bwd_any(&w, base + N.q_off, base + N.k_off, base + N.v_off, base + N.o_off, base + N.do_off, lse,
                          base + N.dq_off, base + N.dk_off, base + N.dv_off, dkv_f32, accumulate_dkv, base + N.inner_off,
                          workspace_bytes - N.inner_off, stream_v);
    if (r != CHUNK_ATTN_OK) return r;
    if ((pe = unpad_rows(base + N.dq_off, dq, qr, 2, st)) != hipSuccess || (pe = unpad_rows(base + N.dk_off, dk, kr, ge, st)) != hipSuccess ||
        (pe = unpad_rows(base + N.dv_off, dv, kr, ge, st)) != hipSuccess)
      return hip_fail(pe, "unpadding launch");
    return CHUNK_ATTN_OK;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  BwdArgs a;
  a.q = static_cast<const __bf16*>(q);
  a.k = static_cast<const __bf16*>(k);
  a.v = static_cast<const __bf16*>(v);
  a.o = static_cast<const __bf16*>(o);
  a.d_o = static_cast<const __bf16*>(d_o);
  a.lse = lse;
  a.dq = static_cast<__bf16*>(dq);
  a.dk = static_cast<__bf16*>(dk);
  a.dv = static_cast<__bf16*>(dv);
  a.accumulate = accumulate_dkv != 0;
  a.dkv_f32 = dkv_f32;
  a.workspace = static_cast<char*>(workspace);
  hipError_t e = hipSuccess;
  if (P.share_waves > 0) return (e = launch_bwd_share(desc, a, P.share_waves, stream)) == hipSuccess ? CHUNK_ATTN_OK : hip_fail(e, "backward launch");
  const std::vector<char> blob = bwd_blob(P);
  if (blob.size() > kInlineBlob && (e = g_ring.upload(a.workspace, blob.data(), blob.size(), stream)) != hipSuccess)
    return hip_fail(e, "schedule upload");
  e = launch_bwd(desc, a, P, blob, stream);  // (its pre-pass brings a smaller one along)
  if (e != hipSuccess) return hip_fail(e, "backward launch");
  return CHUNK_ATTN_OK;
}
}  // namespace

int chunk_attn_bwd(const chunk_attn_desc* desc, const void* q, const void* k, const void* v, const void* o,
                   const void* d_o, const float* lse, void* dq, void* dk, void* dv, int accumulate_dkv,
                   void* workspace, size_t workspace_bytes, void* stream_v) {
  return bwd_any(desc, q, k, v, o, d_o, lse, dq, dk, dv, false, accumulate_dkv, workspace, workspace_bytes, stream_v);
}

int chunk_attn_bwd_f32kv(const chunk_attn_desc* desc, const void* q, const void* k, const void* v, const void* o,
                         const void* d_o, const float* lse, void* dq, float* dk, float* dv, int accumulate_dkv,
                         void* workspace, size_t workspace_bytes, void* stream_v) {
  return bwd_any(desc, q, k, v, o, d_o, lse, dq, dk, dv, true, accumulate_dkv, workspace, workspace_bytes, stream_v);
}

}  // extern "C"

// Fused in-place cross-entropy (include/fused_ce.h; paper section 4, "Fused In-Place Cross-Entropy").
//
// HBM-bound by construction: one workgroup of 512 threads owns one row of logits at a time, loads it once (16 bytes per
// lane and load, consecutive lanes consecutive chunks: fully coalesced), reduces the maximum and the sum of
// exponentials across the workgroup, and stores the gradient over the logits.  Algorithmic traffic: 4 bytes per logit.
// The exponential of an element is evaluated twice (for the sum and for the gradient) rather than kept: the vector work of
// a row is several times shorter than the time HBM needs to deliver it.  Workgroups walk the rows with a grid stride.
//
// Two kernels.  fused_ce_kernel: rows of up to 65536 logits, and of up to 131072 where there are fewer than two per compute unit (or very many, kManyBytes); they stay in at most 128
// registers per lane, maximum and sum are two passes over them.  With 8, 16 and 32 chunks to a lane it takes 70, 118 and 215 registers: two or more workgroups on a compute unit hide each
// other's vector work, but for rows of more than 65536 logits, whose workgroups have the compute unit to themselves.
// fused_ce_long_kernel: longer rows take more registers, the longest LDS, too, so that one workgroup has the compute unit.  It takes the sum while the row
// arrives, against the running maximum of the thread's own chunks (moved once per group of chunks), merges the threads' (maximum, sum) pairs once per row, and as it
// stores a chunk's gradient it loads that chunk of its next row into the same registers: reads stay in flight through the vector work of the gradients, a third of
// a row's time.  us, a row after the other -> so -> and past the caches: 4096 rows of 151936 logits 534 (4.7 TB/s) -> 516 -> 498 (5.0; a copy of
// the same bytes by the runtime: 5.5), 1024 of 262144 276 -> 245 -> 221, 4096 of 128000 454 -> 431 -> 414 (before: fused_ce_kernel), 700 of 140000 86 -> 78.
// Where the long kernel is the slower one: 16384 rows of 8000 119 -> 148; 64 of 128256 19.5 -> 21.4, 300 of 100000 37.7 -> 38.5 (512 of 70000 35.3 -> 31.4).
#include <hip/hip_runtime.h>

#include "../../include/fused_ce.h"
#include "device_common.hpp"
#include "kernels.hpp"
#include "tiles.hpp"

namespace chunk_attn {
namespace {

constexpr int kThreads = 512;
// Logits of more bytes than the last-level cache (256 MiB) holds stream past the caches; what fits is kept for those who wrote it and who read it next.
// Rows of whole cache lines (kStreamAll), us, kept / streamed: fused_ce_long_kernel, 512 rows of 262144 (268 MB) 104 / 113, 1024 of 131072 (268) 103 / 111, 900 of
// 151936 (273) 128 / 123, 4096 of 151936 (1245) 516 / 498; fused_ce_kernel, which has more rows in flight, a little later: 4400 of 32000 (282) 106.2 / 107.2, 6000 of
// 24000 (288) 107.3 / 103.7, 16384 of 16000 (524) 200 / 182, 65536 of 4096 (537) 387 / 324 (stores only: 386).
// Where rows begin inside a line, so does every wave's share of a chunk, and the two waves that share a line may each fetch it from memory.  With rows of up to 16384
// logits that costs less than streaming gains (kept / all: 32768 of 8008 252 / 225, 16384 of 16008 200 / 189); with up to 32768 all is slower and stores only are, too
// (kept / stores / all: 16384 of 32760 422 / 439 / 444, 8192 of 32008 210 / 214 / 210); longer ones stream their stores, from a larger size on: 1100 of 131064 (288)
// 131 / 135 / -, 1024 of 151944 (311) 134 / 138 / -, 1100 of 151944 (334) 163 / 160 / -, 1024 of 262136 (537) 261 / 241 / 245, 4096 of 65528 (537) 225 / 207 / 217.
constexpr int64_t kStreamBytes = (int64_t)256 << 20, kStreamBytesShort = (int64_t)272 << 20, kStreamStoresBytes = (int64_t)320 << 20;
constexpr int kShortRow = 16384;
// (Figures of the operator repeated on its own output.  Where the logits are written first, kept rows leave the cache full of gradients, which costs the next writer, too: refill and operator, kept /
// streamed, 1128 rows of 128256 (289) 247 / 230, 952 of 151936 (289) 243 / 220, and 900 rows or so of 151936 that are not whole lines, 126 us before the next row's loads and 131 with
// them when repeated, take 242 and 239.)
// Above 2 GiB rows of 65544 to 131072 logits lose what they gain below, by measurement: with a compute unit to itself a workgroup of either kernel has nobody to hide its vector work, and why the long
// kernel's loads ahead help less there was not found (a row to each workgroup, handed out in order: 16384 of 131064 1816 -> 1670, of 131072 1663 -> 1640, but with the logits written first only
// 3501 -> 3463 and 3647 -> 3657 of refill and operator).  Whole lines, fused_ce_kernel / long kernel kept / streamed: 16384
// rows of 131072 (4.3 GB) 1686 / 1657 / 1740, 12000 1249 / 1217 / 1268, 8192 (2 GiB) 868 / 837 / 849; others, fused_ce_kernel / long kernel, stores streamed:
// 16384 of 131064 1717 / 1772, 16384 of 100000 1337 / 1338.  Longer rows and shorter ones gain there, too: 14000 of 151936 1727 -> 1660, 32768 of 65536 1653 -> 1602.
constexpr int64_t kManyBytes = (int64_t)2 << 30;
bool whole_lines(const void* logits, int64_t row_stride) { return ((uintptr_t)logits & 127) == 0 && row_stride % 64 == 0; }
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// What passes the caches by.
enum Stream { kKeep, kStreamStores, kStreamAll };
template <Stream STREAM>
__device__ __forceinline__ bf16x8 load_chunk_at(const void* from) {
  const bf16x8* const p = reinterpret_cast<const bf16x8*>(from);
  return STREAM == kStreamAll ? __builtin_nontemporal_load(p) : *p;
}
template <Stream STREAM>
__device__ __forceinline__ void store_chunk_at(void* to, bf16x8 x) {
  bf16x8* const p = reinterpret_cast<bf16x8*>(to);
  if constexpr (STREAM != kKeep) __builtin_nontemporal_store(x, p);
  else *p = x;
}

// NCH: 16-byte chunks per thread (a row has at most 512 * 8 * NCH logits; 32 chunks = 128 registers is what fits)
template <int NCH, Stream STREAM>
__global__ __launch_bounds__(kThreads) void fused_ce_kernel(__bf16* __restrict__ logits, const int32_t* __restrict__ targets,
                                                            float* __restrict__ loss, int64_t rows, int vocab,
                                                            int64_t row_stride, float grad_scale) {
  __shared__ float red[2][kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_chunks = vocab / 8;
  for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
    __bf16* const z = logits + row * row_stride;
    const int y = targets[row];
    const bool ignored = y < 0 || y >= vocab;
    const float zy = ignored ? 0.f : (float)z[y];  // read before the row is overwritten (every thread: one cached load)
    bf16x8 v[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = c * kThreads + tid;
      if (ch < n_chunks) v[c] = load_chunk_at<STREAM>(z + (int64_t)ch * 8);
    }
    // Between the three passes the row is kept as it was loaded (packed bf16): the opaque statements stop the compiler
    // from keeping a widened fp32 copy of the whole row alive, which would not fit the register file.
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if (c * kThreads + tid < n_chunks) {
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, (float)v[c][e]);
      }
    mx = wave_max(mx);
    if (lane == 0) red[0][wave] = mx;
    __syncthreads();
    mx = red[0][0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) mx = fmaxf(mx, red[0][w]);
    const float m2 = mx * kLog2e;
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(v[c]));
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      if (c * kThreads + tid < n_chunks) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += __builtin_amdgcn_exp2f((float)v[c][e] * kLog2e - m2);
      }
    sum = wave_sum(sum);
    if (lane == 0) red[1][wave] = sum;
    __syncthreads();
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) sum += red[1][w];
    const float lse2 = m2 + __builtin_amdgcn_logf(sum);  // log2 of the sum of exponentials
    if (tid == 0) loss[row] = ignored ? 0.f : lse2 * kLn2 - zy;
    const float scale = ignored ? 0.f : grad_scale;
#pragma unroll
    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(v[c]));
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = c * kThreads + tid;
      if (ch < n_chunks) {
        const int d = y - ch * 8;  // position of the target inside this chunk, if it is there
        bf16x8 g;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float pe = __builtin_amdgcn_exp2f((float)v[c][e] * kLog2e - lse2);
          if (d == e) pe -= 1.0f;
          g[e] = (__bf16)(pe * scale);
        }
        store_chunk_at<STREAM>(z + (int64_t)ch * 8, g);
      }
    }
    __syncthreads();  // red[] is reused by the next row
  }
}

// Longer rows, up to 262144 logits.  FULL: chunks that every lane has.  NCH: 16-byte chunks per thread kept in registers, NL: further ones kept in LDS (a row has at most
// 512 * 8 * (NCH + NL) logits).  A compute unit has 512 KB of registers and 160 KB of LDS and a row of 262144 logits takes
// 512 KB, so the longest rows need both: chunks past the NCH-th are copied global -> LDS (wave w's chunk c in 1 KB at
// c * 8 + w; each lane reads back what its own wave copied, so no barrier is needed).
template <int NCH, int NL, int FULL, Stream STREAM>
__global__ __launch_bounds__(kThreads) void fused_ce_long_kernel(__bf16* __restrict__ logits, const int32_t* __restrict__ targets,
                                                            float* __restrict__ loss, int64_t rows, int vocab,
                                                            int64_t row_stride, float grad_scale) {
  constexpr int NW = kThreads / 64;
  constexpr int GRP = NCH % 4 == 0 && NL % 4 == 0 ? 4 : 2;  // chunks per update of the running maximum
  static_assert(NCH % GRP == 0 && NL % GRP == 0, "whole groups");
  extern __shared__ __attribute__((aligned(1024))) char tail_smem[];  // [NL][NW][64] chunks
  __shared__ float red_m[2][NW], red_s[2][NW];  // two sets: the next row's partial results do not wait for this row's readers
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_chunks = vocab / 8;
  lds_bf16* const tail = (lds_bf16*)tail_smem;
  bf16x8 ninf8;
#pragma unroll
  for (int e = 0; e < 8; ++e) ninf8[e] = (__bf16)-INFINITY;
  // The first FULL chunks every lane has.  Of the others it may lack some: of a chunk that only some lanes have the others load the row's last 16 bytes, and what a lane
  // lacks counts as -inf and is not stored.  Loads are only behind wave-uniform branches: behind one that masks lanes the compiler waits for all of them at once.
  const unsigned lane_off = (unsigned)tid * 16u;
  const int last = (n_chunks - 1) / kThreads;  // the chunk that some lanes may lack; all lanes lack the ones behind it
  const unsigned last_off = (unsigned)min(tid, n_chunks - 1 - last * kThreads) * 16u;
  auto load_chunk = [&](const char* zb, int c) __attribute__((always_inline)) {
    unsigned off = lane_off, off_l = last_off;
    asm volatile("" : "+v"(off), "+v"(off_l));  // (the choice is made here, not kept in a register for each chunk)
    if (c >= FULL) off = c < last ? off : off_l;
    return load_chunk_at<STREAM>(zb + c * kThreads * 16 + off);
  };
  auto has_chunk = [&](int c) __attribute__((always_inline)) {
    int t = tid;
    asm volatile("" : "+v"(t));
    return c < FULL || t < n_chunks - c * kThreads;
  };
  auto copy_chunk = [&](const char* zb, int c) __attribute__((always_inline)) {  // (to LDS; lanes past the row copy its last chunk, ignored below)
    if ((NCH + c) * kThreads + wave * 64 < n_chunks) {
      const int ch = min((NCH + c) * kThreads + tid, n_chunks - 1);
      dma16(zb + (int64_t)ch * 16, tail + (c * NW + wave) * 512);
    }
  };
  int64_t row = blockIdx.x;
  char* zb = reinterpret_cast<char*>(logits + row * row_stride);
  int y = targets[row];
  auto target_logit = [&](const char* from, int at) __attribute__((always_inline)) {  // (every thread: one cached load; not used where the row is ignored)
    return reinterpret_cast<const unsigned short*>(from)[at < 0 || at >= vocab ? 0 : at];
  };
  unsigned zy = target_logit(zb, y);  // its bits
  bf16x8 v[NCH];
#pragma unroll 1
  for (int c = 0; c < NL; ++c) copy_chunk(zb, c);
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (c >= FULL) v[c] = ninf8;
    if (c < FULL || c <= last) v[c] = load_chunk(zb, c);
  }
  for (int set = 0;; set ^= 1) {
    const bool ignored = y < 0 || y >= vocab;
    // Maximum (mx, in log2 units: the rounded product is what every exponent is taken against, so that it drops out of
    // the result) and sum of the thread's chunks, group by group.  A thread whose chunks so far are all -inf (or absent) keeps
    // the maximum at -inf and counts against 0 instead, where they contribute exp2(-inf) = 0.
    float mx = -INFINITY, sum = 0.f;
    auto count_group = [&](const bf16x8 (&g)[GRP]) __attribute__((always_inline)) {
      float gm = -INFINITY;
#pragma unroll
      for (int c = 0; c < GRP; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) gm = fmaxf(gm, (float)g[c][e]);
      const float m2 = fmaxf(mx, __fmul_rn(gm, kLog2e));
      const float ref = m2 == -INFINITY ? 0.f : m2;
      sum *= __builtin_amdgcn_exp2f(mx - ref);  // (0 while mx is -inf: there is no sum yet)
      mx = m2;
#pragma unroll
      for (int c = 0; c < GRP; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += __builtin_amdgcn_exp2f((float)g[c][e] * kLog2e - ref);
    };
#pragma unroll
    for (int c0 = 0; c0 < NCH; c0 += GRP) {
      if (c0 >= FULL && c0 * kThreads >= n_chunks) continue;
      bf16x8 g[GRP];
#pragma unroll
      for (int c = 0; c < GRP; ++c) g[c] = has_chunk(c0 + c) ? v[c0 + c] : ninf8;
      count_group(g);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NL > 0) {
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed
#pragma unroll 3
      for (int c0 = 0; c0 < NL; c0 += GRP) {
        if ((NCH + c0) * kThreads >= n_chunks) break;
        bf16x8 g[GRP];
#pragma unroll
        for (int c = 0; c < GRP; ++c) {
          g[c] = lds_load8(tail + ((c0 + c) * NW + wave) * 512 + lane * 8);
          if (!has_chunk(NCH + c0 + c)) g[c] = ninf8;
        }
        count_group(g);
      }
    }
    // merge: the wave's 64 pairs, then the workgroup's 8.  A share whose maximum is -inf has the sum 0, or NaN if a NaN was
    // among its logits (the maximum passes over it), which the row's loss has to show: it is taken as it is.
    const float wm = wave_max(mx);
    sum = mx == -INFINITY ? sum : sum * __builtin_amdgcn_exp2f(mx - wm);
    sum = wave_sum(sum);
    if (lane == 0) {
      red_m[set][wave] = wm;
      red_s[set][wave] = sum;
    }
    asm volatile("" : "+v"(zy));  // (it has arrived before any wave overwrites the row)
    __syncthreads();
    float bm = red_m[set][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) bm = fmaxf(bm, red_m[set][w]);
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w)
      sum += red_m[set][w] == -INFINITY ? red_s[set][w] : red_s[set][w] * __builtin_amdgcn_exp2f(red_m[set][w] - bm);
    const float lse2 = bm + __builtin_amdgcn_logf(sum);  // log2 of the sum of exponentials
    if (tid == 0) loss[row] = ignored ? 0.f : lse2 * kLn2 - __builtin_bit_cast(float, zy << 16);
    const float scale = ignored ? 0.f : grad_scale;
    const int y_lane = y - tid * 8;  // (of this row)
    auto store_chunk = [&](bf16x8 x, int c) __attribute__((always_inline)) {
      const int d = y_lane - c * (kThreads * 8);  // position of the target inside this chunk, if it is there
      bf16x8 g;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float pe = __builtin_amdgcn_exp2f((float)x[e] * kLog2e - lse2);
        if (d == e) pe -= 1.0f;
        g[e] = (__bf16)(pe * scale);
      }
      store_chunk_at<STREAM>(zb + c * kThreads * 16 + lane_off, g);
    };
    // As a chunk is stored its place takes that chunk of the workgroup's next row.
    const int64_t next = row + gridDim.x;
    const bool more = next < rows;
    char* const zn = reinterpret_cast<char*>(logits + next * row_stride);
    if (more) {
      y = targets[next];
      zy = target_logit(zn, y);
    }
    // The row is kept as it was loaded (packed bf16): the opaque statements stop the compiler from keeping a widened
    // fp32 copy of the whole row alive, which would not fit the register file.
#pragma unroll
    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(v[c]));
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (has_chunk(c)) store_chunk(v[c], c);
      if (more && (c < FULL || c <= last)) v[c] = load_chunk(zn, c);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 2
    for (int c = 0; c < NL; ++c) {
      if (has_chunk(NCH + c)) store_chunk(lds_load8(tail + (c * NW + wave) * 512 + lane * 8), NCH + c);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the chunk has been read: a copy may take its place)
      if (more) copy_chunk(zn, c);
    }
    if (!more) break;
    row = next;
    zb = zn;
  }
}

template <int NCH, int NL, int FULL, Stream STREAM>
hipError_t launch_as(void* logits, const int32_t* targets, float* loss, int64_t rows, int vocab, int64_t row_stride,
                     float grad_scale, hipStream_t stream) {
  if constexpr (FULL == 0) {
    // two workgroups per compute unit where the registers allow it, rows dealt round robin (at 32 chunks, one to a compute unit, 256 and 512 workgroups take the same time)
    const dim3 grid((unsigned)(rows < 512 ? rows : 512));
    hipLaunchKernelGGL((fused_ce_kernel<NCH, STREAM>), grid, dim3(kThreads), 0, stream, (__bf16*)logits, targets, loss, rows, vocab,
                       row_stride, grad_scale);
  } else {
    constexpr size_t smem = (size_t)NL * kThreads * 16;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&fused_ce_long_kernel<NCH, NL, FULL, STREAM>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (attr != hipSuccess) return attr;
    const dim3 grid((unsigned)persistent_grid(rows));  // one per compute unit is what the registers allow: each goes through its share of the rows
    hipLaunchKernelGGL((fused_ce_long_kernel<NCH, NL, FULL, STREAM>), grid, dim3(kThreads), smem, stream, (__bf16*)logits, targets, loss, rows,
                       vocab, row_stride, grad_scale);
  }
  return hipGetLastError();
}
template <int NCH, int NL = 0, int FULL = 0>
hipError_t launch(void* logits, const int32_t* targets, float* loss, int64_t rows, int vocab, int64_t row_stride,
                  float grad_scale, hipStream_t stream) {
  auto as = [&](auto stream_c) {
    return launch_as<NCH, NL, FULL, decltype(stream_c)::value>(logits, targets, loss, rows, vocab, row_stride, grad_scale, stream);
  };
  const std::integral_constant<Stream, kKeep> keep;
  if constexpr (FULL == 0 && NCH == 32) return as(keep);  // (fewer than 512 rows, or more than kManyBytes)
  else {
    const int64_t bytes = rows * (int64_t)vocab * 2;
    if (NCH == 32 && bytes > kManyBytes) return as(keep);
    if (whole_lines(logits, row_stride) || (FULL == 0 && vocab <= kShortRow))
      return bytes > (FULL == 0 ? kStreamBytesShort : kStreamBytes) ? as(std::integral_constant<Stream, kStreamAll>{}) : as(keep);
    if constexpr (NCH > 8)
      if (bytes > kStreamStoresBytes) return as(std::integral_constant<Stream, kStreamStores>{});
    return as(keep);
  }
}

}  // namespace
}  // namespace chunk_attn

extern "C" int fused_ce_inplace(void* logits, const int32_t* targets, float* loss, int64_t rows, int32_t vocab,
                                int64_t row_stride, float grad_scale, void* hip_stream) {
  using namespace chunk_attn;
  if (rows < 0 || vocab < 8 || row_stride < vocab) return CHUNK_ATTN_INVALID_ARG;
  if (vocab % 8 != 0 || row_stride % 8 != 0 || vocab > FUSED_CE_MAX_VOCAB) return CHUNK_ATTN_UNSUPPORTED;
  if (rows == 0) return CHUNK_ATTN_OK;  // nothing to do (the pointers of empty buffers may be null)
  if (!logits || !targets || !loss || ((uintptr_t)logits & 15) != 0) return CHUNK_ATTN_INVALID_ARG;
  hipStream_t s = (hipStream_t)hip_stream;
  const int per_thread = (vocab / 8 + kThreads - 1) / kThreads;
  hipError_t e;
  if (per_thread <= 8) e = launch<8>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else if (per_thread <= 16) e = launch<16>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else if (per_thread <= 32 && (rows < 2 * kCus || (rows * (int64_t)vocab * 2 > kManyBytes && !whole_lines(logits, row_stride)))) e = launch<32>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else if (per_thread <= 32) e = launch<32, 0, 16>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else if (per_thread <= 40) e = launch<40, 0, 32>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else e = launch<46, 18, 40>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  static_assert(FUSED_CE_MAX_VOCAB <= kThreads * 8 * (46 + 18), "the longest row fits registers and LDS");
  return e == hipSuccess ? CHUNK_ATTN_OK : CHUNK_ATTN_HIP_ERROR;
}

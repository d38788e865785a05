// Fused in-place cross-entropy (include/fused_ce.h; paper section 4, "Fused In-Place Cross-Entropy").
//
// HBM-bound by construction: one workgroup of 512 threads owns one row of logits at a time, loads it once (16 bytes per
// lane and load, consecutive lanes consecutive chunks: fully coalesced), reduces the maximum and the sum of
// exponentials across the workgroup, and stores the gradient over the logits.  Algorithmic traffic: 4 bytes per logit.
// The exponential of an element is evaluated twice (for the sum and for the gradient) rather than kept: the vector work of
// a row is several times shorter than the time HBM needs to deliver it.  Workgroups walk the rows with a grid stride.
//
// Two kernels.  Rows of up to 131072 logits (fused_ce_kernel) stay in 128 registers per lane; maximum and sum are two passes
// over them.  Longer rows (fused_ce_long_kernel) take more registers and LDS; with one workgroup per compute unit nothing
// hides the vector work between the last load and the first store, so the sum is taken while the row arrives, against the
// running maximum of the thread's own chunks (moved once per group of chunks), and the threads' (maximum, sum) pairs are
// merged once per row.  Measured: 4096 rows of 151936 logits 538 us, 4.6 TB/s (a copy of the same bytes by the runtime: 5.5
// TB/s; with three passes over memory, as such rows took before: 780 us), 2048 of 200064 539 -> 391 us.  On shorter rows the
// one-pass sum is the slower one (16384 rows of 8000: 119 -> 148 us; 256 of 64000: 14.1 -> 15.0).
#include <hip/hip_runtime.h>

#include "../../include/fused_ce.h"
#include "device_common.hpp"
#include "tiles.hpp"

namespace chunk_attn {
namespace {

constexpr int kThreads = 512;
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

// NCH: 16-byte chunks per thread (a row has at most 512 * 8 * NCH logits; 32 chunks = 128 registers is what fits)
template <int NCH>
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
      if (ch < n_chunks) v[c] = *reinterpret_cast<const bf16x8*>(z + (int64_t)ch * 8);
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
        *reinterpret_cast<bf16x8*>(z + (int64_t)ch * 8) = g;
      }
    }
    __syncthreads();  // red[] is reused by the next row
  }
}

// Longer rows, up to 262144 logits.  NCH: 16-byte chunks per thread kept in registers, NL: further ones kept in LDS (a row has at most
// 512 * 8 * (NCH + NL) logits).  A compute unit has 512 KB of registers and 160 KB of LDS and a row of 262144 logits takes
// 512 KB, so the longest rows need both: chunks past the NCH-th are copied global -> LDS (wave w's chunk c in 1 KB at
// c * 8 + w; each lane reads back what its own wave copied, so no barrier is needed).
template <int NCH, int NL>
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
  int set = 0;
  for (int64_t row = blockIdx.x; row < rows; row += gridDim.x, set ^= 1) {
    __bf16* const z = logits + row * row_stride;
    const int y = targets[row];
    const bool ignored = y < 0 || y >= vocab;
    const float zy = ignored ? 0.f : (float)z[y];  // read before the row is overwritten (every thread: one cached load)
    if constexpr (NL > 0) {
#pragma unroll
      for (int c = 0; c < NL; ++c) {  // lanes past the row copy its last chunk (ignored below)
        if ((NCH + c) * kThreads + wave * 64 < n_chunks) {
          const int ch = min((NCH + c) * kThreads + tid, n_chunks - 1);
          dma16(z + (int64_t)ch * 8, tail + (c * NW + wave) * 512);
        }
      }
    }
    // (the row's last chunks are the only ones some lanes lack: they read as -inf and are not stored; everything else
    // branches on wave-uniform conditions, from a scalar base address and one 32-bit offset per lane)
    char* const zb = reinterpret_cast<char*>(z);
    const unsigned lane_off = (unsigned)tid * 16u;
    bf16x8 v[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const char* base = zb + c * kThreads * 16;
      if ((c + 1) * kThreads <= n_chunks) {
        v[c] = *reinterpret_cast<const bf16x8*>(base + lane_off);
      } else {
        v[c] = ninf8;
        if (c * kThreads + tid < n_chunks) v[c] = *reinterpret_cast<const bf16x8*>(base + lane_off);
      }
    }
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
      if (c0 * kThreads >= n_chunks) continue;
      bf16x8 g[GRP];
#pragma unroll
      for (int c = 0; c < GRP; ++c) g[c] = v[c0 + c];
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
          if ((NCH + c0 + c) * kThreads + tid >= n_chunks) g[c] = ninf8;
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
    __syncthreads();
    float bm = red_m[set][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) bm = fmaxf(bm, red_m[set][w]);
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w)
      sum += red_m[set][w] == -INFINITY ? red_s[set][w] : red_s[set][w] * __builtin_amdgcn_exp2f(red_m[set][w] - bm);
    const float lse2 = bm + __builtin_amdgcn_logf(sum);  // log2 of the sum of exponentials
    if (tid == 0) loss[row] = ignored ? 0.f : lse2 * kLn2 - zy;
    const float scale = ignored ? 0.f : grad_scale;
    auto store_chunk = [&](bf16x8 x, int c) __attribute__((always_inline)) {
      const int d = y - (c * kThreads + tid) * 8;  // position of the target inside this chunk, if it is there
      bf16x8 g;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float pe = __builtin_amdgcn_exp2f((float)x[e] * kLog2e - lse2);
        if (d == e) pe -= 1.0f;
        g[e] = (__bf16)(pe * scale);
      }
      *reinterpret_cast<bf16x8*>(zb + c * kThreads * 16 + lane_off) = g;
    };
    // The row is kept as it was loaded (packed bf16): the opaque statements stop the compiler from keeping a widened
    // fp32 copy of the whole row alive, which would not fit the register file.
#pragma unroll
    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(v[c]));
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if ((c + 1) * kThreads <= n_chunks) store_chunk(v[c], c);
      else if (c * kThreads + tid < n_chunks) store_chunk(v[c], c);
    }
    if constexpr (NL > 0) {
#pragma unroll 2
      for (int c = 0; c < NL; ++c) {
        if ((NCH + c) * kThreads + tid < n_chunks) store_chunk(lds_load8(tail + (c * NW + wave) * 512 + lane * 8), NCH + c);
      }
    }
  }
}

template <int NCH, int NL = 0>
hipError_t launch(void* logits, const int32_t* targets, float* loss, int64_t rows, int vocab, int64_t row_stride,
                  float grad_scale, hipStream_t stream) {
  // two workgroups per compute unit when the registers allow it, rows dealt round robin
  const dim3 grid((unsigned)(rows < 512 ? rows : 512));
  if constexpr (NCH <= 32) {
    hipLaunchKernelGGL((fused_ce_kernel<NCH>), grid, dim3(kThreads), 0, stream, (__bf16*)logits, targets, loss, rows, vocab,
                       row_stride, grad_scale);
  } else {
    constexpr size_t smem = (size_t)NL * kThreads * 16;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&fused_ce_long_kernel<NCH, NL>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((fused_ce_long_kernel<NCH, NL>), grid, dim3(kThreads), smem, stream, (__bf16*)logits, targets, loss, rows,
                       vocab, row_stride, grad_scale);
  }
  return hipGetLastError();
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
  else if (per_thread <= 32) e = launch<32>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else if (per_thread <= 40) e = launch<40>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  else e = launch<46, 18>(logits, targets, loss, rows, vocab, row_stride, grad_scale, s);
  static_assert(FUSED_CE_MAX_VOCAB <= kThreads * 8 * (46 + 18), "the longest row fits registers and LDS");
  return e == hipSuccess ? CHUNK_ATTN_OK : CHUNK_ATTN_HIP_ERROR;
}

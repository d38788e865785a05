// LDS tile layouts, global->LDS DMA and MFMA operand reads shared by the attention kernels (gfx950).
//
// Every MFMA operand is fetched with one 16-byte LDS read per lane (8 bf16 along the contraction index).
// Tiles are stored as rows of 16-byte chunks; the chunk position inside a row is permuted per row
// ("swizzle") so that the 16 lanes served together by a ds_read_b128 -- 16 consecutive rows, same logical
// chunk -- fall on 16 distinct bank groups.  Tiles are filled by global_load_lds (the data never passes
// through registers): lane x of a wave-wide load writes LDS bytes [16 x, 16 x + 16) past a wave-uniform
// base, so each lane simply fetches the global chunk that belongs at its LDS position.
#pragma once
#include <type_traits>

#include "device_common.hpp"

namespace chunk_attn {

// physical chunk position of logical chunk c in row `row` of a tile with CHUNKS 16-byte chunks per row
template <int CHUNKS>
__device__ __forceinline__ int swz(int row, int c) {
  if constexpr (CHUNKS == 32) {
    // 512-byte rows: every row starts on the same bank, so the chunk is rotated by the row index; 16 consecutive rows then
    // fall on 16 distinct bank groups
    return (c + row) & 31;
  } else if constexpr (CHUNKS == 16) {
    // 256-byte rows: rotate by a 4x4 bit-transposed row index; conflict-free for 16 consecutive rows
    const int f = ((row & 3) << 2) | ((row >> 2) & 3);
    return (c + f) & 15;
  } else if constexpr (CHUNKS == 12) {
    // 192-byte rows: four consecutive rows start on bank groups 0, 12, 8 and 4 (of 16); rotated by 0 .. 3 for the four
    // rows after them, and so on (a rotation past the row's end is a step of 4 groups, which keeps that set)
    const int x = c + ((row >> 2) & 3);
    return x >= 12 ? x - 12 : x;
  } else if constexpr (CHUNKS == 8) {
    // 128-byte rows: two rows share a 256-byte bank line, so the permutation changes every other row
    return c ^ ((row >> 1) & 7);
  } else {
    static_assert(CHUNKS == 4, "tiles have 4, 8, 12, 16 or 32 chunks per row");
    // 64-byte rows: four rows share a bank line
    return c ^ ((row >> 2) & 3);
  }
}
// logical chunk stored at physical position pc (inverse of swz)
template <int CHUNKS>
__device__ __forceinline__ int unswz(int row, int pc) {
  if constexpr (CHUNKS == 32) {
    return (pc - row) & 31;
  } else if constexpr (CHUNKS == 16) {
    const int f = ((row & 3) << 2) | ((row >> 2) & 3);
    return (pc - f) & 15;
  } else if constexpr (CHUNKS == 12) {
    const int x = pc - ((row >> 2) & 3);
    return x < 0 ? x + 12 : x;
  } else if constexpr (CHUNKS == 8) {
    return pc ^ ((row >> 1) & 7);
  } else {
    return pc ^ ((row >> 2) & 3);
  }
}
// element offset of (row, logical chunk c) in a swizzled tile
template <int CHUNKS>
__device__ __forceinline__ int tile_elem(int row, int c) {
  return (row * CHUNKS + swz<CHUNKS>(row, c)) * 8;
}

__device__ __forceinline__ void dma4(const void* gsrc, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gsrc,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 4, 0, 0);
}
__device__ __forceinline__ void dma16(const void* gsrc, void* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gsrc,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 16, 0, 0);
}

// Explicit LDS address-space pointers: accesses through them are always ds_* instructions, whatever the
// compiler can or cannot prove about a generic pointer.
typedef __attribute__((address_space(3))) __bf16 lds_bf16;
typedef __attribute__((address_space(3))) float lds_f32;
__device__ __forceinline__ bf16x8 lds_load8(const lds_bf16* p) {
  return *(const __attribute__((address_space(3))) bf16x8*)p;
}
__device__ __forceinline__ void lds_store8(lds_bf16* p, bf16x8 v) { *(__attribute__((address_space(3))) bf16x8*)p = v; }
__device__ __forceinline__ f32x4 lds_load4f(const lds_f32* p) {
  return *(const __attribute__((address_space(3))) f32x4*)p;
}
// LDS transpose read (ds_read_b64_tr_b16), see device_common.hpp
__device__ __forceinline__ s16x4 lds_read_tr(const lds_bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}
__device__ __forceinline__ void dma4(const void* gsrc, lds_f32* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gsrc,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 4, 0, 0);
}
__device__ __forceinline__ void dma16(const void* gsrc, lds_bf16* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gsrc,
                                   (__attribute__((address_space(3))) void*)lds_wave_base, 16, 0, 0);
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence would wait for every outstanding
// global->LDS copy, including the ones prefetching later stages.  Callers wait (s_waitcnt vmcnt) for exactly
// the copies the next stage needs before calling this; LDS reads of the finished stage have completed
// because their values were consumed.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Two waves that share a SIMD and run the same MFMA-phase / VALU-phase loop tend to fall into lockstep:
// both want the matrix pipe at the same time, then both want the vector ALU, and the two pipes never
// overlap.  Giving the waves of one SIMD different issue priorities (by the parity of their hardware
// wave slot) breaks the symmetry: the favoured wave runs its phases back to back and the other one
// fills the gaps, so matrix and vector work of different waves overlap.
__device__ __forceinline__ void stagger_wave_priority() {
  // HW_REG_HW_ID (register 4), bits [3:0] = wave slot on the SIMD
  const unsigned slot = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 4);
  if (slot & 1) __builtin_amdgcn_s_setprio(3);
  else __builtin_amdgcn_s_setprio(0);
}

// Chunk-major tile of 32 rows (rows of Q, dO, K or V: D / 8 chunks of 16 bytes each): chunk c of row r sits at slot
// c * 32 + (r ^ 4 (c & 3)).  Such a tile serves both as rows (16-byte reads: operand X[row][k]) and transposed
// (ds_read_b64_tr_b16: operand X^T[column][row]), both kinds of read bank-conflict free and their addresses one
// per-lane base plus constants.  cm_elem: element offset of (row r, chunk c).
__device__ __forceinline__ int cm_elem(int r, int c) { return (c * 32 + (r ^ ((c & 3) << 2))) * 8; }

// Row-major tile of 128-byte rows (head_dim 64) that serves both kinds of read as well: a copy instruction then fetches eight
// whole rows, where a chunk-major tile's fetches 32 bytes of each of 32 rows, four times the cache lines; a kernel with few
// copies in flight waits for that.  Chunk c of row r sits at position c ^ row_swz(r), bits 1 .. 3 of the row index reversed:
// 16 consecutive rows of one chunk, and four consecutive rows of four chunks, fall on all banks once.  Rows r + 16 share it,
// and chunk c ^ 4 is 64 bytes away (in either direction).
__device__ __forceinline__ int row_swz(int r) { return ((r >> 3) & 1) | ((r >> 1) & 2) | ((r & 2) << 1); }
__device__ __forceinline__ int row_elem(int r, int c) { return (r * 8 + (c ^ row_swz(r))) * 8; }

// Tiles of 32 rows of the small chunks' kernels: chunk c of row r sits at c ^ share_swz(r), which serves 16-byte reads of 16 consecutive rows and
// transposed reads of four rows by four chunks without conflicts (64: row_swz).  head_dim 96: rows of 128 columns in LDS, whose last four chunks
// copy the last but them and are never read.
constexpr int share_cols(int d) { return d == 96 ? 128 : d; }
template <int D>
__host__ __device__ constexpr int share_swz(int r) {
  return D == 64 ? ((r >> 3) & 1) | ((r >> 1) & 2) | ((r & 2) << 1) : ((r & 3) << 2) | ((r >> 2) & 3);
}

// LDS accesses as opaque instructions, for the software-pipelined kernels.  The compiler makes a wave wait for ALL of its
// outstanding global->LDS copies before an LDS read it cannot tell apart from their destinations (the
// transpose read in particular), which would serialise the copies of later stages with the reads of the
// current one.  Issued like this, the reads are invisible to that logic; the kernels order them themselves with
// explicit s_waitcnt lgkmcnt(n) (LDS operations of a wave complete in order).  `addr` is a byte address.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_asm_read16(unsigned addr) {
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ f32x4 lds_asm_read16f(unsigned addr) {
  f32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ s16x4 lds_asm_read_tr(unsigned addr) {
  s16x4 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ void lds_asm_write16(unsigned addr, bf16x8 v) {
  asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(v), "n"(OFF) : "memory");
}
__device__ __forceinline__ void lds_asm_write4(unsigned addr, int v) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
// A wait the compiler can see for all but the last N vector memory operations (and for all LDS operations).
template <int N>
__device__ __forceinline__ void wait_all_but() {
  static_assert(N >= 0 && N < 64);
  __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0070);
}
__device__ __forceinline__ unsigned lds_addr(const lds_bf16* p) { return (unsigned)(uintptr_t)p; }
__device__ __forceinline__ unsigned lds_addr(const lds_f32* p) { return (unsigned)(uintptr_t)p; }

// How a software-pipelined step spreads `n` pieces of vector work over its mini-steps first .. last - 1: the number done by the
// end of mini-step m (those of one mini-step are split between its two MFMAs, the first half, rounded up, after the first).
__host__ __device__ constexpr int spread(int n, int first, int last, int m) {
  return m < first ? 0 : m >= last - 1 ? n : n * (m - first + 1) / (last - first);
}
// LDS instructions issued between the read of fragment m and the start of mini-step m, where the wait for it stands: the
// reads of the fragments after it (fragments are read `ahead` mini-steps ahead).  Of a step's `nf` fragments those from
// t_first to t_last - 1 are transposed, two instructions each; the ones past the end are the next step's first.
__host__ __device__ constexpr int fragment_wait(int nf, int t_first, int t_last, int m, int ahead = 4) {
  int n = 0;
  for (int k = m + 1; k < m + ahead; ++k) n += k % nf >= t_first && k % nf < t_last ? 2 : 1;
  return n;
}
static_assert(fragment_wait(16, 0, 8, 0) == 6 && fragment_wait(16, 0, 8, 5) == 5 && fragment_wait(16, 0, 8, 12) == 3 &&
              fragment_wait(16, 0, 8, 13) == 4 && fragment_wait(24, 16, 24, 12) == 3 && fragment_wait(24, 16, 24, 15) == 6 &&
              fragment_wait(24, 16, 24, 21) == 5, "worked out by hand");

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

}  // namespace chunk_attn

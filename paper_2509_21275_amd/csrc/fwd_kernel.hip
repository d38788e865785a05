// Chunk attention forward for gfx950: O = softmax(scale Q K^T + mask) V and LSE, where the mask is the
// chunk mask of the paper's section 3.1 (each segment's queries see their own context and the causal
// part of their own slice; packed sequences see nothing of each other).
//
// A workgroup takes one forward work item -- a tile of query rows of one segment -- for the query heads of
// one group that share a key/value head, and streams that segment's visible keys/values through LDS, copied
// global->LDS without passing through registers.  Scores are computed transposed, S^T = K Q^T, so that after
// the MFMA every lane holds one query column: row maximum and row sum are a loop over the lane's own
// registers plus one exchange with the lane 32 away, and the bf16 probabilities are already laid out as the
// B operand of O^T += V^T P^T (device_common.hpp, "C-order").
//
// Four kernels:
//   fwd_kernel       online softmax with a lazily moved reference maximum, one 32-row query block per wave,
//                    tiles of 64 keys (rows, those of V read transposed, double-buffered).  Used for head_dim 64 unless its walks
//                    are long (pipe_pays).
//                    V as rows instead of a transposed image made by a launch before: four sequences of 1024, 32/8 heads, 51 -> 42 us; 1024
//                    queries on 32768 keys 447 -> 390 us, 2048 on 18432, 8/2 heads, 253 -> 219.  (With one workgroup per
//                    compute unit a tile's chain of copies, reads and products is what a step takes.  V in chunk-major
//                    tiles, whose copies touch four times the cache lines: 460 - 490 and 264; rows, but all transposed
//                    reads in one burst behind the products and the rows of a full tile clamped like the last one's:
//                    447 - 469 and 256.  168 registers, so that three workgroups share a CU: with two more, 64 sequences
//                    of 256 took 83 us instead of 74.)
//   fwd_pipe_kernel  head_dim 96 and 128, and 64 with two workgroups per CU: one wave per SIMD with 64 query rows, software
//                    pipelined over stages of 32 keys, reference maximum fixed by the first stage; a block with a row whose scores
//                    outgrow it is taken a second time, with the true maxima (as a second launch that found out which
//                    blocks to recompute this cost every call 4 us).  Where a chunk of 96 or
//                    128 has too few items for the chip their walks are cut into pieces (plan.hpp); the pieces leave
//                    float32 partial results, which fwd_merge_kernel puts together.
//   fwd_wide_kernel  head_dim 256: the same with 32 query rows per wave.
//   fwd_tall_kernel  head_dim 256, with 64 query rows per wave: chunks of more blocks than compute units, where it ends sooner (fwd_tall_pays).
//   fwd_share_kernel head_dim 64, 96 and 128, small chunks (choose_shared_heads): the waves of a workgroup divide the keys of 32 rows.
#include <cstring>
#include <type_traits>

#include "kernels.hpp"

#ifndef FWD_PIPE_DIST
#define FWD_PIPE_DIST 3  // stages the pipelined forward copies ahead of the one it computes on
#endif
#include "tiles.hpp"

namespace chunk_attn {

// The kernels read their arguments from the kernel argument segment, where a list of items may follow the parameters.
typedef const __attribute__((address_space(4))) FwdArgs* FwdArgsPtr;
__device__ __forceinline__ FwdArgsPtr fwd_args() { return (FwdArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(); }
__device__ __forceinline__ FwdParams load_params(const __attribute__((address_space(4))) FwdParams* src) {
  FwdParams p;
  __builtin_memcpy(&p, (const void*)src, sizeof(p));
  return p;
}
// Item x of the list in device memory, or of the one behind the parameters.  (Through the constant address space, so that the item
// comes in scalar registers either way: nothing writes the lists while a kernel runs.)
__device__ __forceinline__ FwdItem load_item(const FwdItem* list, const __attribute__((address_space(4))) FwdItem* inline_list, int x) {
  typedef const __attribute__((address_space(4))) FwdItem* item_ptr;
  const item_ptr items = list != nullptr ? (item_ptr)(uintptr_t)list : inline_list;
  FwdItem it;
  __builtin_memcpy(&it, (const void*)(items + x), sizeof(it));
  return it;
}

// Puts the pieces of cut walks together: O = sum_s 2^(m_s - M) O_s / l, l = sum_s 2^(m_s - M) l_s over the partial results of a
// whole item (O_s unnormalised, m_s the reference maximum, l_s the sum), M the largest m_s.  A workgroup takes one unit of 32 rows in
// the layout in which the pipelined kernel held it, each of its 4 waves a quarter of the accumulator.  Bound by the latency of
// reading the partial results (128 KB per block and piece, most of it written on another XCD); one workgroup of 8 waves per block, a unit
// each, took 10 us (203 queries on 1704 keys next to 611 short rows, 32/8 heads; now 5).
template <int D>
__global__ __launch_bounds__(256) void fwd_merge_kernel(FwdMergeArgs) {
  constexpr int NQ = D / 8 / 4;  // accumulator quarters per wave
  typedef const __attribute__((address_space(4))) FwdMergeArgs* args_ptr;
  const args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const FwdParams p = load_params(&args->p);
  const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x & 7, block = blockIdx.x >> 3;
  const int inner_n = p.num_kv_heads * p.head_splits, inner = block % inner_n;
  const FwdItem it = load_item(p.wholes, args->wholes, block / inner_n);
  if (it.part < 0) return;  // not cut
  const int kvh = inner % p.num_kv_heads, hs = inner / p.num_kv_heads;
  const int w = unit >> 1;  // wave of the pipelined kernel
  const int head = kvh * p.group + hs * p.heads_per_wg + w % p.heads_per_wg;
  const int r = (w / p.heads_per_wg) * 64 + 32 * (unit & 1) + l32;
  if (r >= it.q_rows) return;
  const int64_t step = (int64_t)inner_n * kPartFloats;
  const float* const part0 = p.parts + (int64_t)it.part * step + (int64_t)inner * kPartFloats;
  const float* const ml = part0 + kPartRowFloats + (unit * 32 + l32) * 2;
  float m = ml[0], l = 0.f;
#pragma unroll 4
  for (int s = 1; s < it.pieces; ++s) m = fmaxf(m, ml[s * step]);
  f32x4 o[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* const src = part0 + unit * 4096 + wave * (NQ * 256) + lane * 4;
#pragma unroll 4
  for (int s = 0; s < it.pieces; ++s) {
    const f32x2 v2 = *reinterpret_cast<const f32x2*>(ml + s * step);
    const float f = __builtin_amdgcn_exp2f(v2[0] - m);
    l += v2[1] * f;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + s * step + i * 256);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[i][e] += v[e] * f;
    }
  }
  const float inv = 1.0f / l;
  __bf16* op = p.o + (int64_t)(it.q_row0 + r) * p.num_q_heads * D + (int64_t)head * D + wave * (NQ * 8) + 4 * hh;
#pragma unroll
  for (int i = 0; i < NQ; ++i)
    *reinterpret_cast<bf16x4*>(op + 8 * i) = pack4(o[i][0] * inv, o[i][1] * inv, o[i][2] * inv, o[i][3] * inv);
  if (wave == 0 && hh == 0) p.lse[(int64_t)head * p.total_q + it.q_row0 + r] = (m + log2f(l)) * 0.6931471805599453f;
}

__global__ __launch_bounds__(256, 3) void fwd_kernel(FwdArgs) {
  constexpr int D = 64, WAVES = 4;
  constexpr int QB = 1;        // 32-row query blocks per wave
  constexpr int BN = 64;       // key rows per LDS tile
  constexpr int KC = D / 8;    // 16-byte chunks per K row
  constexpr int DK = D / 16;   // k-steps of S^T = K Q^T
  constexpr int DB = D / 32;   // 32-row blocks of O^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int WR = 32 * QB;  // query rows per wave
  const FwdArgsPtr args = fwd_args();
  const FwdParams p = load_params(&args->p);

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __bf16* Ks = reinterpret_cast<__bf16*>(smem);  // [2][BN][D]  rows (row_elem)
  __bf16* Vs = Ks + 2 * KT;                      // [2][BN][D]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept in a scalar register
  const int l32 = lane & 31, hh = lane >> 5;
  stagger_wave_priority();

  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = blockIdx.x % inner_n;
  const FwdItem it = load_item(p.items, args->items, blockIdx.x / inner_n);
  const int kvh = inner % p.num_kv_heads, hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int wave_row0 = (wave / p.heads_per_wg) * WR;  // first tile-local row of this wave

  const int n_wg = it.n0 + it.q_rows - 1;              // keys visible to the last valid row
  const int nt_wg = (n_wg + BN - 1) / BN;
  int nt_w = 0;
  if (wave_row0 < it.q_rows) {
    const int last = min(wave_row0 + WR, it.q_rows) - 1;
    nt_w = (it.n0 + last + BN - 1) / BN;
  }

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  // Per-lane source offsets of the global->LDS copies (elements).  A K tile is 64 rows x KC chunks; copy
  // instruction i of wave w fills LDS chunks [(WAVES i + w) 64, +64), so the lane fetches the chunk that the
  // swizzle puts there; a V tile likewise.
  constexpr int PIECES = BN * KC / 64, NK = PIECES / WAVES;
  static_assert(KT == BN * KC * 8 && PIECES % WAVES == 0, "the pieces of a tile divide evenly among the waves");
  unsigned k_src[NK];
  int k_row[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int x = (i * WAVES + wave) * 64 + lane;
    k_row[i] = x / KC;
    const int c = (x % KC) ^ row_swz(k_row[i]);
    k_src[i] = (unsigned)(k_row[i] * (int)kv_stride + c * 8);
  }
  auto dma_tile = [&](int t, int buf) {
    const __bf16* ksrc = Kg + (int64_t)(BN * t) * kv_stride;  // wave-uniform
    const int last_row = n_wg - 1 - BN * t;                   // rows past it are clamped (last tile only)
    __bf16* kdst = Ks + buf * KT;
    __bf16* vdst = Vs + buf * KT;
    auto copy = [&](int i, unsigned off) __attribute__((always_inline)) {
      dma16(ksrc + off, kdst + (i * WAVES + wave) * 512);
      dma16(Vg + (int64_t)(BN * t) * kv_stride + off, vdst + (i * WAVES + wave) * 512);
    };
    if (last_row >= BN - 1) {
#pragma unroll
      for (int i = 0; i < NK; ++i) copy(i, k_src[i]);
    } else {
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        // (the row is computed here, and not kept for the length of the loop)
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));
        const int row = ((i * WAVES + wave) * 64 + ln) / KC;
        copy(i, k_src[i] - (unsigned)((row - min(row, last_row)) * (int)kv_stride));
      }
    }
  };

  dma_tile(0, 0);

  // Q fragments: B operand of S^T = K Q^T; lane holds Q[row = 32 qb + l32][16 ks + 8 hh ..+7]
  bf16x8 qf[QB][DK];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int r = min(wave_row0 + 32 * qb + l32, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
    const __bf16* qp = p.q + (int64_t)(it.q_row0 + r) * q_stride + (int64_t)head * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) qf[qb][ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
  }

  f32x16 oacc[QB][DB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[qb][db][i] = 0.f;
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) { m_run[qb] = -INFINITY; l_run[qb] = 0.f; }
  const float c = p.scale_log2;

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // LDS operand addresses (elements).  Row l32 and row 32 + l32 share their swizzle, so the second block of
  // each tile is a constant offset away; the buffer index is a compile-time constant of the unrolled loop.
  int k_off = row_elem(l32, hh);  // (chunks 2 ks + hh are an XOR apart)
  unsigned vt_lo;  // byte address of the transposed reads (as in the pipelined kernel) in buffer 0
  {
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    vt_lo = lds_addr((lds_bf16*)Vs + row_elem(r0, cl) + 4 * (j & 1));
  }

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x2 ones;
  ones[0] = (__bf16)1.0f; ones[1] = (__bf16)1.0f;

  // One loop body for both LDS buffers: the operand addresses are toggled between the buffers with an XOR
  // (the buffers are KT elements = a power of two bytes apart), so the accumulators are
  // carried by a single loop and never pass through a conditional.
  int buf = 0;
  for (int t = 0; t < nt_wg; ++t) {
    if (t + 1 < nt_wg) dma_tile(t + 1, buf ^ 1);

    if (t < nt_w) {
      const __bf16* Kt = Ks;
      s16x4 v_lo[4][DB], v_hi[4][DB];
      auto read_vt = [&](auto ks_c) __attribute__((always_inline)) {
        static_for<0, DB>([&](auto db_c) __attribute__((always_inline)) {
          constexpr int ks = decltype(ks_c)::value, db = decltype(db_c)::value;
          // (chunks 4 .. 7 of a row: the other half of its 128 bytes)
          v_lo[ks][db] = lds_asm_read_tr<ks * (16 * D) * 2>((vt_lo ^ (db * 64)) + buf * (KT * 2));
          v_hi[ks][db] = lds_asm_read_tr<(ks * 16 + 8) * D * 2>((vt_lo ^ (db * 64 + 16)) + buf * (KT * 2));  // eight rows on
        });
      };
      // ---- S^T = K Q^T : [64 keys] x [32 QB queries]; every K fragment feeds QB products ----
      f32x16 s0[QB], s1[QB];
      auto ldk = [&](int ks, int half) { return *reinterpret_cast<const bf16x8*>(Kt + (k_off ^ (16 * ks)) + half * (32 * D)); };
      auto mma_s = [&](int ks, bf16x8 a, f32x16 (&d)[QB]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) d[qb] = mfma32(a, qf[qb][ks], ks == 0 ? zero16 : d[qb]);
      };
      // the K fragments first, the second half while the first one's products run; a quarter of the V^T fragments behind each
      // of the last four products, where the wave has nothing else to issue: they arrive while the exponentials are computed
      bf16x8 a[4][2];
#pragma unroll
      for (int x = 0; x < 4; ++x) a[x >> 1][x & 1] = ldk(x >> 1, x & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 4; x < 8; ++x) a[x >> 1][x & 1] = ldk(x >> 1, x & 1);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        mma_s(ks, a[ks][0], s0);
        mma_s(ks, a[ks][1], s1);
      }
      __builtin_amdgcn_sched_barrier(0);
      static_for<2, 4>([&](auto ks_c) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_c)::value;
        mma_s(ks, a[ks][0], s0);
        __builtin_amdgcn_sched_barrier(0);
        read_vt(std::integral_constant<int, 2 * ks - 4>{});
        __builtin_amdgcn_sched_barrier(0);
        mma_s(ks, a[ks][1], s1);
        __builtin_amdgcn_sched_barrier(0);
        read_vt(std::integral_constant<int, 2 * ks - 3>{});
        __builtin_amdgcn_sched_barrier(0);
      });
      bf16x8 pf[QB][4];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        // ---- mask: key j of the tile (j = 64 t + local) is visible to tile row r iff j < n0 + r ----
        if (BN * t + BN > it.n0 + wave_row0 + 32 * qb) {
          const int lim = it.n0 + wave_row0 + 32 * qb + l32 - BN * t;  // visible iff local key index < lim
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int j = 8 * (i >> 2) + 4 * hh + (i & 3);
            if (j >= lim) s0[qb][i] = -INFINITY;
            if (j + 32 >= lim) s1[qb][i] = -INFINITY;
          }
        }
        // ---- running max (refreshed lazily), probabilities, running sum ----
        float mx0 = fmaxf(fmaxf(s0[qb][0], s0[qb][1]), s0[qb][2]), mx1 = fmaxf(fmaxf(s1[qb][0], s1[qb][1]), s1[qb][2]);
#pragma unroll
        for (int i = 3; i < 15; i += 2) {
          mx0 = fmaxf(fmaxf(mx0, s0[qb][i]), s0[qb][i + 1]);
          mx1 = fmaxf(fmaxf(mx1, s1[qb][i]), s1[qb][i + 1]);
        }
        float mx = fmaxf(fmaxf(mx0, mx1), fmaxf(s0[qb][15], s1[qb][15]));
        mx = max_halves(mx);
        // The reference maximum only has to keep exp2 in range: it is moved when the tile maximum exceeds it
        // by more than 2^8 (first tile: from -inf), which spares the O^T rescale on almost every tile.
        if (__builtin_expect(__any((mx - m_run[qb]) * c > 8.0f), 0)) {
          const float m_new = fmaxf(m_run[qb], mx);
          const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new) * c);
          l_run[qb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[qb][db][i] *= alpha;
          m_run[qb] = m_new;
        }
        const float mc = m_run[qb] * c;
        {
          float e[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) e[i] = __builtin_amdgcn_exp2f(s0[qb][i] * c - mc);
          pf[qb][0] = pack8(e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]);
          pf[qb][1] = pack8(e[8], e[9], e[10], e[11], e[12], e[13], e[14], e[15]);
#pragma unroll
          for (int i = 0; i < 16; ++i) e[i] = __builtin_amdgcn_exp2f(s1[qb][i] * c - mc);
          pf[qb][2] = pack8(e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]);
          pf[qb][3] = pack8(e[8], e[9], e[10], e[11], e[12], e[13], e[14], e[15]);
        }
        // row sum of the rounded probabilities (the same values the PV product uses), two per instruction
        float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[qb][j], pf[qb][j], 0, 1), ones, ps0, false);
          ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[qb][j], pf[qb][j], 2, 3), ones, ps1, false);
          ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[qb][j], pf[qb][j], 4, 5), ones, ps0, false);
          ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[qb][j], pf[qb][j], 6, 7), ones, ps1, false);
        }
        l_run[qb] += ps0 + ps1;
      }
      // ---- O^T += V^T P^T : [D] x [32 QB queries], contraction over the 64 keys; every V^T fragment feeds QB products ----
      static_for<0, 4>([&](auto ks_c) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_c)::value;
        if constexpr (ks == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          asm volatile("" : "+v"(v_lo[ks][db]), "+v"(v_hi[ks][db]));  // (after the wait, in this order)
          const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v_lo[ks][db], v_hi[ks][db], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) oacc[qb][db] = mfma32(a, pf[qb][ks], oacc[qb][db]);
        }
      });
    }

    buf ^= 1;
    k_off ^= KT;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }

  // ---- epilogue: O = O^T / l, LSE = ln(l) + m scale ----
  auto oval = [&](int qb, int db, int i) { return oacc[qb][db][i]; };
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int r = wave_row0 + 32 * qb + l32;
    const float l_tot = sum_halves(l_run[qb]);
    if (r < it.q_rows) {
      const float inv = 1.0f / l_tot;
      __bf16* op = p.o + (int64_t)(it.q_row0 + r) * q_stride + (int64_t)head * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const bf16x4 v = pack4(oval(qb, db, 4 * g) * inv, oval(qb, db, 4 * g + 1) * inv, oval(qb, db, 4 * g + 2) * inv,
                                 oval(qb, db, 4 * g + 3) * inv);
          *reinterpret_cast<bf16x4*>(op + 32 * db + 8 * g + 4 * hh) = v;
        }
      if (hh == 0)
        p.lse[(int64_t)head * p.total_q + it.q_row0 + r] = (m_run[qb] * c + log2f(l_tot)) * 0.6931471805599453f;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Pipelined forward for head_dim 128, 96 and 64: one wave per SIMD (64: two), 64 query rows per wave (two 32-row "units"), keys
// streamed in stages of 32.
//
// A wave issues at most one instruction every four cycles and an MFMA holds the matrix pipe for 32, so the loop
// is laid out instruction by instruction.  In step t a wave runs
//     O^T += V(t-1)^T P^T(t-1)        S^T(t+1) = K(t+1) Q^T        (matrix pipe)
//     P^T(t) = exp2(S^T(t) c - m c) and its row sums                (vector pipe)
// as 16 (head_dim 96: 12, 64: 8) mini-steps of one LDS operand fragment and the two MFMAs it feeds (one per unit), each MFMA
// followed by its share of the vector work of 32 scores.  K and V tiles are copied global->LDS into a ring of DIST + 3 slots, stored
// chunk-major; V^T is read from the V tile itself with the LDS transpose read.  Fragments are fetched four
// mini-steps ahead with opaque LDS reads and explicit lgkmcnt waits; S^T lives in vector registers, where the
// vector work reads it directly, the Q fragments and O^T in accumulation registers (tiles.hpp).
// The reference maximum of the softmax is fixed by the first stage, so O^T is never rescaled in the loop; with a row
// whose later scores outgrow it the workgroup takes the block again, the maximum over all stages first.
// Steps whose stage needs the causal mask (the last few of the walk) or lies past the end run a second variant of
// the step that masks in the vector work.
// ------------------------------------------------------------------------------------------------
// CUT: some items are pieces.  A kernel of its own, because the few registers and instructions it takes lengthen every block of
// the other one (chunk of 256-token sequences: dQ, which has the same split, 171 -> 178 us, forward 142 -> 144).
template <int D, bool CUT>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void fwd_pipe_kernel(FwdArgs) {
  const FwdArgsPtr args = fwd_args();
  const FwdParams p = load_params(&args->p);
  const int num_blocks = args->num_blocks;
  constexpr int NW = 4;        // waves
  constexpr int BN = 32;       // key rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps of S^T = K Q^T
  constexpr int DB = D / 32;   // 32-row blocks of O^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int DIST = FWD_PIPE_DIST;  // stages copied ahead
  constexpr int NS = DIST + 3; // ring slots: stages t - 1 .. t + 1 in use, t + 2 .. t + 1 + DIST on their way
  constexpr int NF = 2 * DB + DK;      // operand fragments (mini-steps) per step: V^T, then K rows
  constexpr int AHEAD = D == 64 ? 3 : 4;  // fragments in flight
  constexpr int RING = D == 64 ? 4 : NF % 8 == 0 ? 8 : 6;  // registers of the fragment ring: a step starts where the ring does
  constexpr int NP = BN * KC / 64;     // 64-slot pieces per tile
  constexpr int PER = 2 * NP / NW;     // global->LDS copies per wave and stage
  constexpr int BOOK = D == 64 ? NF - 2 : NF - 4;  // mini-step of the bookkeeping, behind the last copy
  static_assert(2 * NP % NW == 0 && NF % RING == 0 && RING > AHEAD && 3 + 2 * (PER - 1) < BOOK, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int K_OFF = 0;               // [NS][KT]  K rows of stage n in slot n % NS (chunk-major)
  constexpr int V_OFF = K_OFF + NS * KT; // [NS][KT]  V rows
  // [NW][64][D] staging of a wave's 64 rows of Q on their way in and of O on their way out, rows of 16-byte chunks,
  // swizzled (tile_elem<KC>): global memory is then touched in whole rows (four per instruction) instead of 32 rows
  // with 32 bytes each, which costs the address unit eight times as long.  Its first word doubles as the slot through
  // which wave 0 announces the next block, between the last read of one block and the first copy of the next.
  constexpr int ST_OFF = V_OFF + NS * KT;
  constexpr int ST_ROWS = 64;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  __bf16* const stage = (__bf16*)smem + ST_OFF + wave * (ST_ROWS * D);  // this wave's staging tile (generic pointer)
  int* const next_block = (int*)((__bf16*)smem + ST_OFF);

  // The workgroup is persistent: it claims one block (work item x key/value head x head split) after the other
  // (device_common.hpp) until none is left.  The next block is claimed before the current one's last few steps: early
  // enough for the answer to arrive by the time it is needed, and not earlier (that would fix the order of the blocks
  // before it is known which workgroup is free first).
  const int xcd = xcd_of_this_wave();
  clock_log_stamp(p.clock_log, 0);
  // (As many workgroups as blocks: block b is workgroup b's, and the counters are not looked at.)
  const bool direct = num_blocks <= (int)gridDim.x;
  int blk = blockIdx.x;
  if (!direct) {
    if (wave == 0) blk = block_claim_finish(p.taken, num_blocks, xcd, block_claim_issue(p.taken, xcd));
    blk = broadcast_from_wave0(next_block, blk);
  }
  bool again = false;  // the block is taken a second time, with every row's true maximum
  int pending_claim = 0;
  while (blk >= 0) {
  wg_barrier();  // every wave has read the announcement: the staging area may be written again
  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = blk % inner_n;
  const FwdItem it = load_item(p.items, args->items, blk / inner_n);
  const int kvh = inner % p.num_kv_heads, hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int wave_row0 = (wave / p.heads_per_wg) * 64;  // the wave's units are rows wave_row0 + 32 u .. + 31 of `head`

  const int n_last = it.n0 + it.q_rows - 1;                // keys the last valid row sees ...
  const int n_wg = CUT ? min(n_last, it.keys) : n_last;  // ... of the item's range
  const int nt = (n_wg + BN - 1) / BN;       // stages

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  // the ring slots the prologue does not fill are read before anything is copied into them (V(-1) in step 0)
  {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    for (int x = tid; x < (NS - DIST - 1) * KT / 8; x += NW * 64) {
      lds_store8(L + K_OFF + (DIST + 1) * KT + x * 8, z);
      lds_store8(L + V_OFF + (DIST + 1) * KT + x * 8, z);
    }
  }

  // ---- staging: the 2 NP pieces of a stage (NP of K, then NP of V) are dealt to the waves round robin; a piece is
  // 64 consecutive slots of a chunk-major tile = two chunk columns of 32 rows.  Past the last stage the last one is
  // copied again. ----
  // byte offset of the lane's chunk from the tile's first row: full tile, last tile (rows past the last key repeat it,
  // masked; head_dim 64, short of registers, computes it when it comes to the last tile)
  const int last_row = n_wg - 1 - (nt - 1) * BN;
  auto chunk_off = [&](int i, int ln, int max_row) __attribute__((always_inline)) {
    const int x = ((i * NW + wave) % NP) * 64 + ln;
    const int off = (x >> 5) * 8, row = (x & 31) ^ (((x >> 5) & 3) << 2);
    return (unsigned)(min(row, max_row) * (int)kv_stride + off) * 2u;
  };
  unsigned v_full[PER], v_last[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v_full[i] = chunk_off(i, lane, BN);
    v_last[i] = D == 64 ? 0 : chunk_off(i, lane, last_row);
  }
  int d_t = 0, d_slot = 0;   // stage to copy next (clamped to the last one) and its slot
  int64_t d_off = 0;         // element offset of its first row
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const int piece = i * NW + wave;  // wave-uniform; the first NP are pieces of K, the others of V
    const bool of_k = NP % NW == 0 ? i < NP / NW : piece < NP;
    unsigned voff = d_t == nt - 1 ? v_last[i] : v_full[i];
    if constexpr (D == 64) {
      voff = v_full[i];
      if (__builtin_expect(d_t == nt - 1, 0)) {
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));  // (computed here and not ahead of the loop)
        voff = chunk_off(i, ln, last_row);
      }
    }
    const char* base = reinterpret_cast<const char*>((of_k ? Kg : Vg) + d_off);
    lds_bf16* dst = L + (of_k ? K_OFF + piece * 512 : V_OFF + (piece - NP) * 512) + d_slot * KT;
    dma16(base + voff, dst);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_t + 1 < nt) {
      ++d_t;
      d_off += BN * kv_stride;
    }
    d_slot = d_slot == NS - 1 ? 0 : d_slot + 1;
  };

  // per-lane operand addresses inside a tile
  int x_off[2], t_off[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) x_off[par] = cm_elem(l32, 2 * par + hh);
  {
    const int j = lane & 15, grp = (lane >> 4) & 1;
    const int cl = 2 * grp + ((j & 3) >> 1);
    const int r0 = 4 * hh + (j >> 2);
#pragma unroll
    for (int half = 0; half < 2; ++half) t_off[half] = cm_elem(r0 + 8 * half, cl) + 4 * (j & 1);
  }
  const unsigned k_ev0 = lds_addr(L + K_OFF + x_off[0]), k_od0 = lds_addr(L + K_OFF + x_off[1]);
  const unsigned t_lo0 = lds_addr(L + V_OFF + t_off[0]), t_hi0 = lds_addr(L + V_OFF + t_off[1]);
  constexpr unsigned SLOT = KT * 2;  // bytes per ring slot
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value;
    constexpr int off = (ks >> 1) * (4 * 32 * 8) * 2;
    return lds_asm_read16<off>((ks & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // prologue: the copies of stages 0 and 1 first, then the wave's rows of Q, so that both travel at the same time, then the later
  // stages, which are waited for step by step
  auto copy_stages = [&](int n) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < n; ++s) {
#pragma unroll
      for (int i = 0; i < PER; ++i) dma_piece(i);
      dma_advance();
    }
  };
  copy_stages(2);
  // the wave's 64 rows of Q (its two units) into its staging tile: slot x = 16 row + position holds the chunk that
  // belongs there; rows past the tile repeat the last one (never stored)
  {
    const __bf16* qbase = p.q + (int64_t)it.q_row0 * q_stride + (int64_t)head * D;
#pragma unroll 4
    for (int i = 0; i < ST_ROWS * KC / 64; ++i) {
      const int x = i * 64 + lane;
      const int row = x / KC, c = unswz<KC>(row, x % KC);
      const int r = min(wave_row0 + row, it.q_rows - 1);
      dma16(qbase + (int64_t)r * q_stride + c * 8, stage + i * 512);
    }
  }
  copy_stages(DIST - 1);
  // One wait the compiler can see for Q (and the copies before it): it then has no reason to put full waits for outstanding
  // loads into the loop.
  wait_all_but<(DIST - 1) * PER>();
  // Q fragments (B operands of S^T = K Q^T): lane holds Q[row = l32 of the unit][16 ks + 8 hh ..+7].  (Opaque reads, as for all that is
  // read or written while copies are on their way.)
  const unsigned stage_addr = lds_addr((lds_bf16*)stage);
  bf16x8 qf[2][DK];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) qf[u][ks] = lds_asm_read16<0>(stage_addr + 2 * tile_elem<KC>(32 * u + l32, 2 * ks + hh));
  // Once Q has been read, the staging tile's first word says whether some wave has seen a row outgrow its reference maximum:
  // one word per wave, written by any and read by its own wave only, as the others may by then write their rows of O.
  lds_asm_write4(stage_addr, 0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // (the fragments settle in their accumulation registers here: an opaque MFMA must not follow a write to one of its operands)
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      asm volatile("" : "+v"(qf[u][ks]));
      asm volatile("" : "+a"(qf[u][ks]));
    }
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 oacc[2][DB];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[u][db] = zero16;
  f32x16 x[2][2];      // S^T: [buffer][unit]
  bf16x8 f[2][2][2];   // P^T as B operands: [buffer][unit][k-step]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) f[b][u][ks][i] = (__bf16)0.0f;
  const float c = p.scale_log2;
  bf16x8 fr[RING];  // ring of operand fragments

  // S^T(0) = K(0) Q^T and the reference maximum of each row; then the first fragments of step 0 (zeros)
  float mc[2], l_run[2];
  {
    bf16x8 a[DK];
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) { a[decltype(ks_c)::value] = load_rows(k_ev0, k_od0, ks_c); });
    {
      const unsigned sT = (NS - 1) * SLOT;
      static_for<0, AHEAD>([&](auto m_c) __attribute__((always_inline)) { fr[decltype(m_c)::value] = load_t(t_lo0 + sT, t_hi0 + sT, m_c); });
    }
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(2 * AHEAD) : "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(a[ks]));  // (after the wait, in this order)
#pragma unroll
    for (int ks = 0; ks < DK; ++ks)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        f32x16& d_ = x[0][u];
        const bf16x8& b_ = qf[u][ks];
        if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a[ks]), "a"(b_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a[ks]), "a"(b_));
      }
    mfma_settle();
    asm volatile("s_nop 15" : "+v"(x[0][0]), "+v"(x[0][1]));  // the reads below come after the MFMAs have written
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int lim = it.n0 + wave_row0 + 32 * u + l32;  // stage 0: visible iff local key index < lim (>= 1)
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int j = 8 * (i >> 2) + 4 * hh + (i & 3);
        if (j < lim) mx = fmaxf(mx, x[0][u][i]);
      }
      mc[u] = max_halves(mx) * c;
      l_run[u] = 0.f;
    }
  }
  if (__builtin_expect(again, 0)) {  // the maximum over all stages: S^T as in the loop, K read from global memory
    float mx[2] = {-INFINITY, -INFINITY};
    for (int s = 0; s < nt; ++s) {
      const __bf16* kr = Kg + (int64_t)min(BN * s + l32, n_wg - 1) * kv_stride + 8 * hh;
      f32x16 d[2] = {zero16, zero16};
#pragma unroll
      for (int ks = 0; ks < DK; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kr + 16 * ks);
#pragma unroll
        for (int u = 0; u < 2; ++u) d[u] = mfma32(a, qf[u][ks], d[u]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int lim = it.n0 + wave_row0 + 32 * u + l32 - BN * s;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * hh + (i & 3) < lim) mx[u] = fmaxf(mx[u], d[u][i]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) mc[u] = max_halves(mx[u]) * c;
  }
  bool risk = false;
  const float big = __builtin_amdgcn_exp2f(p.ref_limit);

  // In program order mini-step m reads fragment m + AHEAD: the transposed fragments (0 .. 2 DB - 1 of this step, 0 .. AHEAD - 1 of the
  // next) take two instructions, the rows fragments one.
  int sV = 0;  // slot of stage t
  auto step = [&](int t, f32x16 (&cur)[2], f32x16 (&nxt)[2], bf16x8 (&f_old)[2][2], bf16x8 (&f_new)[2][2],
                  auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int sK = sV == NS - 1 ? 0 : sV + 1;   // stage t + 1
    const int sM = sV == 0 ? NS - 1 : sV - 1;   // stage t - 1
    const unsigned k_ev = k_ev0 + sK * SLOT, k_od = k_od0 + sK * SLOT;
    const unsigned t_lo = t_lo0 + sM * SLOT, t_hi = t_hi0 + sM * SLOT, n_lo = t_lo0 + sV * SLOT, n_hi = t_hi0 + sV * SLOT;
    // MASKED: element i (key 8 (i / 4) + 4 hh + i % 4 of the stage) of unit u is visible iff 8 (i / 4) + i % 4 < lim[u]
    int lim[2];
    if (MASKED) {
#pragma unroll
      for (int u = 0; u < 2; ++u) lim[u] = t < nt ? it.n0 + wave_row0 + 32 * u + l32 - BN * t - 4 * hh : -0x40000000;
    }
    unsigned pw[2][8];  // P^T(t), packed pairs
    float ps[2] = {0.f, 0.f};
    float e_hold[2];
    // vector work of score 2 dw + q of unit u (pair j = 8 u + dw), pinned to where it is written; a pair is converted
    // one mini-step after its exponentials (a transcendental result cannot be consumed by the very next instruction)
    auto finish_pair = [&](int jp) __attribute__((always_inline)) {
      bf16x2 w;
      w[0] = (__bf16)e_hold[0]; w[1] = (__bf16)e_hold[1];
      // row sums with plain adds: a dot-product instruction next to MFMAs holds the wave up (it costs about as much
      // as 14 cycles of the matrix pipe, an add 1 - 2)
      ps[jp >> 3] += e_hold[0] + e_hold[1];
      asm volatile("" : "+v"(ps[jp >> 3]));
      unsigned wu = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(wu));
      pw[jp >> 3][jp & 7] = wu;
    };
    auto vec_half = [&](auto j_c, auto q_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, q = decltype(q_c)::value;
      constexpr int u = j >> 3, i = 2 * (j & 7) + q;
      if constexpr (j > 0 && q == 0) finish_pair(j - 1);
      float tt = cur[u][i] * c - mc[u];
      if (MASKED) {
        if (8 * (i >> 2) + (i & 3) >= lim[u]) tt = -INFINITY;
      }
      e_hold[q] = __builtin_amdgcn_exp2f(tt);
      asm volatile("" : "+v"(e_hold[q]));
    };
    // the 32 scores' vector work, spread evenly over the step's 2 NF MFMAs: scores [done(k - 1), done(k)) after MFMA k
    auto vec_after = [&](auto k_c) __attribute__((always_inline)) {
      constexpr int k = decltype(k_c)::value, lo = 32 * k / (2 * NF), hi = 32 * (k + 1) / (2 * NF);
      static_for<lo, hi>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int x = decltype(x_c)::value;
        vec_half(std::integral_constant<int, x / 2>{}, std::integral_constant<int, x % 2>{});
      });
    };
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(fragment_wait(NF, 0, 2 * DB, m, AHEAD)));
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's first transposed fragments)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < 2 * DB) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm>{});
        else if constexpr (mm < NF) fr[mm % RING] = load_rows(k_ev, k_od, std::integral_constant<int, mm - 2 * DB>{});
        else fr[mm % RING] = load_t(n_lo, n_hi, std::integral_constant<int, mm - NF>{});
      }
      const bf16x8 fa = fr[m % RING];
      auto mma = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        if constexpr (m < 2 * DB) {
          constexpr int ks = m / DB, db = m % DB;
          oacc[u][db] = mfma32(fa, f_old[u][ks], oacc[u][db]);
        } else {
          constexpr int ks = m - 2 * DB;
          const bf16x8& a_ = fa;  // (named references: variables used only inside an asm statement are not captured)
          f32x16& d_ = nxt[u];
          const bf16x8& b_ = qf[u][ks];
          if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
        }
      };
      constexpr std::integral_constant<int, 0> c0{};
      constexpr std::integral_constant<int, 1> c1{};
      mma(c0);
      vec_after(std::integral_constant<int, 2 * m>{});
      __builtin_amdgcn_sched_barrier(0);
      mma(c1);
      vec_after(std::integral_constant<int, 2 * m + 1>{});
      if constexpr (m >= 3 && m < 3 + 2 * PER && ((m - 3) & 1) == 0) dma_piece((m - 3) >> 1);
      if constexpr (m == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        dma_advance();
        sV = sK;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    finish_pair(15);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      risk |= !(ps[u] < big);
      l_run[u] += ps[u];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        u32x4 v = {pw[u][4 * ks], pw[u][4 * ks + 1], pw[u][4 * ks + 2], pw[u][4 * ks + 3]};
        f_new[u][ks] = __builtin_bit_cast(bf16x8, v);
      }
    }
    // stage t + 2 must have landed; the copies of the DIST - 1 stages after it may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 1) * PER) : "memory");
    wg_barrier();
  };

  // Steps are taken two at a time (the two S^T buffers and the two P^T buffers swap roles without a copy): first the
  // pairs whose stages every row of the wave sees completely, then the rest with the mask, up to step nt (whose only
  // real work is the O^T product of the last stage); a pair may run one step past that, which contributes nothing.
  const int t_full = min(nt, (it.n0 + wave_row0) / BN) & ~1;
  int t = 0;
  for (; t < t_full; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::false_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::false_type{});
  }
  if (wave == 0 && !again && !direct) pending_claim = block_claim_issue(p.taken, xcd);
  for (; t <= nt; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::true_type{});
    // (the scores of stages up to nt - 1 have been looked at by the first of the last two steps; the barrier that ends the
    // second one publishes the word)
    if (__builtin_expect(__any(risk), 0)) {
#pragma unroll
      for (int w = 0; w < NW; ++w) *(volatile int*)((__bf16*)smem + ST_OFF + w * (ST_ROWS * D)) = 1;
    }
    step(t + 1, x[1], x[0], f[1], f[0], std::true_type{});
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  // every copy of this wave has landed (the last ones rewrote a slot nobody reads): after the barrier below the next
  // block may fill the ring again
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  const bool outgrown = __builtin_amdgcn_readfirstlane(*(volatile int*)stage) != 0;
  if (__builtin_expect(outgrown && !again, 0)) {  // (the same for all waves; the barrier at the head of the loop comes before the next copies)
    again = true;
    continue;
  }
  again = false;

  // ---- epilogue: O = O^T / l, LSE = ln(l) + m scale ----
  // (through the wave's staging tile: the lane that holds four values of a row writes them there, then every lane
  // moves one 16-byte chunk of a row to global memory, four whole rows per instruction; one unit after the other, so
  // that few values are in flight at a time)
  if (CUT && it.part >= 0) {  // a piece: O^T as it is, the reference maximum and the sum of each row
    float* const out = p.parts + ((int64_t)it.part * inner_n + inner) * kPartFloats;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float l_tot = sum_halves(l_run[u]);
      if (hh == 0) *reinterpret_cast<f32x2*>(out + kPartRowFloats + ((2 * wave + u) * 32 + l32) * 2) = f32x2{mc[u], l_tot};
      float* const dst = out + (2 * wave + u) * 4096 + lane * 4;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(dst + (db * 4 + g) * 256) =
              f32x4{oacc[u][db][4 * g], oacc[u][db][4 * g + 1], oacc[u][db][4 * g + 2], oacc[u][db][4 * g + 3]};
    }
  } else {
    // (the lane index is made opaque here: the addresses below depend on nothing else, and computed ahead of the loop
    // they would take registers for its whole length)
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int l32_e = lane_e & 31, hh_e = lane_e >> 5;
    __bf16* obase = p.o + (int64_t)it.q_row0 * q_stride + (int64_t)head * D;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = wave_row0 + 32 * u + l32_e;
      const float l_tot = sum_halves(l_run[u]);
      const float inv = 1.0f / l_tot;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const bf16x4 v = pack4(oacc[u][db][4 * g] * inv, oacc[u][db][4 * g + 1] * inv, oacc[u][db][4 * g + 2] * inv,
                                 oacc[u][db][4 * g + 3] * inv);
          *reinterpret_cast<bf16x4*>(stage + tile_elem<KC>(32 * u + l32_e, 4 * db + g) + 4 * hh_e) = v;
        }
      if (r < it.q_rows && hh_e == 0)
        p.lse[(int64_t)head * p.total_q + it.q_row0 + r] = (mc[u] + log2f(l_tot)) * 0.6931471805599453f;
#pragma unroll 2
      for (int i = 0; i < 32 * KC / 64; ++i) {
        const int x = (u * 32 * KC / 64 + i) * 64 + lane_e;
        const int row = x / KC, c = unswz<KC>(row, x % KC);
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + x * 8);
        if (wave_row0 + row < it.q_rows) *reinterpret_cast<bf16x8*>(obase + (int64_t)(wave_row0 + row) * q_stride + c * 8) = v;
      }
    }
  }
  if (direct) break;
  // on to the next block; the stores above are not waited for here
  int nb = 0;
  if (wave == 0) nb = block_claim_finish(p.taken, num_blocks, xcd, pending_claim);
  blk = broadcast_from_wave0(next_block, nb);
  }
  clock_log_stamp(p.clock_log, 1);
}

// ------------------------------------------------------------------------------------------------
// Pipelined forward for head_dim 256: one wave per SIMD, 32 query rows per wave (Q fragments and O^T take 192 accumulation
// registers; 64 rows would take 384), keys streamed in stages of 32.
//
// A step runs the three pieces of fwd_pipe_kernel -- O^T += V(t-1)^T P^T(t-1), S^T(t+1) = K(t+1) Q^T, P^T(t) = exp2(S^T(t) c - m c) -- as
// 16 mini-steps of one K row fragment and the S MFMA it feeds, one V^T fragment and the O MFMA it feeds, and the vector work of one
// score.  Every fragment feeds one MFMA only, so a step is bound by what a wave can issue: 48 LDS reads (16 cycles each) and 32 MFMAs
// (32 each), against half as many reads per MFMA at head_dim 128; the vector work, half of that per MFMA, hides under them.
// LDS holds four stages of K (t + 1 and, read ahead over the end of the step, t + 2 in use in step t; t + 3 and t + 4 on their way) and
// five of V (t - 1 and t in use, t + 1 and t + 2 on their way); a copy has more than a step to land.  Q comes in and O goes
// out through 64 KB of the V ring and behind it, which no stage needs at either end.
// Blocks that outgrow their reference maximum and the masked steps as in fwd_pipe_kernel; the maximum is that of two stages, and O and LSE
// have a sum of probabilities each (2-norm error of O, 1000 causal tokens, 8/2 heads, scores of 1 / 4 / 8 nats: 2.02e-3 / 1.83e-3 / 1.70e-3, with a
// moving maximum 2.02 / 1.80 / 1.66; with one stage and one sum 2.07 / 2.23 / 2.22.  The two cost long walks 1.8 %, short ones nothing).
// Against fwd_kernel's scheme, which it replaces here (online softmax, no pipelining, V^T images made by a launch before; 32/8 heads):
// packed 64K chunk 10.9 -> 8.3 ms, 8192 queries on 32768 keys 10.0 -> 7.5, 64 sequences of 256 342 -> 244 us, 909 queries on 5603 keys 256 -> 169,
// 148 on 595, 8/2 heads, 43 -> 25.  Two to five fragments read ahead and either order of a mini-step's reads make no difference.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 1) void fwd_wide_kernel(FwdArgs) {
  constexpr int D = 256;
  const FwdArgsPtr args = fwd_args();
  const FwdParams p = load_params(&args->p);
  const int num_blocks = args->num_blocks;
  constexpr int NW = 4;        // waves
  constexpr int BN = 32;       // key rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps of S^T = K Q^T
  constexpr int DB = D / 32;   // 32-row blocks of O^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int KS = 4, VS = 5;        // ring slots of K and of V
  constexpr int NF = DK;               // mini-steps per step
  constexpr int AHEAD = 3, RING = 4;   // fragments (of each kind) in flight, registers of the fragment rings
  constexpr int PER = BN * KC / 64 / NW;  // global->LDS copies per wave, tile and stage
  static_assert(2 * DB == DK && NF % RING == 0 && RING > AHEAD && 1 + PER * 3 < NF, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int K_OFF = 0;               // [KS][KT]  K rows of stage n in slot n % KS (chunk-major)
  constexpr int V_OFF = K_OFF + KS * KT; // [VS][KT]  V rows of stage n in slot n % VS
  // [NW][32][D] staging of a wave's 32 rows, rows of swizzled 16-byte chunks: V slots 2 .. 4 and the tile behind them.  Its first word (of
  // wave 0's tile) doubles as the slot through which wave 0 announces the next block.
  constexpr int ST_OFF = V_OFF + 2 * KT;
  constexpr int X_OFF = V_OFF + VS * KT; // the tile behind the V ring: nobody's while the steps run, but for the waves' words

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  __bf16* const stage = (__bf16*)smem + ST_OFF + wave * KT;
  int* const next_block = (int*)((__bf16*)smem + ST_OFF);
  volatile int* const outgrown = (volatile int*)((__bf16*)smem + X_OFF);  // some wave has seen a row outgrow its reference maximum

  const int xcd = xcd_of_this_wave();
  const bool direct = num_blocks <= (int)gridDim.x;
  int blk = blockIdx.x;
  if (!direct) {
    if (wave == 0) blk = block_claim_finish(p.taken, num_blocks, xcd, block_claim_issue(p.taken, xcd));
    blk = broadcast_from_wave0(next_block, blk);
  }
  bool again = false;  // the block is taken a second time, with every row's true maximum
  int pending_claim = 0;
  while (blk >= 0) {
  wg_barrier();  // every wave has read the announcement: the staging area may be written again
  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = __builtin_amdgcn_readfirstlane(blk % inner_n);
  const FwdItem it = load_item(p.items, args->items, __builtin_amdgcn_readfirstlane(blk / inner_n));
  const int kvh = __builtin_amdgcn_readfirstlane(inner % p.num_kv_heads), hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int wave_row0 = (wave / p.heads_per_wg) * 32;  // the wave's rows are wave_row0 .. + 31 of `head`
  const int n_wg = it.n0 + it.q_rows - 1;              // keys the last valid row sees
  const int nt = (n_wg + BN - 1) / BN;                 // stages

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  // ---- staging: copy i of a wave is piece 4 i + wave of a tile, 64 consecutive slots = two chunk columns of 32 rows.  Past the last
  // stage the last one is copied again. ----
  unsigned v_full[PER], v_last[PER];  // byte offset of the lane's chunk from the tile's first row: full tile, last tile
  {
    const int last_row = n_wg - 1 - (nt - 1) * BN;  // rows past the last key repeat it (masked)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int x = (i * NW + wave) * 64 + lane;
      const int off = (x >> 5) * 8, row = (x & 31) ^ (((x >> 5) & 3) << 2);
      v_full[i] = (unsigned)(row * (int)kv_stride + off) * 2u;
      v_last[i] = (unsigned)(min(row, last_row) * (int)kv_stride + off) * 2u;
    }
  }
  struct Stream {  // the next stage to copy, its first row, its slot
    int t, slot;
    const char* row;
  };
  Stream ks{0, 0, reinterpret_cast<const char*>(Kg)}, vs{0, 0, reinterpret_cast<const char*>(Vg)};
  auto copy_piece = [&](const Stream& st, int ring, int i) __attribute__((always_inline)) {
    dma16(st.row + (st.t == nt - 1 ? v_last[i] : v_full[i]), L + ring + st.slot * KT + (i * NW + wave) * 512);
  };
  auto advance = [&](Stream& st, int slots) __attribute__((always_inline)) {
    if (st.t + 1 < nt) {
      ++st.t;
      st.row += BN * kv_stride * 2;
    }
    st.slot = st.slot == slots - 1 ? 0 : st.slot + 1;
  };

  // per-lane operand addresses inside a tile (as in fwd_pipe_kernel)
  int x_off[2], t_off[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) x_off[par] = cm_elem(l32, 2 * par + hh);
  {
    const int j = lane & 15, grp = (lane >> 4) & 1;
    const int cl = 2 * grp + ((j & 3) >> 1);
    const int r0 = 4 * hh + (j >> 2);
#pragma unroll
    for (int half = 0; half < 2; ++half) t_off[half] = cm_elem(r0 + 8 * half, cl) + 4 * (j & 1);
  }
  const unsigned k_ev0 = lds_addr(L + K_OFF + x_off[0]), k_od0 = lds_addr(L + K_OFF + x_off[1]);
  const unsigned t_lo0 = lds_addr(L + V_OFF + t_off[0]), t_hi0 = lds_addr(L + V_OFF + t_off[1]);
  constexpr unsigned SLOT = KT * 2;  // bytes per ring slot
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c) __attribute__((always_inline)) {
    constexpr int k = decltype(ks_c)::value;
    return lds_asm_read16<(k >> 1) * (4 * 32 * 8) * 2>((k & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // prologue: K of stages 0 .. 2, V of stage 0 and the wave's rows of Q, then K(3) and V(1), which step 0 waits for at its end
  auto copy_tile = [&](Stream& st, int ring, int slots) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER; ++i) copy_piece(st, ring, i);
    advance(st, slots);
  };
#pragma unroll
  for (int n = 0; n < 3; ++n) copy_tile(ks, K_OFF, KS);
  copy_tile(vs, V_OFF, VS);
  {
    const __bf16* qbase = p.q + (int64_t)it.q_row0 * q_stride + (int64_t)head * D;
#pragma unroll 4
    for (int i = 0; i < 32 * KC / 64; ++i) {
      const int x = i * 64 + lane;
      const int row = x / KC, c = unswz<KC>(row, x % KC);
      const int r = min(wave_row0 + row, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
      dma16(qbase + (int64_t)r * q_stride + c * 8, stage + i * 512);
    }
  }
  copy_tile(ks, K_OFF, KS);
  copy_tile(vs, V_OFF, VS);
  // One wait the compiler can see for Q (and the copies before it): it then has no reason to put full waits for outstanding
  // loads into the loop.
  wait_all_but<2 * PER>();
  // Q fragments (B operands of S^T = K Q^T): lane holds Q[row = l32][16 ks + 8 hh ..+7].  (Opaque reads, as for all that is read or
  // written while copies are on their way.)
  const unsigned stage_addr = lds_addr((lds_bf16*)stage);
  bf16x8 qf[DK];
#pragma unroll
  for (int k = 0; k < DK; ++k) qf[k] = lds_asm_read16<0>(stage_addr + 2 * tile_elem<KC>(l32, 2 * k + hh));
  if (wave == 2) {  // V(-1), read in step 0: its slot is this wave's staging tile
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    static_assert(ST_OFF + 2 * KT == V_OFF + (VS - 1) * KT, "the slot of V(-1)");
    static_for<0, KT / 512>([&](auto i_c) __attribute__((always_inline)) { lds_asm_write16<decltype(i_c)::value * 1024>(stage_addr + lane * 16, z); });
  }
  if (wave == 3) lds_asm_write4(lds_addr(L + X_OFF), 0);  // (*outgrown, in its staging tile)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // (the fragments settle in their accumulation registers here: an opaque MFMA must not follow a write to one of its operands)
#pragma unroll
  for (int k = 0; k < DK; ++k) {
    asm volatile("" : "+v"(qf[k]));
    asm volatile("" : "+a"(qf[k]));
  }
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = zero16;
  f32x16 x[2];       // S^T, two buffers
  bf16x8 f[2][2];    // P^T as B operands: [buffer][k-step]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < 8; ++i) f[b][k][i] = (__bf16)0.0f;
  const float c = p.scale_log2;
  bf16x8 fv[RING], fk[RING];  // rings of V^T and of K fragments

  // S^T(0) = K(0) Q^T and the reference maximum of each row, over stages 0 and 1 (S^T(1) is formed for that alone, and again in step 0): the
  // largest probability is the one whose rounding matters most, and it is exact where the maximum is the reference.
  // Two sums: O is divided by the sum of the probabilities as they are rounded to bf16 for the product with V, so that a dominant
  // one's rounding cancels; LSE takes the unrounded sum.
  float mc, l_run = 0.f, l_rnd = 0.f;
  bf16x2 ones;
  ones[0] = (__bf16)1.0f; ones[1] = (__bf16)1.0f;
  {
    bf16x8 a[DK];
#pragma unroll
    for (int n = 1; n >= 0; --n) {
      static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) { a[decltype(ks_c)::value] = load_rows(k_ev0 + n * SLOT, k_od0 + n * SLOT, ks_c); });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int k = 0; k < DK; ++k) asm volatile("" : "+v"(a[k]));  // (after the wait, in this order)
      if (n == 0) wg_barrier();  // every wave has read K(0): step 0 copies K(4) over it
#pragma unroll
      for (int k = 0; k < DK; ++k) {
        f32x16& d_ = x[n];
        const bf16x8& b_ = qf[k];
        if (k == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a[k]), "a"(b_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a[k]), "a"(b_));
      }
    }
    mfma_settle();
    asm volatile("s_nop 15" : "+v"(x[0]), "+v"(x[1]));  // the reads below come after the MFMAs have written
    const int lim = it.n0 + wave_row0 + l32;  // visible iff key index < lim (>= 1)
    float mx = -INFINITY;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (BN * n + 8 * (i >> 2) + 4 * hh + (i & 3) < lim) mx = fmaxf(mx, x[n][i]);
    mc = max_halves(mx) * c;
  }
  if (__builtin_expect(again, 0)) {  // the maximum over all stages: S^T as in the loop, K read from global memory
    float mx = -INFINITY;
    for (int n = 0; n < nt; ++n) {
      const __bf16* kr = Kg + (int64_t)min(BN * n + l32, n_wg - 1) * kv_stride + 8 * hh;
      f32x16 d = zero16;
#pragma unroll
      for (int k = 0; k < DK; ++k) d = mfma32(*reinterpret_cast<const bf16x8*>(kr + 16 * k), qf[k], d);
      const int lim = it.n0 + wave_row0 + l32 - BN * n;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + 4 * hh + (i & 3) < lim) mx = fmaxf(mx, d[i]);
    }
    mc = max_halves(mx) * c;
  }
  bool risk = false;
  const float big = __builtin_amdgcn_exp2f(p.ref_limit);

  // the first fragments of step 0: V(-1) (zeros) and K(1)
  {
    const unsigned sT = (VS - 1) * SLOT;
    static_for<0, AHEAD>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      fv[m] = load_t(t_lo0 + sT, t_hi0 + sT, m_c);
      fk[m] = load_rows(k_ev0 + SLOT, k_od0 + SLOT, m_c);
    });
  }

  // Mini-step m reads the fragments of mini-step m + AHEAD (past the end: the next step's first ones), three instructions, so that
  // "the fragments of mini-step m have arrived" is "at most 3 (AHEAD - 1) LDS reads are outstanding" at its start.
  int sV = 0, sK = 1;  // slots of V(t) and of K(t + 1)
  auto step = [&](int t, f32x16& cur, f32x16& nxt, bf16x8 (&f_old)[2], bf16x8 (&f_new)[2], auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int sM = sV == 0 ? VS - 1 : sV - 1, sN = sK == KS - 1 ? 0 : sK + 1;  // V(t - 1), K(t + 2)
    const unsigned t_lo = t_lo0 + sM * SLOT, t_hi = t_hi0 + sM * SLOT, n_lo = t_lo0 + sV * SLOT, n_hi = t_hi0 + sV * SLOT;
    const unsigned k_ev = k_ev0 + sK * SLOT, k_od = k_od0 + sK * SLOT, n_ev = k_ev0 + sN * SLOT, n_od = k_od0 + sN * SLOT;
    // MASKED: element i (key 8 (i / 4) + 4 hh + i % 4 of the stage) is visible iff 8 (i / 4) + i % 4 < lim
    int lim = 0;
    if (MASKED) lim = t < nt ? it.n0 + wave_row0 + l32 - BN * t - 4 * hh : -0x40000000;
    unsigned pw[8];  // P^T(t), packed pairs
    float ps = 0.f, pr = 0.f;
    float e_hold[2];
    // (a pair is converted one mini-step after its exponentials: a transcendental result cannot be consumed by the very next instruction)
    auto finish_pair = [&](int j) __attribute__((always_inline)) {
      bf16x2 w;
      w[0] = (__bf16)e_hold[0]; w[1] = (__bf16)e_hold[1];
      ps += e_hold[0] + e_hold[1];
      asm volatile("" : "+v"(ps));
      pr = __builtin_amdgcn_fdot2_f32_bf16(w, ones, pr, false);
      asm volatile("" : "+v"(pr));
      unsigned wu = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(wu));
      pw[j] = wu;
    };
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(fv[m % RING]), "+v"(fk[m % RING]) : "n"(3 * (AHEAD - 1)));
      {
        constexpr int mm = m + AHEAD;
        if constexpr (mm < NF) {
          fk[mm % RING] = load_rows(k_ev, k_od, std::integral_constant<int, mm>{});
          fv[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm>{});
        } else {
          fk[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{});
          fv[mm % RING] = load_t(n_lo, n_hi, std::integral_constant<int, mm - NF>{});
        }
      }
      {
        const bf16x8& a_ = fk[m % RING];
        f32x16& d_ = nxt;
        const bf16x8& b_ = qf[m];
        if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
      }
      // K(t + 4) and V(t + 2), one copy in mini-steps 1, 2, 4, 5, 7, 8, 10, 11
      if constexpr (m % 3 != 0 && m / 3 < PER) {
        if constexpr (m % 3 == 1) copy_piece(ks, K_OFF, m / 3);
        else copy_piece(vs, V_OFF, m / 3);
      }
      __builtin_amdgcn_sched_barrier(0);
      oacc[m % DB] = mfma32(fv[m % RING], f_old[m / DB], oacc[m % DB]);
      {  // the vector work of score m
        if constexpr (m > 0 && m % 2 == 0) finish_pair(m / 2 - 1);
        float tt = cur[m] * c - mc;
        if (MASKED) {
          if (8 * (m >> 2) + (m & 3) >= lim) tt = -INFINITY;
        }
        e_hold[m % 2] = __builtin_amdgcn_exp2f(tt);
        asm volatile("" : "+v"(e_hold[m % 2]));
      }
      if constexpr (m == NF - 2) {  // bookkeeping for the next step (this step's copies have been issued)
        advance(ks, KS);
        advance(vs, VS);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    finish_pair(7);
    sV = sV == VS - 1 ? 0 : sV + 1;
    sK = sN;
    risk |= !(ps < big);
    l_run += ps;
    l_rnd += pr;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      u32x4 v = {pw[4 * k], pw[4 * k + 1], pw[4 * k + 2], pw[4 * k + 3]};
      f_new[k] = __builtin_bit_cast(bf16x8, v);
    }
    // the copies of the step before (K(t + 3), V(t + 1)) must have landed; this step's may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
    wg_barrier();
  };

  // (as in fwd_pipe_kernel)
  const int t_full = min(nt, (it.n0 + wave_row0) / BN) & ~1;
  int t = 0;
  for (; t < t_full; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::false_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::false_type{});
  }
  if (wave == 0 && !again && !direct) pending_claim = block_claim_issue(p.taken, xcd);
  for (; t <= nt; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::true_type{});
    if (__builtin_expect(__any(risk), 0)) *outgrown = 1;
    step(t + 1, x[1], x[0], f[1], f[0], std::true_type{});
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < RING; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fv[i]), "+v"(fk[i]));
  // every copy of this wave has landed (the last ones rewrote slots nobody reads)
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  const bool retake = __builtin_amdgcn_readfirstlane(*outgrown) != 0 && !again;
  wg_barrier();  // nobody reads the rings, and nobody copies into them, any more: O may be staged there
  if (__builtin_expect(retake, 0)) {  // (the same for all waves)
    again = true;
    continue;
  }
  again = false;

  // ---- epilogue: O = O^T / l, LSE = ln(l) + m scale, through the wave's staging tile (as in fwd_pipe_kernel) ----
  {
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int l32_e = lane_e & 31, hh_e = lane_e >> 5;
    __bf16* obase = p.o + (int64_t)it.q_row0 * q_stride + (int64_t)head * D;
    const int r = wave_row0 + l32_e;
    const float l_tot = sum_halves(l_run);
    const float inv = 1.0f / sum_halves(l_rnd);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const bf16x4 v = pack4(oacc[db][4 * g] * inv, oacc[db][4 * g + 1] * inv, oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv);
        *reinterpret_cast<bf16x4*>(stage + tile_elem<KC>(l32_e, 4 * db + g) + 4 * hh_e) = v;
      }
    if (r < it.q_rows && hh_e == 0) p.lse[(int64_t)head * p.total_q + it.q_row0 + r] = (mc + log2f(l_tot)) * 0.6931471805599453f;
#pragma unroll 4
    for (int i = 0; i < 32 * KC / 64; ++i) {
      const int y = i * 64 + lane_e;
      const int row = y / KC, ch = unswz<KC>(row, y % KC);
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(stage + y * 8);
      if (wave_row0 + row < it.q_rows) *reinterpret_cast<bf16x8*>(obase + (int64_t)(wave_row0 + row) * q_stride + ch * 8) = v;
    }
  }
  if (direct) break;
  // on to the next block; the stores above are not waited for here
  int nb = 0;
  if (wave == 0) nb = block_claim_finish(p.taken, num_blocks, xcd, pending_claim);
  blk = broadcast_from_wave0(next_block, nb);
  }
}

// ------------------------------------------------------------------------------------------------
// Forward of head_dim 256 with 64 query rows per wave, where that ends sooner than fwd_wide_kernel (fwd_tall_pays)
//
// As in the backward's dkv_tall_blocks the accumulators (O^T of 64 rows) fill the accumulation registers and Q takes half of the others, so that every
// fragment feeds two MFMAs (one per 32-row unit): half the LDS reads and copies per MFMA.  Step t is
//     S^T(t) = K(t) Q^T      O^T += V(t-1)^T P^T(t-1)                                  (matrix pipe, in this order)
//     P^T(t) = exp2(S^T(t) c - m c)  from the end of S^T(t) until the next step's second half needs it       (vector)
// as 32 mini-steps of one LDS fragment and the two MFMAs it feeds, each MFMA with its even share of the vector work behind it.  Four ring slots of K and of V:
// K(t), V(t - 1) and what is read ahead in use, K(t + 3) and V(t + 2) on their way.  Reference maxima, both sums and blocks that are taken again
// as in fwd_wide_kernel.
// Bound by the rate at which MFMAs issue (their share of the cycles times the clock that the chip's power leaves).  fwd_wide_kernel -> this, us, 32/8 heads:
// packed 64K tokens 8254 -> 6471, 8192 queries on 32768 keys 7329 -> 5658, 4096 causal tokens 302 -> 242, 64 sequences of 256 253 -> 235.
// ------------------------------------------------------------------------------------------------
// The schedule of a step: mini-step m issues the read of fragment m + AHEAD (two instructions for those of V^T, the second half).
template <int DK, int AHEAD>
struct FwdTallOrder {
  static constexpr int NF = 2 * DK, DB = DK / 2;
  static constexpr int EXP0 = DK + 2;  // mini-step in which the vector work starts
  static constexpr int cost(int k) { return (k % NF) >= DK ? 2 : 1; }
  static constexpr int exps(int m) { return spread(32, EXP0, EXP0 + 2 * DK - 4, m); }  // scores done by the end of mini-step m (from NF on: of the next step)
  static constexpr int wait(int m) {
    int n = 0;
    for (int i = m - AHEAD + 1; i < m; ++i) n += cost((i + AHEAD + NF) % NF);
    return n;
  }
  // P of a k-step's keys is packed before the first product that reads it (pair 7 when score 16 has been done)
  static_assert(exps(NF + DK - 1) >= 17 && exps(NF + DK + DB - 1) == 32 && exps(NF + DK - 2) == 32, "the order of a step");
};

__global__ __launch_bounds__(256, 1) void fwd_tall_kernel(FwdArgs) {
  constexpr int D = 256;
  const FwdArgsPtr args = fwd_args();
  const FwdParams p = load_params(&args->p);
  const int num_blocks = args->num_blocks;
  constexpr int NW = 4;        // waves
  constexpr int BN = 32;       // key rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps of S^T = K Q^T
  constexpr int DB = D / 32;   // 32-row blocks of O^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int NS = 4;        // ring slots of K and of V
  constexpr int NF = 2 * DK;   // fragments (mini-steps) per step: K rows, V^T
  constexpr int AHEAD = 4, RING = 8;      // fragments in flight, names of the fragment ring
  constexpr int PER = BN * KC / 64 / NW;  // global->LDS copies per wave, tile and stage
  constexpr int COPY_EVERY = NF / (2 * PER);
  using Order = FwdTallOrder<DK, AHEAD>;
  static_assert(2 * DB == DK && NF % RING == 0 && NF % (2 * PER) == 0 && COPY_EVERY > 1, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int V_OFF = NS * KT;         // [NS][KT] K rows of stage n in slot n % NS (chunk-major), then V likewise; at the end the waves' rows of O
  int* const next_block = (int*)((__bf16*)smem + 2 * NS * KT);
  volatile int* const outgrown = (volatile int*)(next_block + 1);  // some wave has seen a row outgrow its reference maximum

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the lane is counted anew where it is needed, as in dkv_tall_blocks)
  auto lane_id = []() __attribute__((always_inline)) {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
  };

  const int xcd = xcd_of_this_wave();
  const bool direct = num_blocks <= (int)gridDim.x;
  int blk = blockIdx.x;
  if (!direct) {
    if (wave == 0) blk = block_claim_finish(p.taken, num_blocks, xcd, block_claim_issue(p.taken, xcd));
    blk = broadcast_from_wave0(next_block, blk);
  }
  bool again = false;  // the block is taken a second time, with every row's true maximum
  int pending_claim = 0;
  while (blk >= 0) {
  wg_barrier();  // every wave has read the announcement and `outgrown`
  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = __builtin_amdgcn_readfirstlane(blk % inner_n);
  const FwdItem it = load_item(p.items, args->items, __builtin_amdgcn_readfirstlane(blk / inner_n));
  const int kvh = __builtin_amdgcn_readfirstlane(inner % p.num_kv_heads), hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int wave_row0 = (wave / p.heads_per_wg) * 64;  // the wave's rows are wave_row0 .. + 63 of `head`
  const int n_wg = it.n0 + it.q_rows - 1;              // keys the last valid row sees
  const int nt = (n_wg + BN - 1) / BN;                 // stages
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  // ---- staging: copy i of a wave is piece 4 i + wave of a tile, 64 consecutive slots = two chunk columns of 32 rows, which have the same order of rows for all
  // copies of a wave.  Past the last stage the last one is copied again, rows past the last key repeat it (masked). ----
  unsigned v_full, v_last;  // byte offset of the lane's chunk from the tile's first row, but for the piece's own 32 bytes: full tile, last tile
  {
    const int lane = lane_id(), hh = lane >> 5, row = (lane & 31) ^ ((2 * (wave & 1) + hh) << 2);
    v_full = (unsigned)(row * (int)kv_stride + 8 * hh) * 2u;
    v_last = (unsigned)(min(row, n_wg - 1 - (nt - 1) * BN) * (int)kv_stride + 8 * hh) * 2u;
  }
  struct Stream {  // the next stage to copy, its first row, its slot
    int t, slot;
    const char* row;
  };
  Stream ks{0, 0, reinterpret_cast<const char*>(Kg)}, vs{0, 0, reinterpret_cast<const char*>(Vg)};
  auto copy_piece = [&](const Stream& st, int ring, int i) __attribute__((always_inline)) {
    const int piece = i * NW + wave;
    unsigned off = st.t == nt - 1 ? v_last : v_full;
    asm volatile("" : "+v"(off));
    dma16(st.row + piece * 32 + off, L + ring + st.slot * KT + piece * 512);
  };
  auto advance = [&](Stream& st) __attribute__((always_inline)) {
    if (st.t + 1 < nt) {
      ++st.t;
      st.row += BN * kv_stride * 2;
    }
    st.slot = st.slot == NS - 1 ? 0 : st.slot + 1;
  };
  auto copy_tile = [&](Stream& st, int ring) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER; ++i) copy_piece(st, ring, i);
    advance(st);
  };

  // byte addresses of this lane's operand reads in the tile of slot 0 (as in dkv_tall_blocks)
  constexpr unsigned ROW8 = 8 * 16;
  unsigned ev0, lo0;
  {
    const int lane = lane_id(), l32 = lane & 31, hh = lane >> 5;
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    ev0 = lds_addr(L + cm_elem(l32, hh));
    lo0 = lds_addr(L + V_OFF + cm_elem(r0, cl) + 4 * (j & 1));
  }
  constexpr unsigned SLOT = KT * 2;  // bytes per ring slot
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c) __attribute__((always_inline)) {
    constexpr int k = decltype(ks_c)::value;
    return lds_asm_read16<(k >> 1) * (4 * 32 * 8) * 2 + (k & 1) * 1024>((k & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // prologue: K of stages 0 .. 2, V of stages 0 and 1, the wave's rows of Q
#pragma unroll
  for (int n = 0; n < 3; ++n) copy_tile(ks, 0);
#pragma unroll
  for (int n = 0; n < 2; ++n) copy_tile(vs, V_OFF);
  bf16x8 qf[2][DK];  // B operands of S^T = K Q^T: lane holds Q[row = 32 u + l32][16 ks + 8 hh ..+7]
  {
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = min(wave_row0 + 32 * u + (lane & 31), it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
      const __bf16* const src = p.q + (int64_t)(it.q_row0 + r) * q_stride + (int64_t)head * D + 8 * (lane >> 5);
#pragma unroll
      for (int k = 0; k < DK; ++k) qf[u][k] = *reinterpret_cast<const bf16x8*>(src + 16 * k);
    }
    bf16x8 z;  // V(-1), read in step 0 (P(-1) = 0)
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
#pragma unroll
    for (int i = 0; i < KT / (NW * 64 * 8); ++i) lds_store8(L + V_OFF + (NS - 1) * KT + (i * NW * 64 + wave * 64 + lane) * 8, z);
    if (threadIdx.x == 0) *outgrown = 0;
  }
  wait_all_but<0>();  // (a wait the compiler can see, so that it puts none for these loads into the loop)
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float c = p.scale_log2;
  f32x16 x[2][2];    // S^T, then P^T: [buffer][unit]
  u32x4 f[2][2][2];  // P^T as B operands: [buffer][unit][k-step], pairs of bf16
  bf16x8 fr[RING];

  // The reference maximum of each row, over stages 0 and 1 (fwd_wide_kernel)
  float mc[2], l_run[2] = {0.f, 0.f}, l_rnd[2] = {0.f, 0.f}, ps[2] = {0.f, 0.f}, pr[2] = {0.f, 0.f};  // (ps, pr: a stage's own sums)
  bf16x2 ones;
  ones[0] = (__bf16)1.0f; ones[1] = (__bf16)1.0f;
  {
    const int lane = lane_id();
    bf16x8 a[DK];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) { a[decltype(ks_c)::value] = load_rows(ev0 + n * SLOT, (ev0 + n * SLOT) ^ ROW8, ks_c); });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int k = 0; k < DK; ++k) asm volatile("" : "+v"(a[k]));  // (after the wait, in this order)
#pragma unroll
      for (int k = 0; k < DK; ++k)
#pragma unroll
        for (int u = 0; u < 2; ++u) x[n][u] = mfma32(a[k], qf[u][k], k == 0 ? zero16 : x[n][u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int lim = it.n0 + wave_row0 + 32 * u + (lane & 31);  // visible iff key index < lim (>= 1)
      float mx = -INFINITY;
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (BN * n + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) < lim) mx = fmaxf(mx, x[n][u][i]);
      mc[u] = max_halves(mx) * c;
    }
  }
  if (__builtin_expect(again, 0)) {  // the maximum over all stages: K read from global memory
    const int lane = lane_id();
    float mx[2] = {-INFINITY, -INFINITY};
    for (int n = 0; n < nt; ++n) {
      const __bf16* kr = Kg + (int64_t)min(BN * n + (lane & 31), n_wg - 1) * kv_stride + 8 * (lane >> 5);
      f32x16 d[2] = {zero16, zero16};
#pragma unroll
      for (int k = 0; k < DK; ++k) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kr + 16 * k);
#pragma unroll
        for (int u = 0; u < 2; ++u) d[u] = mfma32(a, qf[u][k], d[u]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int lim = it.n0 + wave_row0 + 32 * u + (lane & 31) - BN * n;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) < lim) mx[u] = fmaxf(mx[u], d[u][i]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) mc[u] = max_halves(mx[u]) * c;
  }

  f32x16 oacc[2][DB];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[u][db] = zero16;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[1][u][i] = i < 8 ? 0.f : -INFINITY;  // P(-1) = 0, of which the second half is still S(-1)
#pragma unroll
    for (int k = 0; k < 2; ++k) f[0][u][k] = f[1][u][k] = u32x4{0, 0, 0, 0};
  }
  static_for<0, AHEAD>([&](auto k_c) __attribute__((always_inline)) { fr[decltype(k_c)::value] = load_rows(ev0, ev0 ^ ROW8, k_c); });

  int slot = 0;  // of K(t) and V(t)
  auto step = [&](int t, f32x16 (&so)[2], f32x16 (&sn)[2], u32x4 (&po)[2][2], u32x4 (&pn)[2][2]) __attribute__((always_inline)) {
    const int prv = slot == 0 ? NS - 1 : slot - 1, nxt = slot == NS - 1 ? 0 : slot + 1;
    const unsigned k_ev = ev0 + slot * SLOT, k_od = k_ev ^ ROW8, n_ev = ev0 + nxt * SLOT, n_od = n_ev ^ ROW8;
    const unsigned t_lo = lo0 + prv * SLOT, t_hi = t_lo ^ ROW8;
    // Element y of the vector work: 4 g4 + (y % 4) of unit (y / 4) % 2, g4 = y / 8; the rows of a k-step come first.  A pair is packed, and added to
    // the sums, one element late (an exponential cannot be used by the next instruction).
    auto exp_one = [&](f32x16 (&s)[2], auto y_c) __attribute__((always_inline)) {
      constexpr int y = decltype(y_c)::value, u = y / 4 % 2, i = 4 * (y / 8) + y % 4;
      float e = __builtin_amdgcn_exp2f(s[u][i] * c - mc[u]);
      asm volatile("" : "+v"(e));
      s[u][i] = e;
    };
    auto pack = [&](f32x16 (&s)[2], u32x4 (&pw)[2][2], auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, u = j / 2 % 2, w = 2 * (j / 4) + j % 2;
      bf16x2 v;
      v[0] = (__bf16)s[u][2 * w]; v[1] = (__bf16)s[u][2 * w + 1];
      ps[u] += s[u][2 * w] + s[u][2 * w + 1];
      asm volatile("" : "+v"(ps[u]));
      pr[u] = __builtin_amdgcn_fdot2_f32_bf16(v, ones, pr[u], false);
      asm volatile("" : "+v"(pr[u]));
      unsigned b = __builtin_bit_cast(unsigned, v);
      asm volatile("" : "+v"(b));
      pw[u][w / 4][w % 4] = b;
    };
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(Order::wait(m)));
      if constexpr (m == Order::EXP0) {  // keys that a row does not see, and whole stages past the end of the walk
        if (__builtin_expect(BN * (t + 1) > it.n0 + wave_row0, 0)) {
          const int lane = lane_id();
          const int lim0 = t < nt ? it.n0 + wave_row0 + (lane & 31) - BN * t - 4 * (lane >> 5) : -0x40000000, lim1 = lim0 + 32;
          const float none = -INFINITY;
          asm volatile("s_nop 15\n\ts_nop 7" : "+v"(sn[0]), "+v"(sn[1]));  // S(t) has been written
#pragma unroll
          for (int u = 0; u < 2; ++u)
            static_for<0, 16>([&](auto i_c) __attribute__((always_inline)) {
              constexpr int i = decltype(i_c)::value;
              float v = sn[u][i];
              const int lim = u ? lim1 : lim0;
              asm volatile("v_cmp_ge_i32 vcc, %1, %2\n\ts_nop 1\n\tv_cndmask_b32 %0, %0, %3, vcc" : "+v"(v) : "n"(8 * (i >> 2) + (i & 3)), "v"(lim), "v"(none) : "vcc");
              sn[u][i] = v;
            });
        }
      }
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's K rows)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < DK) fr[mm % RING] = load_rows(k_ev, k_od, std::integral_constant<int, mm>{});
        else if constexpr (mm < NF) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm - DK>{});
        else fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{});
      }
      const bf16x8 fa = fr[m % RING];
      auto mma = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        if constexpr (m < DK) {
          const bf16x8& a_ = fa;  // (named references: variables used only inside an asm statement are not captured)
          f32x16& d_ = sn[u];
          const bf16x8& b_ = qf[u][m];
          if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "v"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "v"(b_));
        } else {
          constexpr int k = (m - DK) / DB, db = (m - DK) % DB;
          oacc[u][db] = mfma32(fa, __builtin_bit_cast(bf16x8, po[u][k]), oacc[u][db]);
        }
      };
      constexpr int M = m >= Order::EXP0 ? m : m + NF;  // (from EXP0 on the work is this stage's, before it the last one's)
      constexpr int e0 = Order::exps(M - 1), e1 = Order::exps(M), em = e0 + (e1 - e0 + 1) / 2;
      auto work = [&](auto lo_c, auto hi_c, auto last_c) __attribute__((always_inline)) {
        constexpr int lo = decltype(lo_c)::value, hi = decltype(hi_c)::value;
        constexpr int j0 = lo == 32 ? 16 : lo > 0 ? (lo - 1) / 2 : 0, j1 = hi == 32 && decltype(last_c)::value ? 16 : hi > 0 ? (hi - 1) / 2 : 0;
        f32x16(&s)[2] = m >= Order::EXP0 ? sn : so;
        u32x4(&pw)[2][2] = m >= Order::EXP0 ? pn : po;
        static_for<lo, hi>([&](auto y_c) __attribute__((always_inline)) { exp_one(s, y_c); });
        if constexpr (j0 < j1) static_for<j0, j1>([&](auto j_c) __attribute__((always_inline)) { pack(s, pw, j_c); });
      };
      mma(std::integral_constant<int, 0>{});
      if constexpr (e0 < em) work(std::integral_constant<int, e0>{}, std::integral_constant<int, em>{}, std::bool_constant<em == 32 && em == e1>{});
      __builtin_amdgcn_sched_barrier(0);
      mma(std::integral_constant<int, 1>{});
      if constexpr (em < e1) work(std::integral_constant<int, em>{}, std::integral_constant<int, e1>{}, std::true_type{});
      if constexpr (m == Order::EXP0 - 1) {  // (the stage before is complete)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          l_run[u] += ps[u];
          l_rnd[u] += pr[u];
          ps[u] = pr[u] = 0.f;
        }
      }
      if constexpr (m % COPY_EVERY == 1) {  // K(t + 3) and V(t + 2), one copy every COPY_EVERY mini-steps
        if constexpr (m / COPY_EVERY % 2 == 0) copy_piece(ks, 0, m / COPY_EVERY / 2);
        else copy_piece(vs, V_OFF, m / COPY_EVERY / 2);
      }
      if constexpr (m == NF - 2) {  // bookkeeping for the next step (this step's copies have been issued)
        advance(ks);
        advance(vs);
        slot = nxt;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // the copies of the step before (K(t + 2), V(t + 1)) must have landed; this step's may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
    wg_barrier();
  };
  // the last product is O^T of stage nt - 1 in step nt; a pair of steps may run one past that, which contributes nothing
  const int claim_at = max(0, nt - 3) & ~1;
  for (int t = 0; t <= nt; t += 2) {
    if (t == claim_at && wave == 0 && !again && !direct) pending_claim = block_claim_issue(p.taken, xcd);
    step(t, x[1], x[0], f[1], f[0]);
    step(t + 1, x[0], x[1], f[0], f[1]);
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  const float big = __builtin_amdgcn_exp2f(p.ref_limit);
  if (__builtin_expect(__any(!(l_run[0] < big) || !(l_run[1] < big)), 0)) *outgrown = 1;
  // every copy of this wave has landed (the last ones rewrote slots nobody reads)
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  wg_barrier();  // nobody reads the rings, and nobody copies into them, any more: O may be staged there
  const bool retake = __builtin_amdgcn_readfirstlane(*outgrown) != 0 && !again;
  if (__builtin_expect(retake, 0)) {  // (the same for all waves)
    again = true;
    continue;
  }
  again = false;

  // ---- epilogue: O = O^T / l, LSE = ln(l) + m scale, through 64 rows of LDS of the wave's own ----
  {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int l32 = lane & 31, hh = lane >> 5;
    lds_bf16* const stage = L + wave * (64 * D);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float l_tot = sum_halves(l_run[u]), inv = 1.0f / sum_halves(l_rnd[u]);
      const int r = wave_row0 + 32 * u + l32;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(__attribute__((address_space(3))) bf16x4*)(stage + tile_elem<KC>(32 * u + l32, 4 * db + g) + 4 * hh) =
              pack4(oacc[u][db][4 * g] * inv, oacc[u][db][4 * g + 1] * inv, oacc[u][db][4 * g + 2] * inv, oacc[u][db][4 * g + 3] * inv);
      if (r < it.q_rows && hh == 0) p.lse[(int64_t)head * p.total_q + it.q_row0 + r] = (mc[u] + log2f(l_tot)) * 0.6931471805599453f;
    }
    __bf16* const obase = p.o + (int64_t)(it.q_row0 + wave_row0) * q_stride + (int64_t)head * D;
#pragma unroll 4
    for (int i = 0; i < 64 * KC / 64; ++i) {
      const int y = i * 64 + lane, row = y / KC, ch = unswz<KC>(row, y % KC);
      const bf16x8 v = lds_load8(stage + y * 8);
      if (wave_row0 + row < it.q_rows) *reinterpret_cast<bf16x8*>(obase + (int64_t)row * q_stride + ch * 8) = v;
    }
  }
  if (direct) break;
  // on to the next block; the stores above are not waited for here
  int nb = 0;
  if (wave == 0) nb = block_claim_finish(p.taken, num_blocks, xcd, pending_claim);
  blk = broadcast_from_wave0(next_block, nb);
  }
}

// ------------------------------------------------------------------------------------------------
// Forward of small chunks: a workgroup takes 32 query rows of HG heads of one group, and KS waves per head divide the keys: those of split x
// take stages x, x + KS, ... of 32 keys.  The HG waves of a split share its stages (one barrier per step; a single head's waves wait for
// nothing but their own copies), and the splits' sums meet in LDS at the end, where they are put together as fwd_merge_kernel does it.
// What a small chunk waits for is one wave's chain of stages (a copy, reads, products, exponentials, products: 0.9 - 1.4 us a stage), so the
// chain is cut eight ways where there is one head to a workgroup, and two waves per SIMD overlap.  More heads per workgroup read
// a stage fewer times from the L2 and cut the chain less; choose_shared_heads weighs it.  Kernel before -> now, us: 1024 tokens, 8/8
// heads, head_dim 64, 16.9 -> 7.9, 100 queries on 10100 keys, 32/8, 124 -> 40; head_dim 128, 500 tokens, 32/8, 21.5 -> 10.7, 8/8, 22.2 -> 8.0; 203
// queries on 1704 keys with 611 packed tokens, 32/8, 30.1 -> 21.6.  One head with four waves and two slots each instead of eight with
// one: 1000 tokens, 8/8, 15.1 instead of 11.2; there K of the next stage is copied once K has been read, V once V has been (both after V: 11.2 -> 11.0,
// 3000 tokens, 8/8, 44.6 -> 42.1).  Two heads in one wave with four waves: 203 + 611 queries as above 29.0.
//
// Tiles are rows (a copy instruction fetches whole rows; chunk-major tiles touch up to eight times the cache lines), swizzled by share_swz.
// ------------------------------------------------------------------------------------------------
constexpr float kNoMax = -3.4028234e38f;  // reference maximum of a row that has seen no key yet
template <int D, int HG, int KS, int NS>
constexpr size_t share_smem() {  // the splits' slots of a K and a V tile and the heads' Q tiles, or each wave's O; a maximum and a sum per wave and row
  const size_t tiles = (size_t)(KS * NS * 2 + HG) * 32 * share_cols(D) * 2, sums = (size_t)HG * KS * 32 * D * 4;
  return (tiles > sums ? tiles : sums) + (size_t)HG * KS * 32 * 2 * sizeof(float);
}

template <int D, int HG, int KS, int NS>
__global__ __launch_bounds__(HG * KS * 64, D == 64 ? 4 : HG * KS / 4) void fwd_share_kernel(FwdArgs) {
  constexpr int W = HG * KS;
  constexpr int ROW = share_cols(D) * 2;  // bytes of a row in LDS
  constexpr int C = ROW / 16, DK = D / 16, DB = D / 32;
  constexpr int TILE = 32 * ROW;      // bytes of a tile
  constexpr int PT = C / 2;           // copies of 64 chunks per tile
  constexpr int RPC = 64 / C;         // rows per copy
  constexpr int PPW = 2 * PT / HG;    // copies of a stage per wave
  constexpr int NQ = DB * 4;          // accumulator quarters of a head
  constexpr int NQW = (NQ + KS - 1) / KS;  // of which a wave puts together: consecutive ones, or every KS-th where they do not divide evenly
  static_assert(PPW % (D == 64 ? 2 : 4) == 0 && (HG == 1 || PT % PPW == 0));
  static_assert(HG == 1 ? NS <= 2 : NS == 2 || NS == 3);
  const FwdArgsPtr args = fwd_args();
  const FwdParams p = load_params(&args->p);

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), unit = wave % HG, split = wave / HG;
  const int l32 = lane & 31, hh = lane >> 5;
  lds_bf16* const region = (lds_bf16*)(smem + split * (NS * 2 * TILE));
  lds_bf16* const q_tiles = (lds_bf16*)(smem + KS * NS * 2 * TILE);  // [HG][32][D]
  lds_f32* const ml = (lds_f32*)(smem + share_smem<D, HG, KS, NS>() - W * 32 * 2 * sizeof(float));
  if constexpr (W > 4) stagger_wave_priority();

  const int inner_n = p.num_kv_heads * p.head_splits, inner = blockIdx.x % inner_n;
  const FwdItem it = load_item(p.items, args->items, blockIdx.x / inner_n);
  const int kvh = inner % p.num_kv_heads, hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * HG + unit;
  const int n_keys = it.n0 + it.q_rows - 1;  // keys visible to the last row
  const int nt = (n_keys + 31) / 32;
  const int n_mine = nt > split ? (nt - split + KS - 1) / KS : 0;

  const int64_t q_stride = (int64_t)p.num_q_heads * D;
  const int kv_stride = p.num_kv_heads * D;

  // copy i of a tile fills rows RPC i .. RPC (i + 1) - 1; a row's index splits into the lane's part and the copy's
  const int c_row = lane / C, c_chunk = (lane % C) ^ share_swz<D>(c_row);
  auto column = [&](int row_of_copy) __attribute__((always_inline)) {  // of the lane's chunk
    const int chunk = c_chunk ^ share_swz<D>(row_of_copy);
    return (D == 96 ? min(chunk, D / 8 - 1) : chunk) * 8;
  };
  // ---- Q: the waves of a head copy every KS-th piece of its tile ----
#pragma unroll
  for (int x = 0; x < PT; x += KS) {
    const int i = x + split;
    if (PT % KS != 0 && i >= PT) break;
    const int row = min(RPC * i + c_row, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
    dma16(p.q + (int64_t)(it.q_row0 + row) * q_stride + (int64_t)head * D + column(RPC * i),
          q_tiles + (unit * PT + i) * 512);
  }
  // ---- K and V: wave `unit` of a split copies pieces PPW unit .. + PPW - 1 of the 2 PT pieces of a stage (K, then V) ----
  const int piece0 = unit * PPW;
  const __bf16* const Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* const Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const int row0 = HG == 1 ? 0 : RPC * (piece0 % PT);  // first row the wave copies
  const __bf16* const Xg = HG == 1 || piece0 < PT ? Kg : Vg;
  const int c_off = c_row * kv_stride;
  auto copy_pieces = [&](int i, int slot, auto first_c, auto end_c) __attribute__((always_inline)) {
    const int t = split + KS * i;
    const int64_t toff = (int64_t)(32 * t + row0) * kv_stride;  // wave-uniform
    lds_bf16* const dst = region + slot * TILE + piece0 * 512;
    const int last_row = n_keys - 1 - 32 * t - row0;
    auto src = [&](int x) __attribute__((always_inline)) { return (HG > 1 || x < PT ? Xg : Vg) + toff; };
    if (last_row >= 31) {  // (a scalar base and a 32-bit offset in bytes)
      static_for<decltype(first_c)::value, decltype(end_c)::value>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int x = decltype(x_c)::value, j = x % PT;
        const char* const row = reinterpret_cast<const char*>(src(x) + (int64_t)(RPC * j) * kv_stride);
        dma16(row + (unsigned)(2 * (c_off + column(RPC * j))), dst + x * 512);
      });
    } else {  // (rows past the last one repeat it)
      static_for<decltype(first_c)::value, decltype(end_c)::value>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int x = decltype(x_c)::value, j = x % PT;
        dma16(src(x) + (int64_t)min(RPC * j + c_row, last_row) * kv_stride + column(RPC * j), dst + x * 512);
      });
    }
  };
  const std::integral_constant<int, 0> first;
  const std::integral_constant<int, PT> half;
  const std::integral_constant<int, PPW> all;
  auto copy_stage = [&](int i, int slot) __attribute__((always_inline)) { copy_pieces(i, slot, first, all); };
  constexpr int AHEAD = HG == 1 ? NS : NS - 1;  // stages copied before the first step
  constexpr bool HALVES = HG == 1 && NS == 1;   // one slot: K of the next stage is copied once K has been read, V once V has been
#pragma unroll
  for (int s = 0; s < AHEAD; ++s)
    if (s < n_mine) copy_stage(s, s);

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = zero16;
  float m_run = kNoMax, l_run = 0.f;
  const float c = p.scale_log2, limit = fminf(8.0f, p.ref_limit);
  const float c_move = fmaxf(c, 1e-30f);  // moves the reference off kNoMax for every score, however small the scale is

  // the Q copies have landed when at most those of the stages are outstanding
  if (AHEAD > 1 && n_mine > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD * PPW) : "memory");
  else if (n_mine > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PPW) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  wg_barrier();

  // addresses inside a tile (bytes): rows (l32, chunk 2 ks + hh), k-steps an XOR apart; transposed: four rows by four chunks, blocks of
  // 32 columns an XOR apart, rows r + 8 another one
  const unsigned row_at = (unsigned)(l32 * ROW + ((hh ^ share_swz<D>(l32)) * 16));
  unsigned tr_at;
  {
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    tr_at = (unsigned)(r0 * ROW + ((cl ^ share_swz<D>(r0)) * 16) + 8 * (j & 1));
  }
  bf16x8 qf[DK];
  {
    const unsigned base = lds_addr(q_tiles) + unit * TILE + row_at;
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      qf[ks] = lds_asm_read16<0>(base ^ (ks * 32));
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(qf[ks]));
  }

  const unsigned k_base = lds_addr(region) + row_at, v_base = lds_addr(region) + TILE + tr_at;
  int slot = 0;
  const int n_steps = HG == 1 ? n_mine : (nt + KS - 1) / KS;
  for (int i = 0; i < n_steps; ++i) {
    const int t = split + KS * i;
    constexpr int LATER = HG == 1 ? NS - 1 : NS - 2;  // stages after this one that may be outstanding
    if constexpr (HALVES) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PT) : "memory");  // (V may be outstanding)
    else if (LATER > 0 && i + 1 < n_mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LATER * PPW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (HG > 1) {
      wg_barrier();  // every wave's share of the stage has landed, and every wave is done with the stage before it
      if (i + NS - 1 < n_mine) copy_stage(i + NS - 1, slot == 0 ? NS - 1 : slot - 1);
      if (i >= n_mine) continue;
    }
    const unsigned ka = k_base + slot * (2 * TILE), va = v_base + slot * (2 * TILE);
    // ---- S^T = K Q^T: [32 keys] x [32 queries] ----
    bf16x8 kf[DK];
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      kf[ks] = lds_asm_read16<0>(ka ^ (ks * 32));
    });
    f32x16 s;
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(DK / 2) : "memory");
#pragma unroll
    for (int ks = 0; ks < DK / 2; ++ks) asm volatile("" : "+v"(kf[ks]));
#pragma unroll
    for (int ks = 0; ks < DK / 2; ++ks) s = mfma32(kf[ks], qf[ks], ks == 0 ? zero16 : s);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = DK / 2; ks < DK; ++ks) asm volatile("" : "+v"(kf[ks]));
    // the operands of O^T += V^T P^T arrive while the second half of the scores and the probabilities are computed
    s16x4 v_lo[2][DB], v_hi[2][DB];
    auto read_v = [&]() __attribute__((always_inline)) {
      static_for<0, 2 * DB>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int ks = decltype(x_c)::value / DB, db = decltype(x_c)::value % DB;
        v_lo[ks][db] = lds_asm_read_tr<ks * 16 * ROW>(va ^ (db * 64));
        v_hi[ks][db] = lds_asm_read_tr<(ks * 16 + 8) * ROW>(va ^ (db * 64 + share_swz<D>(8) * 16));
      });
    };
    if constexpr (HALVES) {
      if (i + 1 < n_mine) copy_pieces(i + 1, 0, first, half);
    } else {
      read_v();
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = DK / 2; ks < DK; ++ks) s = mfma32(kf[ks], qf[ks], s);
    if constexpr (HALVES) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 < n_mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PT) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      read_v();
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- mask: key j of the stage is visible to row r iff 32 t + j < n0 + r ----
    if (32 * t + 32 > it.n0) {
      const int lim = it.n0 + l32 - 32 * t;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + 4 * hh + (e & 3) >= lim) s[e] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
    for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(mx, s[e]), s[e + 1]);
    mx = max_halves(fmaxf(mx, s[15]));
    // (the reference only has to keep exp2 in range, so it follows the maximum when that is 2^8 past it, as in fwd_kernel)
    if (__builtin_expect(__any((mx - m_run) * c_move > limit), 0)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      m_run = m_new;
    }
    const float mc = m_run == kNoMax ? 0.f : m_run * c;  // (no key of the row seen yet: every score is -inf)
    float w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] = __builtin_amdgcn_exp2f(s[e] * c - mc);
    bf16x8 pf[2];
    pf[0] = pack8(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]);
    pf[1] = pack8(w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]);
    float ps0 = 0.f, ps1 = 0.f;
    if constexpr (D == 64) {  // (the sums are those of fwd_kernel at 64, of the pipelined kernel at 96 and 128)
      bf16x2 ones;
      ones[0] = (__bf16)1.0f; ones[1] = (__bf16)1.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[j], pf[j], 0, 1), ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[j], pf[j], 2, 3), ones, ps1, false);
        ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[j], pf[j], 4, 5), ones, ps0, false);
        ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pf[j], pf[j], 6, 7), ones, ps1, false);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        ps0 += w[e];
        ps1 += w[e + 1];
      }
    }
    l_run += ps0 + ps1;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int x = 0; x < 2 * DB; ++x) asm volatile("" : "+v"(v_lo[x / DB][x % DB]), "+v"(v_hi[x / DB][x % DB]));
    if constexpr (HG == 1) {
      if (i + NS < n_mine) {  // (every read of the slot has returned)
        if constexpr (HALVES) copy_pieces(i + 1, 0, half, all);
        else copy_stage(i + NS, slot);
      }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v_lo[ks][db], v_hi[ks][db], 0, 1, 2, 3, 4, 5, 6, 7));
        oacc[db] = mfma32(a, pf[ks], oacc[db]);
      }
    if constexpr (NS > 1) slot = slot + 1 == NS ? 0 : slot + 1;
  }

  // ---- the splits' results in LDS, then put together: the waves of a head take a share of its columns each ----
  wg_barrier();  // every wave has read its last stage (and its last copies have landed)
  if (n_mine > 0) {
    lds_f32* const out = (lds_f32*)smem + wave * (NQ * 256) + lane * 4;
#pragma unroll
    for (int x = 0; x < NQ; ++x)
      *(__attribute__((address_space(3))) f32x4*)(out + x * 256) =
          f32x4{oacc[x / 4][4 * (x % 4)], oacc[x / 4][4 * (x % 4) + 1], oacc[x / 4][4 * (x % 4) + 2], oacc[x / 4][4 * (x % 4) + 3]};
    const float l = sum_halves(l_run);
    if (hh == 0) *(__attribute__((address_space(3))) f32x2*)(ml + (wave * 32 + l32) * 2) = f32x2{m_run, l};
  }
  __syncthreads();
  constexpr int QS = NQ % KS == 0 ? 1 : KS;
  const int quarter0 = NQ % KS == 0 ? split * NQW : split, parts = min(nt, KS);
  float m = kNoMax, l = 0.f;
  for (int w = 0; w < parts; ++w) m = fmaxf(m, ml[((w * HG + unit) * 32 + l32) * 2]);
  f32x4 o[NQW];
#pragma unroll
  for (int x = 0; x < NQW; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  const lds_f32* const src = (const lds_f32*)smem + (unit * NQ + quarter0) * 256 + lane * 4;
  for (int w = 0; w < parts; ++w) {
    const lds_f32* const e = ml + ((w * HG + unit) * 32 + l32) * 2;
    const float f = __builtin_amdgcn_exp2f((e[0] - m) * c);
    l += e[1] * f;
#pragma unroll
    for (int x = 0; x < NQW; ++x) {
      if (QS > 1 && quarter0 + QS * x >= NQ) break;
      const f32x4 v = lds_load4f(src + w * (HG * NQ * 256) + x * (QS * 256));
#pragma unroll
      for (int r = 0; r < 4; ++r) o[x][r] += v[r] * f;
    }
  }
  if (l32 < it.q_rows) {
    const float inv = 1.0f / l;
    __bf16* const op = p.o + (int64_t)(it.q_row0 + l32) * q_stride + (int64_t)head * D + 4 * hh;
#pragma unroll
    for (int x = 0; x < NQW; ++x)
      if (QS == 1 || quarter0 + QS * x < NQ)
        *reinterpret_cast<bf16x4*>(op + (quarter0 + QS * x) * 8) = pack4(o[x][0] * inv, o[x][1] * inv, o[x][2] * inv, o[x][3] * inv);
    if (split == 0 && hh == 0) p.lse[(int64_t)head * p.total_q + it.q_row0 + l32] = (m * c + log2f(l)) * 0.6931471805599453f;
  }
}

// The dynamic-LDS limit of a kernel is raised once per process (thread-safe: a function-local static).
template <class K>
static hipError_t raise_smem_limit(K kernel, size_t smem) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

// (the arguments' trailing list of items is only filled, and only read, where the items have no other place)
static FwdArgs fwd_launch_args(const FwdParams& p, const FwdLists& lists) {
  FwdArgs a;
  a.p = p;
  a.num_blocks = lists.num_blocks;
  if (p.items == nullptr) std::memcpy(a.items, lists.items, (size_t)lists.num_items * sizeof(FwdItem));
  return a;
}

template <int D, bool CUT>
static hipError_t launch_fwd_items(const FwdArgs& a, size_t smem, hipStream_t stream) {
  static const hipError_t attr = raise_smem_limit(&fwd_pipe_kernel<D, CUT>, smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((fwd_pipe_kernel<D, CUT>), dim3(persistent_grid(a.num_blocks, fwd_per_cu(D))), dim3(256), smem, stream, a);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_fwd_pipe(const FwdArgs& a, const FwdLists& lists, hipStream_t stream) {
  // ring slots of a K and a V tile, then the staging tiles of the four waves (64 rows each)
  const size_t smem = (size_t)2 * (FWD_PIPE_DIST + 3) * 32 * D * 2 + (size_t)4 * 64 * D * 2;
  if constexpr (pipelined(D)) {
    if (lists.num_wholes > 0) {
      const hipError_t e = launch_fwd_items<D, true>(a, smem, stream);
      if (e != hipSuccess) return e;
      FwdMergeArgs m;
      m.p = a.p;
      if (a.p.wholes == nullptr) std::memcpy(m.wholes, lists.wholes, (size_t)lists.num_wholes * sizeof(FwdItem));
      const unsigned units = 8u * (unsigned)lists.num_wholes * (unsigned)(a.p.num_kv_heads * a.p.head_splits);
      hipLaunchKernelGGL((fwd_merge_kernel<D>), dim3(units), dim3(256), 0, stream, m);
      return hipGetLastError();
    }
  }
  return launch_fwd_items<D, false>(a, smem, stream);
}

template <int D, int HG, int KS, int NS>
static hipError_t launch_fwd_share(const FwdArgs& a, hipStream_t stream) {
  constexpr size_t smem = share_smem<D, HG, KS, NS>();
  static_assert(smem <= 160 * 1024);
  static const hipError_t attr = raise_smem_limit(&fwd_share_kernel<D, HG, KS, NS>, smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((fwd_share_kernel<D, HG, KS, NS>), dim3(a.num_blocks), dim3(HG * KS * 64), smem, stream, a);
  return hipGetLastError();
}

hipError_t launch_fwd(const FwdParams& p, int head_dim, FwdKind kind, const FwdLists& lists, hipStream_t stream) {
  const FwdArgs a = fwd_launch_args(p, lists);
  if (kind == kFwdShare) {
    const int heads = p.heads_per_wg;
    if (head_dim == 64)
      return heads == 4 ? launch_fwd_share<64, 4, 2, 3>(a, stream) : heads == 2 ? launch_fwd_share<64, 2, 4, 2>(a, stream) : launch_fwd_share<64, 1, 8, 2>(a, stream);
    if (head_dim == 96)
      return heads == 4 ? launch_fwd_share<96, 4, 2, 3>(a, stream) : heads == 2 ? launch_fwd_share<96, 2, 4, 2>(a, stream) : launch_fwd_share<96, 1, 8, 1>(a, stream);
    return heads == 4 ? launch_fwd_share<128, 4, 2, 3>(a, stream) : heads == 2 ? launch_fwd_share<128, 2, 4, 2>(a, stream) : launch_fwd_share<128, 1, 8, 1>(a, stream);
  }
  if (kind == kFwdTall) {
    const size_t smem = (size_t)8 * 32 * 256 * 2 + 16;  // four slots of K and of V, two words
    static const hipError_t attr = raise_smem_limit(&fwd_tall_kernel, smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(fwd_tall_kernel, dim3(persistent_grid(a.num_blocks)), dim3(256), smem, stream, a);
    return hipGetLastError();
  }
  if (head_dim == 256) {
    const size_t smem = (size_t)10 * 32 * 256 * 2;  // four slots of K, five of V, and one tile more for the staging
    static const hipError_t attr = raise_smem_limit(&fwd_wide_kernel, smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(fwd_wide_kernel, dim3(persistent_grid(a.num_blocks)), dim3(256), smem, stream, a);
    return hipGetLastError();
  }
  if (kind != kFwdPipe) {
    const size_t smem = (size_t)4 * 64 * 64 * 2;  // two K tiles, two V tiles
    static const hipError_t attr = raise_smem_limit(&fwd_kernel, smem);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(fwd_kernel, dim3(a.num_blocks), dim3(256), smem, stream, a);
    return hipGetLastError();
  }
  return head_dim == 64 ? launch_fwd_pipe<64>(a, lists, stream)
         : head_dim == 96 ? launch_fwd_pipe<96>(a, lists, stream)
                          : launch_fwd_pipe<128>(a, lists, stream);
}

}  // namespace chunk_attn

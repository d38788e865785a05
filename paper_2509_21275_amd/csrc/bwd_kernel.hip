// Chunk attention backward for gfx950 (gradients of L = sum(O .* dO) under the chunk mask of the
// paper's section 3.1; key/value gradients include the context rows, section 2.1 / 3.2.2).
//
// Two reductions are needed -- dQ sums over keys, dK/dV sum over queries -- and a workgroup can keep
// only one of them in registers.  Float atomics for the other one are far too slow on this chip at the
// rate an attention backward produces them, so each reduction gets blocks of its own kind and every output
// element is written exactly once, or put together from the partial results of a walk that was cut, in a fixed order (the result is
// also bit-reproducible).  Both kinds of block share a launch (bwd_pipe_kernel, bwd_short_kernel) except where they do not end sooner so (head_dim 64 and 256, bwd_layout):
//
//   bwd_pre   D_i = <dO_i, O_i> and LSE_i log2(e) per (head, row), stored in arrays padded to 64-row
//             tiles per segment (+inf / 0 in the padding, so padded rows yield P = 0);
//   bwd_dq    query-stationary, like the forward: S^T = K Q^T and dP^T = V dO^T per 32-key tile,
//             dS^T = P^T (dP^T - D), dQ^T += K^T dS^T with dS^T fed back from the accumulator registers;
//   bwd_dkv   key-stationary: one workgroup per 64 to 256 keys of one key/value head (dkv_block_keys), walking the query heads of
//             the group and the 32-row query tiles that see those keys: S = Q K^T, P, dV^T += dO^T P  and  dP = dO V^T, dS,
//             dK^T += Q^T dS, in two wave roles (dkv_pipe_blocks) or all in each wave (the others).
// P is recomputed from the saved log-sum-exp in both.  All operands reach LDS by global->LDS copies.
#include <cstring>
#include <cstdlib>
#include <type_traits>

#include "kernels.hpp"
#include "tiles.hpp"

namespace chunk_attn {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

#ifndef DKV_PIPE_DIST
#define DKV_PIPE_DIST 3
#endif
#ifndef DQ_PIPE_DIST
#define DQ_PIPE_DIST 3  // stages the pipelined dQ kernel copies ahead
#endif

// ------------------------------------------------------------------------------------------------
// bwd_pre: one workgroup per (64-row query tile, head); D / 8 threads per row (head_dim 96: 16, of which 12 read), one
// 16-byte chunk of O and of dO each, so that a wave reads whole rows (the kernel is bound by memory: it reads O and dO once).
// Its arguments may carry the call's schedule, which the first workgroup then copies into the workspace for the kernels behind it.
// ------------------------------------------------------------------------------------------------
struct BwdPreArgs {
  const __bf16 *o, *d_o;
  const float* lse;
  const TileJob* jobs;  // null: in the blob
  float *lse2p, *dsp;
  int64_t total_q_tiles;
  int32_t total_q, num_q_heads;
  u32x4* blob_dst;
  int32_t blob_n16, jobs_off;  // the blob's size in units of 16 bytes (0: it is not here) and the place of the jobs in it
  u32x4 blob[kInlineBlob / 16];
};
template <int D>
__global__ __launch_bounds__(256) void bwd_pre_kernel(BwdPreArgs) {
  typedef const __attribute__((address_space(4))) BwdPreArgs* args_ptr;
  typedef const __attribute__((address_space(4))) TileJob* job_ptr;
  const args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const __bf16* const o = args->o;
  const __bf16* const d_o = args->d_o;
  const float* const lse = args->lse;
  float* const lse2p = args->lse2p;
  float* const dsp = args->dsp;
  const int64_t total_q_tiles = args->total_q_tiles;
  const int total_q = args->total_q, num_q_heads = args->num_q_heads;
  if (blockIdx.x == 0 && (int)threadIdx.x < args->blob_n16) args->blob_dst[threadIdx.x] = args->blob[threadIdx.x];
  constexpr int TPR = D == 96 ? 16 : D / 8;  // threads per row
  constexpr int RPP = 256 / TPR;     // rows per pass
  const int head = blockIdx.x % num_q_heads;
  const job_ptr jobs = args->jobs != nullptr ? (job_ptr)(uintptr_t)args->jobs
                                             : (job_ptr)((const __attribute__((address_space(4))) char*)args->blob + args->jobs_off);
  TileJob job;
  __builtin_memcpy(&job, (const void*)(jobs + blockIdx.x / num_q_heads), sizeof(job));
  const int part = threadIdx.x % TPR;
#pragma unroll
  for (int pass = 0; pass < 64 / RPP; ++pass) {
    const int r = pass * RPP + threadIdx.x / TPR;
    const bool valid = r < job.valid_rows;
    float acc = 0.f;
    if (valid && part < D / 8) {
      const int64_t base = ((int64_t)(job.src_row0 + r) * num_q_heads + head) * D + part * 8;
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(o + base);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(d_o + base);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc += (float)a[i] * (float)b[i];
    }
#pragma unroll
    for (int w = 1; w < TPR; w *= 2) acc += __shfl_xor(acc, w);
    if (part == 0) {
      const int64_t slot = ((int64_t)head * total_q_tiles + job.image) * 64 + r;
      dsp[slot] = valid ? -acc : 0.f;  // stored negated: the kernels add it (or start an accumulation from it)
      lse2p[slot] = valid ? lse[(int64_t)head * total_q + job.src_row0 + r] * kLog2e : INFINITY;
    }
  }
}

// zero `n16` 16-byte units starting at p
__global__ __launch_bounds__(256) void zero_fill_kernel(u32x4* __restrict__ p, int64_t n16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) p[i] = u32x4{0u, 0u, 0u, 0u};
}

// ------------------------------------------------------------------------------------------------
// bwd_dq
// ------------------------------------------------------------------------------------------------
struct DqParams {
  const __bf16 *q, *k, *v, *d_o;
  const float* lse2p;    // [Hq][total_q_tiles * 64]
  const float* dsp;
  __bf16* dq;
  const DqItem* items;
  int64_t total_q_tiles;
  int32_t num_q_heads, num_kv_heads, group, heads_per_wg, head_splits;
  float scale, scale_log2;
  float* parts;          // partial results of pieces (pipelined kernel), kPartRowFloats per (slot, inner index)
  int32_t* taken;        // 8 block-queue counters of the pipelined kernel (zero before the launch)
  int32_t num_blocks;
  unsigned long long* clock_log;  // null, or where the pipelined kernel's workgroups log their clocks
};

// (head_dim 64 unless its walks are long, and 256 with short walks.)  K^T is read transposed out of the K tile; with an image of K made by a
// launch before, as this kernel had it, the backward of four sequences of 1024, 32/8 heads, took 144 us instead of 141, of
// 64 of 256 220 instead of 211, and at head_dim 256 the packed 64K chunk 41.2 ms (forward included) instead of 40.2.
// With one wave per SIMD a tile's chain of products, exponentials and products is what a step takes, and the transposed
// reads (twice as many instructions as an image takes) lengthen it unless they are issued behind the last products of S^T and
// dP^T and the second half of dS is made behind the first half's products.  Backward with an image / with the reads in one
// burst behind the products / as they are now: head_dim 64, 128 queries on 16384 keys, 8/8 heads, 314 / 334 / 293 us, 512
// queries, 32/8 heads, 476 / 484 / 450; head_dim 256, 64 queries on 8192 keys, 8/8 heads, 413 / 427 / 388.
template <int D, int WAVES>
__device__ __forceinline__ void dq_block(const DqParams& p, int blk) {
  constexpr int NTH = WAVES * 64;  // threads
  constexpr int BN = 32;       // key rows per LDS tile
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dQ^T
  constexpr int KT = BN * D;   // elements per tile

  constexpr int NS = 3;        // LDS stages: tiles are fetched NS - 1 iterations ahead

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __bf16* Ks = reinterpret_cast<__bf16*>(smem);  // [NS][BN][D]  chunk-major; K^T is read from it, too
  __bf16* Vs = Ks + NS * KT;                     // [NS][BN][D]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  stagger_wave_priority();

  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = blk % inner_n;
  const DqItem it = p.items[blk / inner_n];
  const int kvh = inner % p.num_kv_heads, hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int wave_row0 = (wave / p.heads_per_wg) * 32;

  const int n_wg = it.n0 + it.q_rows - 1;
  const int nt_wg = (n_wg + BN - 1) / BN;
  int nt_w = 0;
  if (wave_row0 < it.q_rows) {
    const int last = min(wave_row0 + 32, it.q_rows) - 1;
    nt_w = (it.n0 + last + BN - 1) / BN;
  }

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  constexpr int NK = BN * KC / NTH;
  static_assert(NK >= 1, "every thread copies at least one chunk of each tile");
  unsigned k_src[NK];
  int k_row[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int x = (i * WAVES + wave) * 64 + lane;
    k_row[i] = (x & 31) ^ (((x >> 5) & 3) << 2);
    k_src[i] = (unsigned)(k_row[i] * (int)kv_stride + (x >> 5) * 8);
  }
  // One tile is copied by NK pieces per lane (a K and a V chunk each), so that the copies can be issued between MFMAs
  // instead of in one burst.
  auto dma_piece = [&](int t, int buf, int i) {
    const int64_t toff = (int64_t)(BN * t) * kv_stride;  // wave-uniform
    const int last_row = n_wg - 1 - BN * t;
    unsigned off = k_src[i];
    if (last_row < BN - 1) off -= (unsigned)((k_row[i] - min(k_row[i], last_row)) * (int)kv_stride);
    dma16(Kg + toff + off, Ks + buf * KT + (i * WAVES + wave) * 512);
    dma16(Vg + toff + off, Vs + buf * KT + (i * WAVES + wave) * 512);
  };
  auto dma_tile = [&](int t, int buf) {
#pragma unroll
    for (int i = 0; i < NK; ++i) dma_piece(t, buf, i);
  };

  // Q and dO fragments (B operands): lane holds X[row = l32][16 ks + 8 hh ..+7]
  bf16x8 qf[DK], gf[DK];
  const int r_own = min(wave_row0 + l32, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
  {
    const int64_t off = (int64_t)(it.q_row0 + r_own) * q_stride + (int64_t)head * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8*>(p.q + off + 16 * ks);
      gf[ks] = *reinterpret_cast<const bf16x8*>(p.d_o + off + 16 * ks);
    }
  }
  const int64_t slot = (int64_t)head * p.total_q_tiles * 64 + it.q_slot0 + r_own;
  const float lse2 = p.lse2p[slot], dsum = p.dsp[slot];

  // prologue: the first NS - 1 tiles (issued after the register loads so that vmcnt below counts only copies)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nt_wg) dma_tile(s, s);

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16;
  const float c = p.scale_log2;

  // (addresses inside a tile as in the pipelined kernels)
  const int x_off[2] = {cm_elem(l32, hh), cm_elem(l32, 2 + hh)};
  auto k_off = [&](int ks) { return x_off[ks & 1] + (ks >> 1) * (4 * 32 * 8); };
  unsigned t_lo, t_hi;
  {
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    t_lo = lds_addr((lds_bf16*)Ks + cm_elem(r0, cl) + 4 * (j & 1));
    t_hi = lds_addr((lds_bf16*)Ks + cm_elem(r0 + 8, cl) + 4 * (j & 1));
  }

  // wait until at most `tiles_in_flight` later tiles are still being copied (each is 2 NK copies per lane)
  auto wait_tiles = [&](int tiles_in_flight) {
    constexpr int PER = 2 * NK;
    if (tiles_in_flight <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
  };
  wait_tiles(min(nt_wg, NS - 1) - 1);
  wg_barrier();

  auto tile_step = [&](int t, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    const bool prefetch = t + NS - 1 < nt_wg;
    if (t >= nt_w && prefetch) dma_tile(t + NS - 1, (buf + NS - 1) % NS);  // idle wave: still does its share of the copies

    if (t < nt_w) {
      const __bf16* Kt = Ks + buf * KT;
      const __bf16* Vt = Vs + buf * KT;
      // The loop body is laid out as stages separated by scheduling fences: each stage issues the LDS reads
      // of the next stage's operands together with the MFMAs of the current one, so the reads' latency is
      // covered by matrix work instead of stalling every MFMA on the read issued just before it.
      auto ldk = [&](int ks) { return *reinterpret_cast<const bf16x8*>(Kt + k_off(ks)); };
      auto ldv = [&](int ks) { return *reinterpret_cast<const bf16x8*>(Vt + k_off(ks)); };
      // ---- S^T = K Q^T, dP^T = V dO^T : [32 keys] x [32 queries] ----
      f32x16 s, dp;
      bf16x8 ak[2][2], av[2][2];  // [parity of the k-step pair][step in the pair]
      ak[0][0] = ldk(0); av[0][0] = ldv(0); ak[0][1] = ldk(1); av[0][1] = ldv(1);
      // operands of dQ^T += K^T dS^T (k-step m / DB, block m % DB), fetched between the last products of S^T and dP^T: a
      // quarter behind each, where the wave has nothing else to issue
      s16x4 a_lo[2 * DB], a_hi[2 * DB];
      auto read_kt = [&](auto quarter_c) __attribute__((always_inline)) {
        constexpr int quarter = decltype(quarter_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        static_for<quarter * (DB / 2), (quarter + 1) * (DB / 2)>([&](auto m_c) __attribute__((always_inline)) {
          constexpr int m = decltype(m_c)::value;
          constexpr int off = (buf * KT + (m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2;
          a_lo[m] = lds_asm_read_tr<off>(t_lo);
          a_hi[m] = lds_asm_read_tr<off>(t_hi);
        });
        __builtin_amdgcn_sched_barrier(0);
      };
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, DK / 2>([&](auto g_c) __attribute__((always_inline)) {
        constexpr int g = decltype(g_c)::value, cur = g & 1, nxt = cur ^ 1;
        constexpr bool last = g == DK / 2 - 1;
        if constexpr (!last) {
          ak[nxt][0] = ldk(2 * g + 2); av[nxt][0] = ldv(2 * g + 2);
          ak[nxt][1] = ldk(2 * g + 3); av[nxt][1] = ldv(2 * g + 3);
        }
        s = mfma32(ak[cur][0], qf[2 * g], g == 0 ? zero16 : s);
        if constexpr (last) read_kt(std::integral_constant<int, 0>{});
        dp = mfma32(av[cur][0], gf[2 * g], g == 0 ? zero16 : dp);
        if constexpr (last) read_kt(std::integral_constant<int, 1>{});
        if (g < NK && prefetch) dma_piece(t + NS - 1, (buf + NS - 1) % NS, g);
        s = mfma32(ak[cur][1], qf[2 * g + 1], s);
        if constexpr (last) read_kt(std::integral_constant<int, 2>{});
        dp = mfma32(av[cur][1], gf[2 * g + 1], dp);
        if constexpr (last) read_kt(std::integral_constant<int, 3>{});
        __builtin_amdgcn_sched_barrier(0);
      });
      // ---- P = exp2(S c - LSE), dS = P (dP - D); masked keys give P = 0 ----
      float pe[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) pe[i] = __builtin_amdgcn_exp2f(s[i] * c - lse2);
      if (BN * t + BN > it.n0 + wave_row0) {
        const int lim = it.n0 + wave_row0 + l32 - BN * t;  // visible iff local key index < lim
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int j = 8 * (i >> 2) + 4 * hh + (i & 3);
          if (j >= lim) pe[i] = 0.f;
        }
      }
      // ---- dQ^T += K^T dS^T : [D] x [32 queries], contraction over the 32 keys, the second 16 keys' dS while the first 16's
      // products run ----
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float ds[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) ds[i] = pe[8 * h + i] * (dp[8 * h + i] + dsum);
        const bf16x8 f = pack8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const int m = h * DB + db;
          asm volatile("" : "+v"(a_lo[m]), "+v"(a_hi[m]));  // (after the wait, in this order)
          const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a_lo[m], a_hi[m], 0, 1, 2, 3, 4, 5, 6, 7));
          dq[db] = mfma32(a, f, dq[db]);
        }
      }
    }
    // tile t + 1 must have landed; tiles t + 2 .. may still be in flight
    wait_tiles(min(nt_wg - 1, t + NS - 1) - (t + 1));
    wg_barrier();
  };

  for (int t = 0; t < nt_wg; t += NS) {
    tile_step(t, std::integral_constant<int, 0>{});
    if (t + 1 < nt_wg) tile_step(t + 1, std::integral_constant<int, 1>{});
    if (t + 2 < nt_wg) tile_step(t + 2, std::integral_constant<int, 2>{});
  }

  // ---- epilogue: dQ = scale * dQ^T ----
  {
    const int r = wave_row0 + l32;
    if (r < it.q_rows) {
      __bf16* op = p.dq + (int64_t)(it.q_row0 + r) * q_stride + (int64_t)head * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const bf16x4 v = pack4(dq[db][4 * g] * p.scale, dq[db][4 * g + 1] * p.scale, dq[db][4 * g + 2] * p.scale,
                                 dq[db][4 * g + 3] * p.scale);
          *reinterpret_cast<bf16x4*>(op + 32 * db + 8 * g + 4 * hh) = v;
        }
    }
  }
}

template <int D, int WAVES>
__global__ __launch_bounds__(WAVES * 64, D > 128 ? 1 : 8 / WAVES) void bwd_dq_kernel(DqParams p) {
  dq_block<D, WAVES>(p, blockIdx.x);
}

// ------------------------------------------------------------------------------------------------
// bwd_dkv
//
// One workgroup = 128 consecutive keys of one segment and one key/value head, 8 waves.  The four
// contractions of a (32-query, 32-key) block are split between two waves that share the block's keys:
//   wave A (waves 0..3): S = Q K^T, P = exp2(S c - LSE), dV^T += dO^T P;  hands P (bf16) to wave B through LDS
//   wave B (waves 4..7): dP = dO V^T, dS = P (dP - D),   dK^T += Q^T dS;  runs one step behind wave A
// so each wave keeps one fragment set (K or V) and one accumulator (dV^T or dK^T) and the whole kernel
// fits 256 registers per lane: two waves per SIMD, whose matrix and vector phases overlap.
// The workgroup walks the group's query heads and, per head, the 32-row query tiles that see its keys.
//
// Only the rows of Q and dO are streamed (global->LDS copies into 4-slot rings, two steps ahead); each tile
// serves both contractions that need it: as rows (16-byte reads, operand of Q K^T / dO V^T) and transposed
// (ds_read_b64_tr_b16, operand of Q^T dS / dO^T P).  A tile is stored chunk-major: 16-byte chunk c of row r
// sits at slot c * 32 + (r ^ 4 (c & 3)).  With that layout both kinds of read are bank-conflict free and
// their addresses are one per-lane base plus constants.
// ------------------------------------------------------------------------------------------------
struct DkvParams {
  const __bf16 *q, *k, *v, *d_o;
  const float* lse2p;   // [Hq][total_q_tiles * 64]
  const float* dsp;
  __bf16 *dk, *dv;
  const DkvItem* items;
  int64_t total_q_tiles;
  int32_t num_q_heads, num_kv_heads, group;
  float scale, scale_log2;
  int32_t accumulate;
  int32_t out_f32;      // dk / dv point to fp32 arrays of the same shape
  int32_t* taken;       // 8 block-queue counters of the pipelined kernel (zero before the launch)
  int32_t* ended;       // per queue, the blocks that have ended (zero before the launch)
  int32_t side_by_side; // blocks of a queue that run at the same time, of which long equal walks start together (dkv_pipe_blocks); 0: none do
  float* parts;         // partial results of pieces (dkv_pipe_blocks), kPartRowFloats per (slot, key/value head)
  unsigned long long* clock_log;  // null, or where the pipelined kernel's workgroups log their clocks
  int32_t num_blocks;
};

// Four consecutive elements of a dK / dV row: stored, or added to what is there, as bf16 or as fp32.
__device__ __forceinline__ void dkv_store4(const DkvParams& p, __bf16* out, int64_t elem, float v0, float v1, float v2,
                                           float v3) {
  if (p.out_f32) {
    f32x4* op = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + elem);
    if (p.accumulate) {
      const f32x4 old = *op;
      v0 += old[0]; v1 += old[1]; v2 += old[2]; v3 += old[3];
    }
    const f32x4 nv = {v0, v1, v2, v3};
    *op = nv;
  } else {
    bf16x4* op = reinterpret_cast<bf16x4*>(out + elem);
    if (p.accumulate) {
      const bf16x4 old = *op;
      v0 += (float)old[0]; v1 += (float)old[1]; v2 += (float)old[2]; v3 += (float)old[3];
    }
    *op = pack4(v0, v1, v2, v3);
  }
}


template <int D, int KB, bool CUT>  // KB: 32-key blocks per workgroup (2 KB waves); CUT: some items are pieces
__device__ __forceinline__ void dkv_block(const DkvParams& p, int blk) {
  constexpr int NW = 2 * KB;   // waves
  constexpr int NTH = NW * 64; // threads
  constexpr int BM = 32;       // query rows per step
  constexpr int KC = D / 8;    // 16-byte chunks per operand row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dK^T / dV^T
  constexpr int QT = BM * D;   // elements per operand tile
  constexpr int NS = 4;        // ring slots
  constexpr int PT = KB * 64 * 16;     // elements of one P hand-over slot: KB key blocks x 64 lanes x 16 values
  constexpr int CH = BM * KC;          // 16-byte chunks per operand tile
  constexpr int PER = 2 * CH / NTH;    // global->LDS copies per thread and stage
  constexpr int NP = CH / 64;          // 64-slot pieces per tile
  constexpr int RV = 64;               // floats per slot of the LSE / D rows (32 used; a whole wave copies them)
  static_assert(PER >= 1 && 2 * NP % NW == 0, "the pieces of the two tiles divide evenly among the waves");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int Q_OFF = 0;                 // [NS][QT]  Q rows of stage n in slot n % NS   (wave A: step n, wave B: step n + 1)
  constexpr int G_OFF = Q_OFF + NS * QT;   // [NS][QT]  dO rows                            (both waves: step n)
  constexpr int P_OFF = G_OFF + NS * QT;   // [2][PT]   P hand-over
  lds_f32* const lse_s = (lds_f32*)(L + P_OFF + 2 * PT);  // [NS][RV]  slot n % NS        (wave A, step n)
  lds_f32* const dsum_s = lse_s + NS * RV;                // [NS][RV]  slot n % NS        (wave B, step n + 1)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = wave / KB, kb = wave % KB;
  const int l32 = lane & 31, hh = lane >> 5;

  const int kvh = blk % p.num_kv_heads;
  const DkvItem it = p.items[blk / p.num_kv_heads];
  const int G = p.group;
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const float c = p.scale_log2;

  // this wave's K (wave A) or V (wave B) fragments, B operands: lane holds X[key = 32 kb + l32][16 ks + 8 hh ..+7]
  bf16x8 bfrag[DK];
  {
    const __bf16* src = role ? p.v : p.k;
    const int64_t grow = it.kv_row0 + min(32 * kb + l32, it.kv_rows - 1);
    const int64_t off = grow * kv_stride + (int64_t)kvh * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) bfrag[ks] = *reinterpret_cast<const bf16x8*>(src + off + 16 * ks);
  }

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 acc[DB];  // dV^T (wave A) or dK^T (wave B): [D] x [32 keys of this wave]
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = zero16;

  const int nqt = it.n_qt - it.qt_first;
  const int n_iter = nqt * G;  // stages: (head in group, query tile), head-major

  // ---- staging: a copy instruction of a wave fills 64 consecutive slots of a tile = two chunk columns of 32 rows;
  // the lane fetches the chunk that belongs in its slot.  The 2 NP pieces of a stage (NP of Q, then NP of dO) are
  // dealt to the waves round robin.  Wave 0 also copies the stage's LSE rows, wave 1 its D rows. ----
  int s_off[PER];  // element offset of the lane's chunk inside its row ...
  int s_row[PER];  // ... and the row, per piece
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int x = ((i * NW + wave) % NP) * 64 + lane;
    s_off[i] = (x >> 5) * 8;
    s_row[i] = (x & 31) ^ (((x >> 5) & 3) << 2);
  }
  const float* row_values = (wave == 0 ? p.lse2p : p.dsp) + lane;
  asm volatile("" : "+v"(row_values));  // (kept as it is: put together anew it costs every stage five scalar instructions)
  int d_qt = it.qt_first, d_hg = 0;  // (query tile, head in group) of the next stage to copy
  auto dma_stage = [&](auto slot_c) {
    constexpr int sl = decltype(slot_c)::value;
    const int head = kvh * G + d_hg;
    const int last_row = it.q_len - 1 - d_qt * BM;  // >= 0; rows past it repeat it (their P is 0)
    const int64_t roff = (int64_t)(it.q_row_seg + d_qt * BM) * q_stride + (int64_t)head * D;
    const int64_t slot = ((int64_t)head * p.total_q_tiles + it.q_tile0) * 64 + d_qt * BM;
    if (wave < 2) dma4(row_values + slot, (wave == 0 ? lse_s : dsum_s) + sl * RV);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int piece = i * NW + wave;  // wave-uniform: < NP: Q, else dO
      const unsigned row_off = (unsigned)(min(s_row[i], last_row) * (int)q_stride + s_off[i]);
      if (piece < NP) dma16(p.q + roff + row_off, L + Q_OFF + sl * QT + piece * 512);
      else dma16(p.d_o + roff + row_off, L + G_OFF + sl * QT + (piece - NP) * 512);
    }
    if (++d_qt == it.n_qt) { d_qt = it.qt_first; ++d_hg; }
  };

  // ---- per-lane operand addresses (elements) inside a tile ----
  // rows: A operand of the first contraction, X[row = l32][chunk 2 ks + hh]; k-steps of equal parity are a constant apart
  int x_off[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) x_off[par] = cm_elem(l32, 2 * par + hh);
  // transposed: A operand of the second contraction, X^T[32 db + l32][k-slots of 16 ks2 ..] in accumulator order.
  // Lane j of a 16-lane group addresses the 8 bytes (row k0 + j / 4, elements 16 grp + 4 (j % 4) ..+3); the low and
  // the high half of the operand come from rows 8 apart.  Blocks db and k-steps ks2 are a constant apart.
  int t_off[2];
  {
    const int j = lane & 15, grp = (lane >> 4) & 1;
    const int cl = 2 * grp + ((j & 3) >> 1);  // chunk (mod 4) of the lane's 8 bytes
    const int r0 = 4 * hh + (j >> 2);
#pragma unroll
    for (int half = 0; half < 2; ++half) t_off[half] = cm_elem(r0 + 8 * half, cl) + 4 * (j & 1);
  }
  auto load_rows = [&](const lds_bf16* tile, bf16x8 (&a)[DK]) {
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) a[ks] = lds_load8(tile + x_off[ks & 1] + (ks >> 1) * (4 * 32 * 8));
  };
  auto load_transposed = [&](const lds_bf16* tile, bf16x8 (&t)[2][DB]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const s16x4 lo = lds_read_tr(tile + t_off[0] + ks * (16 * 8) + db * (4 * 32 * 8));
        const s16x4 hi = lds_read_tr(tile + t_off[1] + ks * (16 * 8) + db * (4 * 32 * 8));
        t[ks][db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
  };

  // key index of this lane's column relative to the context: query i of the segment sees it iff i >= jrel
  const int jrel = it.j0 + 32 * kb + l32 - it.ctx;
  const int jrel_lo = it.j0 + 32 * kb - it.ctx;  // of the wave's first key

  // prologue: stages 0 and 1 (after the fragment loads, so that the waits below count only copies)
  dma_stage(std::integral_constant<int, 0>{});
  if (n_iter > 1) {
    dma_stage(std::integral_constant<int, 1>{});
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  wg_barrier();

  int c_qt = it.qt_first, p_qt = it.qt_first;  // query tile of stage g and of stage g - 1
  // end of step g: stage g + 1 must have landed and wave A's P must be visible; the copies issued in this
  // step (stage g + 2) may still be in flight
  auto end_step = [&](bool more) {
    p_qt = c_qt;
    if (++c_qt == it.n_qt) c_qt = it.qt_first;
    if (more) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(PER) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    // lgkmcnt(0) once more, for the compiler to see: as it does not know which reads of a stage that a wave skips are still out, it
    // otherwise waits for all of a step's reads before the first is used (this kernel alone, 6415 queries on 6424 keys, 64/8 heads, d = 64:
    // 1087 us, now 1034; without row_values, whose address was put together anew for every stage, between the two)
    __builtin_amdgcn_s_waitcnt(0xc07f);
    wg_barrier();
  };

  // Wave A defers the second contraction of a block to the beginning of the next step: its operands are in
  // registers by then, so its step opens with eight MFMAs that need nothing from LDS and cover the latency of
  // the operand reads issued at the top of the step.  (The same order measured slower for wave B, which opens
  // with the vector work of the previous block instead.)
  if (role == 0) {
    // ================= wave A: S = Q K^T, P, dV^T += dO^T P =================
    const lds_f32* const rv = lse_s + 4 * hh;
    lds_bf16* const pex = L + P_OFF + kb * 1024 + lane * 8;
    bf16x8 tp[2][DB], fp[2];  // dO^T operands and P of the block whose dV^T product is pending
    bool pend = false;
    auto second = [&]() {
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] = mfma32(tp[0][db], fp[0], acc[db]);
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] = mfma32(tp[1][db], fp[1], acc[db]);
    };

    auto step = [&](int g, auto u_c) {
      constexpr int u = decltype(u_c)::value;
      const bool more = g + 2 < n_iter;
      const int i0 = c_qt * BM;  // first query (inside the segment) of block g
      const bool vis = g < n_iter && i0 + BM - 1 >= jrel_lo;  // else: no block, or nothing of it visible to this wave
      bf16x8 a[DK], t[2][DB];
      f32x4 r4[4];  // LSE of rows 8 g4 + 4 hh + 0..3
      if (vis) {
        load_rows(L + Q_OFF + u * QT, a);
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) r4[g4] = lds_load4f(rv + u * RV + 8 * g4);
        load_transposed(L + G_OFF + u * QT, t);
      }
      if (pend) second();
      pend = vis;
      if (vis) {
        f32x16 s;
#pragma unroll
        for (int ks = 0; ks < DK; ++ks) s = mfma32(a[ks], bfrag[ks], ks == 0 ? zero16 : s);
        __builtin_amdgcn_sched_barrier(0);
        if (more) dma_stage(std::integral_constant<int, (u + 2) % NS>{});
        __builtin_amdgcn_sched_barrier(0);
        // P = exp2(S c - LSE); entries a query does not see give P = 0
        float w[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = __builtin_amdgcn_exp2f(s[i] * c - r4[i >> 2][i & 3]);
        if (i0 < jrel_lo + 31) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int qi = i0 + 8 * (i >> 2) + 4 * hh + (i & 3);
            if (qi < jrel) w[i] = 0.f;
          }
        }
        fp[0] = pack8(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]);
        fp[1] = pack8(w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]);
        lds_store8(pex + (u & 1) * PT, fp[0]);
        lds_store8(pex + (u & 1) * PT + 512, fp[1]);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int db = 0; db < DB; ++db) tp[ks][db] = t[ks][db];
      } else if (more) {
        dma_stage(std::integral_constant<int, (u + 2) % NS>{});
      }
      end_step(more);
    };
    for (int g = 0; g <= n_iter; g += NS) {
      step(g, std::integral_constant<int, 0>{});
      if (g + 1 <= n_iter) step(g + 1, std::integral_constant<int, 1>{});
      if (g + 2 <= n_iter) step(g + 2, std::integral_constant<int, 2>{});
      if (g + 3 <= n_iter) step(g + 3, std::integral_constant<int, 3>{});
    }
    if (pend) second();
  } else {
    // ================= wave B: dP = dO V^T, dS = P (dP - D), dK^T += Q^T dS =================
    // In step g it first finishes block g - 1 (vector work with wave A's P, then dK^T) and then starts block g
    // (dP): right after the barrier one wave of each SIMD begins with matrix work and the other with vector work.
    const lds_f32* const rv = dsum_s + 4 * hh;
    const lds_bf16* const pex = L + P_OFF + kb * 1024 + lane * 8;
    f32x16 dp = zero16;  // dP of the block whose dS is formed in the next step

    auto step = [&](int g, auto u_c) {
      constexpr int u = decltype(u_c)::value;
      constexpr int up = (u + NS - 1) % NS;  // slot of stage g - 1
      const bool more = g + 2 < n_iter;
      const bool cur_vis = g < n_iter && (c_qt * BM + BM - 1 >= jrel_lo);
      const bool prev_vis = g >= 1 && (p_qt * BM + BM - 1 >= jrel_lo);
      bf16x8 a[DK];
      if (cur_vis) load_rows(L + G_OFF + u * QT, a);
      if (prev_vis) {
        // ---- dS = P (dP - D) with wave A's P of block g - 1, then dK^T += Q^T dS ----
        const bf16x8 p0 = lds_load8(pex + ((u & 1) ^ 1) * PT);
        const bf16x8 p1 = lds_load8(pex + ((u & 1) ^ 1) * PT + 512);
        f32x4 r4[4];  // D of rows 8 g4 + 4 hh + 0..3
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) r4[g4] = lds_load4f(rv + up * RV + 8 * g4);
        bf16x8 t[2][DB];  // Q^T operands
        load_transposed(L + Q_OFF + up * QT, t);
        float w[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          w[i] = (float)p0[i] * (dp[i] + r4[i >> 2][i & 3]);
          w[8 + i] = (float)p1[i] * (dp[8 + i] + r4[2 + (i >> 2)][i & 3]);
        }
        const bf16x8 f0 = pack8(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]);
        const bf16x8 f1 = pack8(w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]);
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = mfma32(t[0][db], f0, acc[db]);
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = mfma32(t[1][db], f1, acc[db]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (more) dma_stage(std::integral_constant<int, (u + 2) % NS>{});
      __builtin_amdgcn_sched_barrier(0);
      if (cur_vis) {
#pragma unroll
        for (int ks = 0; ks < DK; ++ks) dp = mfma32(a[ks], bfrag[ks], ks == 0 ? zero16 : dp);
      }
      end_step(more);
    };
    for (int g = 0; g <= n_iter; g += NS) {
      step(g, std::integral_constant<int, 0>{});
      if (g + 1 <= n_iter) step(g + 1, std::integral_constant<int, 1>{});
      if (g + 2 <= n_iter) step(g + 2, std::integral_constant<int, 2>{});
      if (g + 3 <= n_iter) step(g + 3, std::integral_constant<int, 3>{});
    }
  }

  // ---- epilogue: dV = dV^T (wave A), dK = scale * dK^T (wave B), written (or added) as bf16 ----
  if (CUT && it.part >= 0) {  // a piece: the accumulators as they are, put together by bwd_merge_kernel
    float* const out = p.parts + ((int64_t)it.part * p.num_kv_heads + kvh) * kPartRowFloats + wave * part_unit_floats(D) + lane * 4;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(out + (db * 4 + g) * 256) = f32x4{acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]};
  } else {
    const int kr = 32 * kb + l32;
    if (kr < it.kv_rows) {
      const int64_t off = ((int64_t)it.kv_row0 + kr) * kv_stride + (int64_t)kvh * D;
      __bf16* const out = role ? p.dk : p.dv;
      const float f = role ? p.scale : 1.0f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          dkv_store4(p, out, off + 32 * db + 8 * g + 4 * hh, acc[db][4 * g] * f, acc[db][4 * g + 1] * f,
                     acc[db][4 * g + 2] * f, acc[db][4 * g + 3] * f);
        }
    }
  }
}

template <int D, int KB, bool CUT>
__global__ __launch_bounds__(KB * 128, D > 128 ? 1 : 4 / KB) void bwd_dkv_kernel(DkvParams p) {
  dkv_block<D, KB, CUT>(p, blockIdx.x);
}

// LDS instructions of one step of dkv_pipe_blocks in program order, per wave role, and the waits that follow from
// it.  Mini-step m issues the read of fragment m + 4 (two instructions for a transposed fragment: the first NT of a step;
// fragments past the end are the next step's first ones), then E0(m) instructions after its first MFMA and E1(m) after
// its second: role A spreads its four hand-over stores and four row-value reads over mini-steps 0 .. 3 (issued in one go
// they keep the matrix pipe waiting), role B reads the hand-over in mini-step 0 and its row values in mini-step 1.
// LDS operations of a wave complete in order, so "fragment m has arrived" = "at most wait(m) LDS instructions issued
// since its read are outstanding".  The vector work starts in mini-step 4, which therefore also waits for the last of
// the hand-over / row-value instructions.
template <int ROLE, int NF, int NT>
struct DkvLdsOrder {
  static constexpr int cost(int k) { return ((k % NF + NF) % NF) < NT ? 2 : 1; }
  static constexpr int e0(int m) { return ROLE == 0 ? (m < 4 ? 1 : 0) : (m < 2 ? 4 : 0); }
  static constexpr int e1(int m) { return ROLE == 0 ? (m < 2 ? 2 : 0) : 0; }
  static constexpr int after_fragment(int m) {
    int n = m >= 4 ? e0(m - 4) + e1(m - 4) : 0;
    for (int i = m - 3; i < m; ++i) n += cost(i + 4) + (i >= 0 ? e0(i) + e1(i) : 0);
    return n;
  }
  static constexpr int after_extras() {  // instructions between the last E0 / E1 instruction and mini-step 4
    int n = 0;
    for (int i = 3; i >= 0; --i) {
      if (e0(i) + e1(i) > 0) return n;  // nothing of mini-step i follows its last extra instruction
      n += cost(i + 4);
    }
    return n;
  }
  static constexpr int wait(int m) {
    const int a = after_fragment(m);
    return m == 4 && after_extras() < a ? after_extras() : a;
  }
};
// (pins: the counts worked out by hand for head_dim 128, where a step has 16 fragments of which the first 8 are transposed)
static_assert(DkvLdsOrder<1, 16, 8>::wait(0) == 6 && DkvLdsOrder<1, 16, 8>::wait(1) == 10 && DkvLdsOrder<1, 16, 8>::wait(2) == 14 &&
              DkvLdsOrder<1, 16, 8>::wait(3) == 14 && DkvLdsOrder<1, 16, 8>::wait(4) == 4 && DkvLdsOrder<1, 16, 8>::wait(6) == 4 &&
              DkvLdsOrder<1, 16, 8>::wait(7) == 3 && DkvLdsOrder<1, 16, 8>::wait(12) == 3 && DkvLdsOrder<1, 16, 8>::wait(13) == 4 &&
              DkvLdsOrder<1, 16, 8>::wait(14) == 5 && DkvLdsOrder<1, 16, 8>::wait(15) == 6, "role B");
static_assert(DkvLdsOrder<0, 16, 8>::wait(0) == 6 && DkvLdsOrder<0, 16, 8>::wait(1) == 9 && DkvLdsOrder<0, 16, 8>::wait(2) == 12 &&
              DkvLdsOrder<0, 16, 8>::wait(3) == 13 && DkvLdsOrder<0, 16, 8>::wait(4) == 0 && DkvLdsOrder<0, 16, 8>::wait(6) == 6 &&
              DkvLdsOrder<0, 16, 8>::wait(7) == 4 && DkvLdsOrder<0, 16, 8>::wait(8) == 3 && DkvLdsOrder<0, 16, 8>::wait(15) == 6, "role A");

// ------------------------------------------------------------------------------------------------
// dkv_pipe_blocks (head_dim 128 and 96): the dK/dV blocks of bwd_pipe_kernel
//
// Same work split as bwd_dkv_kernel, laid out for one wave per SIMD: a workgroup of 4 waves covers 128
// keys; each wave owns 64 keys (two 32-key blocks), waves 0, 1 in role A (S, P, dV^T), waves 2, 3 in role B
// (dP, dS, dK^T).  Every operand fragment read from LDS feeds two MFMAs (the wave's two key blocks), and
// with nobody else on the SIMD the wave overlaps its own matrix and vector work by software pipelining:
// in step g it runs
//     role A:  S(g) = Q K^T           P(g-1) = exp2(S(g-1) c - LSE)       dV^T += dO^T P(g-2)
//     role B:  dP(g-2) = dO V^T       dS(g-3) = P(g-3) (dP(g-3) - D)      dK^T += Q^T dS(g-4)
// (stage n = the n-th (head, 32-row query tile) of the workgroup's walk).  The three pieces of a step are
// independent of each other.  A wave issues at most one instruction every four cycles and an MFMA holds the
// matrix pipe for 32, so the step is laid out instruction by instruction: 16 (head_dim 96: 12) mini-steps of one operand
// fragment and the two MFMAs it feeds, each MFMA followed by its share of everything else (the vector work
// of one score, an LDS read, a copy), so that the next MFMA finds the pipe just free.  Fragments are fetched
// four mini-steps ahead (the first four of a step before the barrier that ends the previous one).  Role A
// writes P(g-2) to LDS in step g, role B picks it up one step later.  Stages live in a ring of DIST + 5 slots
// (5 in use, DIST on their way from global memory).
// A step runs the same straight-line code whatever the stage.  Stages outside the walk compute on zeros or
// on stale (finite) data and contribute nothing: LDS starts zeroed, and role A starts the S accumulation of
// such a stage from -inf (P = 0), just as it does for the entries a query does not see.
// head_dim 96 is 12 mini-steps of the same kind with the same vector work, which is why a step gets shorter by less than the
// quarter its MFMAs do.  Against zero-padded copies run as head_dim 128, 8192 queries on 32768 keys, 32/8 heads: this kernel
// 5.95 -> 5.56 ms, dQ 3.78 -> 3.33, forward 2.80 -> 2.53, and twelve padding passes of 20 us less.
// S and dP are kept in vector registers, where the vector work reads them directly; the compiler would keep
// every MFMA result of a kernel this size in accumulation registers (one extra move per element), so those
// MFMAs are written as opaque instructions.
// ------------------------------------------------------------------------------------------------
// (CUT: some items are pieces; see fwd_pipe_kernel)
// Kernel arguments read anew, through a pointer the compiler cannot see through, wherever a block needs them: held in scalar registers for
// the length of a kernel they push out values that the steps use (one v_readlane per use).
template <class P>
__device__ __forceinline__ P fresh(const __attribute__((address_space(4))) P* args) {
  asm volatile("" : "+s"(args));
  P p;
  __builtin_memcpy(&p, (const void*)args, sizeof(p));
  return p;
}
// Element x (the same for all lanes) of a list that nothing writes while the kernel runs, in scalar registers.
template <class T>
__device__ __forceinline__ T load_uniform(const T* list, int x) {
  T v;
  __builtin_memcpy(&v, (const void*)((const __attribute__((address_space(4))) T*)(uintptr_t)list + x), sizeof(v));
  return v;
}
template <class P>
using ArgsPtr = const __attribute__((address_space(4))) P*;

constexpr int kStepsInStep = 2048;  // steps of dK/dV walks that start together
template <int D, bool CUT>
__device__ __forceinline__ void dkv_pipe_blocks(const ArgsPtr<DkvParams> args, const int mine) {
  constexpr int NW = 4;        // waves
  constexpr int BM = 32;       // query rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per operand row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dK^T / dV^T
  constexpr int QT = BM * D;   // elements per operand tile
  constexpr int DIST = DKV_PIPE_DIST;  // stages copied ahead of the step that first reads them
  constexpr int NS = DIST + 5; // ring slots: stages g - 4 .. g in use, g + 1 .. g + DIST on their way
  constexpr int NF = 2 * DB + DK;      // operand fragments (mini-steps) per step
  constexpr int AHEAD = 4;             // fragments in flight
  constexpr int PS = 2 * 4 * 64 * 8;   // elements of one P hand-over slot: 2 wave pairs x 4 fragments x 64 lanes x 8
  constexpr int CH = BM * KC;          // 16-byte chunks per operand tile
  constexpr int RING = NF % 8 == 0 ? 8 : 6;  // registers of the fragment ring: a step starts where the ring does
  constexpr int NP = CH / 64;          // 64-slot pieces per tile
  // global->LDS copies per wave and stage: the 2 NP operand pieces and the two sets of row values (LSE, D) are dealt
  // unevenly, because issuing a copy costs a wave about as long as an MFMA and role A (the exponentials) is the one the
  // step waits for: a role A wave copies two pieces and one set of row values, a role B wave six pieces
  constexpr int PER_A = 2, PER_B = (2 * NP - 2 * PER_A) / 2;  // pieces per wave
  constexpr int CPS_A = PER_A + 1, CPS_B = PER_B;              // copies per wave and stage
  constexpr int RV = 64;               // floats per slot of the LSE / D rows (32 used; a whole wave copies them)
  constexpr int VEC0 = NF - 8;         // first mini-step of the vector work (one pair of scores per MFMA)
  constexpr int BOOK = NF - 2;         // mini-step of the bookkeeping, behind the last copy
  static_assert(PER_B % 2 == 0 && NF % RING == 0 && RING > AHEAD && VEC0 >= 4 && 3 + 2 * (PER_B - 1) < BOOK, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int Q_OFF = 0;                 // [NS][QT]  Q rows of stage n in slot n % NS
  constexpr int G_OFF = Q_OFF + NS * QT;   // [NS][QT]  dO rows
  constexpr int P_OFF = G_OFF + NS * QT;   // [2][PS]   P hand-over
  constexpr int R_OFF = P_OFF + 2 * PS;    // [NS][RV] floats LSE rows, then [NS][RV] floats D rows
  lds_f32* const lse_s = (lds_f32*)(L + R_OFF);
  lds_f32* const dsum_s = lse_s + NS * RV;
  constexpr int LDS_ELEMS = R_OFF + 2 * NS * RV * 2;  // in bf16 units

  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int role = wave >> 1, pair = wave & 1;
  const int l32 = lane & 31, hh = lane >> 5;

  // The workgroup is persistent: it claims one block (128 keys of one key/value head) after the other
  // (device_common.hpp) until none is left.  The next block is claimed before the current one's last few steps: early
  // enough for the answer to arrive by the time it is needed, and not earlier (that would fix the order of the blocks
  // before it is known which workgroup is free first).
  // Long equal walks (key blocks that every query sees) wait for the groups of `side_by_side` blocks before theirs, so that a group starts together and
  // shares its rows in the L2: last of eight slices of 16384 queries, 64/8 heads, 84 - 126 -> 53 - 97 GB (two runs each), the eight and a packed chunk together
  // 50 - 55 -> 45 - 48 per launch; that slice, forward and backward, 232.3 -> 231.5 ms.  With shorter walks workgroups only stand idle: 873 queries on 5197 keys, 32/8, whole
  // walks, backward 323 us with the waits, 238 without; 405 on 17711, 64/8, 829 / 740; walks of 1024 steps +- 0.1 %.  And where dQ blocks
  // come first workgroups reach these one by one.  (Head_dim 64, whose steps are half as long, does not wait: of six
  // chunks with such walks none was faster with the waits: 12719 queries on 13105 keys, 64/8 heads, 4441 with, 4341 without, on another box 4442 / 4441, 21790 on 65580, 32/8, 29391 / 29148.)
  int* const next_block = (int*)((__bf16*)smem + LDS_ELEMS);
  const int xcd = xcd_of_this_wave();
  clock_log_stamp(fresh(args).clock_log, 0);
  int blk = mine;
  auto start_in_step = [&](const DkvParams& p, int b) __attribute__((always_inline)) {
    if (CUT || p.side_by_side == 0 || b < 0) return;
    const DkvItem it = load_uniform(p.items, b / p.num_kv_heads);
    if (it.j0 + it.kv_rows <= it.ctx && (int64_t)it.n_qt * p.group >= kStepsInStep) wait_for_earlier_groups(p.ended, b, p.side_by_side);
  };
  if (mine == kClaimBlocks) {
    if (wave == 0) {
      const DkvParams p = fresh(args);
      blk = block_claim_finish(p.taken, p.num_blocks, xcd, block_claim_issue(p.taken, xcd));
      start_in_step(p, blk);
    }
    blk = broadcast_from_wave0(next_block, blk);
  }
  while (blk >= 0) {
  int pending_claim = 0;
  const DkvParams p = fresh(args);
  const int kvh = blk % p.num_kv_heads;
  const DkvItem it = load_uniform(p.items, blk / p.num_kv_heads);
  const int G = p.group;
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const float c = p.scale_log2;

  // zero everything but the ring slots of tiles that the prologue fills
  {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    for (int x = tid; x < (NS - DIST) * QT / 8; x += NW * 64) {
      lds_store8(L + Q_OFF + DIST * QT + x * 8, z);
      lds_store8(L + G_OFF + DIST * QT + x * 8, z);
    }
    for (int x = tid; x < (LDS_ELEMS - P_OFF) / 8; x += NW * 64) lds_store8(L + P_OFF + x * 8, z);
    // (the row values of the first stages are among it: a store by a wave that comes late would undo another wave's copy.  Leaving those out
    // instead of waiting takes scalar registers that the steps then miss: last of eight slices of 128K 229.6 -> 231.6 ms)
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    wg_barrier();
  }

  const int nqt = it.n_qt - it.qt_first;
  // stages: (query tile, head in group), the heads of a tile one after the other, the tiles upwards from the first one
  // that sees the block's keys or (it.reverse, the host's choice) downwards from the segment's last one.  Workgroups that walk the same rows at
  // about the same time (the key blocks of one key/value head run on one XCD) then touch, per query row, one run of
  // G x D contiguous elements, and blocks of different walk lengths stay side by side for the whole of their common
  // part instead of drifting apart head by head.
  const int n_iter = nqt * G;

  // ---- staging: copy i of a role A wave is piece `pair` of Q (i = 0) or of dO (i = 1), the first of the two waves
  // also copies the stage's LSE rows, the second its D rows; copy i of a role B wave is piece 2 + 2 (i % h) + pair of Q
  // (i < h = PER_B / 2) or of dO.  Past the last stage the last one is copied again (into a slot nobody reads any more), so
  // that every step issues the same number of copies. ----
  // byte offset of the lane's chunk of copy i from the tile's first row, for a full tile and for the segment's
  // last tile (rows past the last query repeat it; their P is 0)
  auto piece_in_tile = [&](int i) { return role == 0 ? pair : 2 + 2 * (i % (PER_B / 2)) + pair; };
  unsigned v_full[PER_B], v_last[PER_B];
  {
    const int last_row = it.q_len - 1 - (it.n_qt - 1) * BM;
#pragma unroll
    for (int i = 0; i < PER_B; ++i) {
      const int x = piece_in_tile(i) * 64 + lane;
      const int off = (x >> 5) * 8, row = (x & 31) ^ (((x >> 5) & 3) << 2);
      v_full[i] = (unsigned)(row * (int)q_stride + off) * 2u;
      v_last[i] = (unsigned)(min(row, last_row) * (int)q_stride + off) * 2u;
    }
  }
  // Wave-uniform state of the copies, kept as running byte pointers so that a step spends only a handful of scalar
  // instructions on it: the first row of the next stage to copy in Q and in dO, its LSE / D rows, the stages left in
  // the current head's walk (counting that one), the heads left (counting the current one), the ring slot.
  const bool down = it.reverse != 0;
  const int qt_start = down ? it.n_qt - 1 : it.qt_first;
  const int64_t roff0 = (int64_t)(it.q_row_seg + qt_start * BM) * q_stride + (int64_t)(kvh * G) * D;
  const int64_t rv0 = ((int64_t)(kvh * G) * p.total_q_tiles + it.q_tile0) * 64 + qt_start * BM;
  const char* d_q = reinterpret_cast<const char*>(p.q + roff0);
  const char* d_g = reinterpret_cast<const char*>(p.d_o + roff0);
  const char* d_r = reinterpret_cast<const char*>(((wave & 1) ? p.dsp : p.lse2p) + rv0);
  const int64_t head_bytes = (int64_t)D * 2;                             // to the next head of the group, same tile
  const int64_t head_rows_bytes = p.total_q_tiles * 64 * 4;
  const int64_t tile_bytes = (down ? -1 : 1) * (int64_t)BM * q_stride * 2 - (G - 1) * head_bytes;   // from the last head to the first, next tile
  const int64_t tile_rows_bytes = (down ? -1 : 1) * (int64_t)BM * 4 - (G - 1) * head_rows_bytes;
  int d_heads = G, d_tiles = nqt;
  const int d_ragged = down ? nqt : 1;  // d_tiles while the segment's last query tile is the one to copy
  unsigned d_slot = 0;  // element offset of the ring slot inside the Q / dO rings (slot index x QT)
  const unsigned lane4 = (unsigned)lane * 4u;
  lds_f32* const rows_dst = (wave & 1) ? dsum_s : lse_s;
  auto dma_rows = [&]() __attribute__((always_inline)) { dma4(d_r + lane4, rows_dst + d_slot / (QT / RV)); };
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const bool of_q = role == 0 ? i == 0 : i < PER_B / 2;
    const unsigned voff = d_tiles == d_ragged ? v_last[i] : v_full[i];  // the segment's last query tile
    const char* base = of_q ? d_q : d_g;
    lds_bf16* dst = L + (of_q ? Q_OFF : G_OFF) + piece_in_tile(i) * 512 + d_slot;
    dma16(base + voff, dst);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_heads > 1) {
      --d_heads;
      d_q += head_bytes; d_g += head_bytes; d_r += head_rows_bytes;
    } else {  // on to the next query tile; after the last stage, stay on it
      const bool more = d_tiles > 1;
      d_tiles -= more ? 1 : 0;
      d_heads = more ? G : 1;
      const int64_t tb = more ? tile_bytes : 0, tr = more ? tile_rows_bytes : 0;
      d_q += tb; d_g += tb; d_r += tr;
    }
    d_slot = d_slot == (unsigned)((NS - 1) * QT) ? 0u : d_slot + (unsigned)QT;
  };

  // ---- per-lane operand addresses (elements) inside a tile, as in bwd_dkv_kernel ----
  int x_off[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) x_off[par] = cm_elem(l32, 2 * par + hh);
  int t_off[2];
  {
    const int j = lane & 15, grp = (lane >> 4) & 1;
    const int cl = 2 * grp + ((j & 3) >> 1);
    const int r0 = 4 * hh + (j >> 2);
#pragma unroll
    for (int half = 0; half < 2; ++half) t_off[half] = cm_elem(r0 + 8 * half, cl) + 4 * (j & 1);
  }
  auto prev_slot = [&](int s) __attribute__((always_inline)) { return s == 0 ? NS - 1 : s - 1; };

  // Everything from here on is instantiated once per role, with its own accumulators.
  auto body = [&](auto role_c) __attribute__((always_inline)) {
    constexpr int ROLE = decltype(role_c)::value;
    const lds_bf16* const a_tile = L + (ROLE ? G_OFF : Q_OFF);  // rows operand: Q (role A) or dO (role B)
    const lds_bf16* const t_tile = L + (ROLE ? Q_OFF : G_OFF);  // transposed operand: dO^T (role A) or Q^T (role B)
    const lds_f32* const rv_rows = (ROLE ? dsum_s : lse_s) + 4 * hh;
    lds_bf16* const pex = L + P_OFF + pair * (4 * 512) + lane * 8;

    // this wave's K (role A) or V (role B) fragments, B operands: lane holds X[key = 64 pair + 32 kb + l32][16 ks + 8 hh ..+7]
    bf16x8 bfrag[2][DK];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const __bf16* src = ROLE ? p.v : p.k;
      const int64_t grow = it.kv_row0 + min(64 * pair + 32 * kb + l32, it.kv_rows - 1);
      const int64_t off = grow * kv_stride + (int64_t)kvh * D + 8 * hh;
#pragma unroll
      for (int ks = 0; ks < DK; ++ks) bfrag[kb][ks] = *reinterpret_cast<const bf16x8*>(src + off + 16 * ks);
    }

    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc[2][DB];  // dV^T (role A) or dK^T (role B): [D] x [32 keys of block kb]
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[kb][db] = zero16;

    // key index of this lane's column of block 0 relative to the context: query i of the segment sees the column of
    // block kb iff i >= jrel + 32 kb
    const int jrel = it.j0 + 64 * pair + l32 - it.ctx;
    const int jrel_hi = it.j0 + 64 * pair + 63 - it.ctx;  // of the wave's last key

    // prologue: stages 0 .. DIST - 1 (after the fragment loads, so that the waits below count only copies)
    constexpr int CPS = ROLE ? CPS_B : CPS_A;      // copies of this wave per stage
    constexpr int PIECES = ROLE ? PER_B : PER_A;
#pragma unroll
    for (int s = 0; s < DIST; ++s) {
      if (ROLE == 0) dma_rows();
#pragma unroll
      for (int i = 0; i < PIECES; ++i) dma_piece(i);
      dma_advance();
    }
    // A wait the compiler can see, for the fragments and stage 0 (the later stages are waited for step by step): without it the
    // compiler's own bookkeeping of outstanding loads makes it put a full vmcnt(0) wait inside the loop (before role A's first S MFMA).
    wait_all_but<(DIST - 1) * CPS>();
    wg_barrier();

    // pipeline state
    int sA = ROLE ? NS - 2 : 0;  // slot of stage g - 2 ROLE (rows operand); one before: row values and the next step's
                                 // transposed operand; two before: this step's transposed operand
    int s_qt = qt_start;         // role A: query tile of stage g (whose S is computed in step g)
    int s_heads = G;             //         and the heads of that tile still to come, counting stage g's
    // Role A masks through the accumulator: the first MFMA of S starts from a tile that holds -inf where the query
    // does not see the key (and everywhere for a stage past the end of the walk) and 0 elsewhere.  The tile is
    // rebuilt only for the stages that need it.
    f32x16 mask_c[2] = {zero16, zero16};
    bool mask_set = false;
    f32x16 x[2][2];              // S or dP: [buffer][key block]
    bf16x8 f[2][2][2];           // P or dS as B operands: [buffer][key block][k-step]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int i = 0; i < 16; ++i) x[b][kb][i] = ROLE ? 0.f : -INFINITY;  // role A: P = 0 before the first stage
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int i = 0; i < 8; ++i) f[b][kb][ks][i] = (__bf16)0.0f;
      }
    bf16x8 fr[RING];  // ring of operand fragments

    // byte addresses of this lane's operand reads inside slot 0
    const unsigned t_lo0 = lds_addr(t_tile + t_off[0]), t_hi0 = lds_addr(t_tile + t_off[1]);
    const unsigned a_ev0 = lds_addr(a_tile + x_off[0]), a_od0 = lds_addr(a_tile + x_off[1]);
    const unsigned rv0 = lds_addr(rv_rows), pex0 = lds_addr(pex);
    constexpr unsigned SLOT = QT * 2;  // bytes per ring slot
    // transposed fragment m = ks2 * DB + db of the tile at (lo, hi)
    auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2;
      const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
      const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // rows fragment of k-step ks of the tile at (even, odd)
    auto load_a = [&](unsigned ev_addr, unsigned od_addr, auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      constexpr int off = (ks >> 1) * (4 * 32 * 8) * 2;
      return lds_asm_read16<off>((ks & 1) ? od_addr : ev_addr);
    };

    // the first fragments of step 0 (zeros)
    {
      const unsigned sT = prev_slot(prev_slot(sA)) * SLOT;
      static_for<0, AHEAD>([&](auto m_c) __attribute__((always_inline)) {
        fr[decltype(m_c)::value] = load_t(t_lo0 + sT, t_hi0 + sT, m_c);
      });
    }

    using Lds = DkvLdsOrder<ROLE, NF, 2 * DB>;  // the waits for LDS data (see there)
    auto step = [&](int g, f32x16 (&cur)[2], f32x16 (&nxt)[2], bf16x8 (&f_old)[2][2],
                    bf16x8 (&f_new)[2][2]) __attribute__((always_inline)) {
      const int sR = prev_slot(sA), sT = prev_slot(sR);
      const unsigned oA = sA * SLOT, oR = sR * SLOT, oT = sT * SLOT;
      const unsigned t_lo = t_lo0 + oT, t_hi = t_hi0 + oT, a_ev = a_ev0 + oA, a_od = a_od0 + oA;
      const unsigned n_lo = t_lo0 + oR, n_hi = t_hi0 + oR;
      if (ROLE == 0) {
        // entry (query 8 (i / 4) + 4 hh + i % 4 of the tile, column of block kb) is visible iff 8 (i / 4) + i % 4 >= lim[kb]
        const bool valid = g < n_iter;
        if (__builtin_expect(!valid || s_qt * BM < jrel_hi, 0)) {  // rare: keep it out of the loop's straight line
          const int lim0 = valid ? jrel - s_qt * BM - 4 * hh : 0x40000000;
          const int lim1 = valid ? lim0 + 32 : 0x40000000;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            mask_c[0][i] = 8 * (i >> 2) + (i & 3) < lim0 ? -INFINITY : 0.f;
            mask_c[1][i] = 8 * (i >> 2) + (i & 3) < lim1 ? -INFINITY : 0.f;
          }
          mask_set = true;
        } else if (__builtin_expect(mask_set, 0)) {
          mask_c[0] = zero16;
          mask_c[1] = zero16;
          mask_set = false;
        }
      }
      // hand-over and row values are issued between the MFMAs of the first mini-steps, so that the matrix pipe restarts
      // right after the barrier; the vector work starts at mini-step 4
      bf16x8 ph[2][2];
      f32x4 r4[4];  // LSE (role A) or -D (role B) of rows 8 g4 + 4 hh + 0..3
      const unsigned pa = pex0 + (ROLE == 0 ? (g & 1) : ((g & 1) ^ 1)) * (PS * 2);
      const unsigned ra = rv0 + sR * (RV * 4);
      unsigned pw[2][8];
      float e_hold[2];  // role A: exponentials of the previous pair (converted one mini-step later: a transcendental
                        // result cannot be consumed by the very next instruction)
      // vector work of score 2 dw + q of block kb (pair j = 8 kb + dw), pinned to where it is written (the compiler
      // would gather the vector work elsewhere)
      auto vec_half = [&](auto j_c, auto q_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value, q = decltype(q_c)::value;
        constexpr int kb = j >> 3, dw = j & 7, i = 2 * dw + q;
        if (ROLE == 0) {
          if constexpr (j > 0 && q == 0) {  // the previous pair's exponentials
            bf16x2 w;
            w[0] = (__bf16)e_hold[0]; w[1] = (__bf16)e_hold[1];
            unsigned wu = __builtin_bit_cast(unsigned, w);
            asm volatile("" : "+v"(wu));
            pw[(j - 1) >> 3][(j - 1) & 7] = wu;
          }
          e_hold[q] = __builtin_amdgcn_exp2f(cur[kb][i] * c - r4[i >> 2][i & 3]);
          asm volatile("" : "+v"(e_hold[q]));
        } else {
          const float e = (float)ph[kb][i >> 3][i & 7] * (cur[kb][i] + r4[i >> 2][i & 3]);  // r4 = -D
          if constexpr (q == 0) {
            e_hold[0] = e;
            asm volatile("" : "+v"(e_hold[0]));
          } else {
            bf16x2 w;
            w[0] = (__bf16)e_hold[0]; w[1] = (__bf16)e;
            unsigned wu = __builtin_bit_cast(unsigned, w);
            asm volatile("" : "+v"(wu));
            pw[kb][dw] = wu;
          }
        }
      };
      auto vec_pair = [&](auto j_c) __attribute__((always_inline)) {
        vec_half(j_c, std::integral_constant<int, 0>{});
        vec_half(j_c, std::integral_constant<int, 1>{});
      };
      asm volatile("s_nop 7" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value;
        {  // wait for fragment m (and, in mini-step 4, for the hand-over and the row values)
          constexpr int lgkm = Lds::wait(m);
          static_assert(lgkm >= 0 && lgkm <= 15, "lgkmcnt is a 4-bit counter");
          if constexpr (m == 4) {
            if (ROLE == 0)
              asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(fr[m % RING]), "+v"(r4[0]), "+v"(r4[1]), "+v"(r4[2]), "+v"(r4[3]) : "n"(lgkm));
            else
              asm volatile("s_waitcnt lgkmcnt(%9)" : "+v"(fr[m % RING]), "+v"(r4[0]), "+v"(r4[1]), "+v"(r4[2]), "+v"(r4[3]),
                           "+v"(ph[0][0]), "+v"(ph[0][1]), "+v"(ph[1][0]), "+v"(ph[1][1]) : "n"(lgkm));
          } else {
            asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(lgkm));
          }
        }
        {  // read the fragment of mini-step m + AHEAD (past the end: the next step's first transposed fragments)
          constexpr int mm = m + AHEAD;
          if constexpr (mm < 2 * DB) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm>{});
          else if constexpr (mm < NF) fr[mm % RING] = load_a(a_ev, a_od, std::integral_constant<int, mm - 2 * DB>{});
          else fr[mm % RING] = load_t(n_lo, n_hi, std::integral_constant<int, mm - NF>{});
        }
        const bf16x8 fa = fr[m % RING];
        // S / dP live in vector registers (the vector work reads them directly) and K / V fragments in accumulation
        // registers; written as opaque instructions since the compiler keeps every MFMA result of a kernel with more
        // than 256 registers in accumulation registers.  Their results are first read one step later.
        auto mma = [&](auto kb_c) __attribute__((always_inline)) {
          constexpr int kb = decltype(kb_c)::value;
          if constexpr (m < 2 * DB) {
            constexpr int ks = m / DB, db = m % DB;
            acc[kb][db] = mfma32(fa, f_old[kb][ks], acc[kb][db]);
          } else {
            constexpr int ks = m - 2 * DB;
            if (ks == 0 && ROLE == 0)
              asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(nxt[kb]) : "v"(fa), "a"(bfrag[kb][ks]), "v"(mask_c[kb]));
            else if (ks == 0)
              asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(nxt[kb]) : "v"(fa), "a"(bfrag[kb][ks]));
            else
              asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(nxt[kb]) : "v"(fa), "a"(bfrag[kb][ks]));
          }
        };
        // The mini-step's two MFMAs are kept apart by half of its other work: issued back to back, the second one would
        // hold up the wave (the only one on this SIMD) until the first has left the matrix pipe.
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, 1> c1{};
        mma(c0);
        // hand-over and row values (DkvLdsOrder: E0)
        if constexpr (ROLE == 0) {
          if constexpr (m < 4) lds_asm_write16<1024 * m>(pa, f_old[m >> 1][m & 1]);
        } else {
          if constexpr (m == 0) {
            ph[0][0] = lds_asm_read16<0>(pa);
            ph[0][1] = lds_asm_read16<1024>(pa);
            ph[1][0] = lds_asm_read16<2048>(pa);
            ph[1][1] = lds_asm_read16<3072>(pa);
          }
          if constexpr (m == 1) {
            r4[0] = lds_asm_read16f<0>(ra);
            r4[1] = lds_asm_read16f<32>(ra);
            r4[2] = lds_asm_read16f<64>(ra);
            r4[3] = lds_asm_read16f<96>(ra);
          }
        }
        if (m == 2 && ROLE == 0) dma_rows();
        // Vector work next to the MFMAs: one pair (two scores of a key block) after each MFMA of the second half of the
        // step; the MFMAs of the first half run unhindered.  Measured for role A (fma + exponential) against an even
        // spread over the whole step (2.1 % slower), one score per MFMA from mini-step 4 on and two in the last four
        // mini-steps (0.5 - 1 % slower) and everything in the last four mini-steps (9.6 % slower); for role B against
        // the second of these (1.2 % slower).
        if constexpr (m >= VEC0) vec_pair(std::integral_constant<int, 2 * (m - VEC0)>{});
        __builtin_amdgcn_sched_barrier(0);
        mma(c1);
        if constexpr (ROLE == 0 && m < 2) {  // (E1)
          r4[2 * m] = lds_asm_read16f<64 * m>(ra);
          r4[2 * m + 1] = lds_asm_read16f<64 * m + 32>(ra);
        }
        if (m >= 3 && m < 3 + 2 * PIECES && ((m - 3) & 1) == 0) dma_piece((m - 3) >> 1);
        if constexpr (m >= VEC0) vec_pair(std::integral_constant<int, 2 * (m - VEC0) + 1>{});
        if constexpr (m == BOOK) {  // bookkeeping for the next step (the copies of this step have been issued)
          dma_advance();
          sA = sA == NS - 1 ? 0 : sA + 1;
          if (ROLE == 0 && --s_heads == 0) {
            s_heads = G;
            s_qt += down ? -1 : 1;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if (ROLE == 0) {
        bf16x2 w;
        w[0] = (__bf16)e_hold[0]; w[1] = (__bf16)e_hold[1];
        pw[1][7] = __builtin_bit_cast(unsigned, w);
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          u32x4 v = {pw[kb][4 * ks], pw[kb][4 * ks + 1], pw[kb][4 * ks + 2], pw[kb][4 * ks + 3]};
          f_new[kb][ks] = __builtin_bit_cast(bf16x8, v);
        }
      // Stage g + 1 must have landed; the copies of the DIST - 1 stages after it may still be in flight.  This wave's
      // hand-over stores completed long ago (mini-step 4 waited for them).
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 1) * CPS) : "memory");
      wg_barrier();
    };
    // role A's last product is dV^T of stage n - 1 in step n + 1, role B's dK^T of stage n - 1 in step n + 3
    const int n_steps = n_iter + 4;
    const int claim_at = max(0, n_steps - 4) & ~1;  // the step pair before which wave 0 claims the next block
    for (int g = 0; g < n_steps; g += 2) {
      if (g == claim_at && wave == 0 && mine == kClaimBlocks) pending_claim = block_claim_issue(fresh(args).taken, xcd);
      step(g, x[0], x[1], f[0], f[1]);
      step(g + 1, x[1], x[0], f[1], f[0]);
    }
    // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
    // every copy of this wave has landed (the last ones rewrote a slot nobody reads): once all waves have met at the
    // barrier that hands out the next block, the ring may be filled again
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)

    // ---- epilogue: dV = dV^T (role A), dK = scale * dK^T (role B), written (or added) as bf16 ----
    const DkvParams p = fresh(args);
    const int64_t kv_stride = (int64_t)p.num_kv_heads * D;
    if (CUT && it.part >= 0) {  // a piece: the accumulators as they are, put together by bwd_merge_kernel
      float* const out = p.parts + ((int64_t)it.part * p.num_kv_heads + kvh) * kPartRowFloats + (4 * ROLE + 2 * pair) * 4096 + lane * 4;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4*>(out + kb * 4096 + (db * 4 + g) * 256) =
                f32x4{acc[kb][db][4 * g], acc[kb][db][4 * g + 1], acc[kb][db][4 * g + 2], acc[kb][db][4 * g + 3]};
    } else
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int kr = 64 * pair + 32 * kb + l32;
      if (kr < it.kv_rows) {
        const int64_t off = ((int64_t)it.kv_row0 + kr) * kv_stride + (int64_t)kvh * D;
        __bf16* const out = ROLE ? p.dk : p.dv;
        const float fs = ROLE ? p.scale : 1.0f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            dkv_store4(p, out, off + 32 * db + 8 * g + 4 * hh, acc[kb][db][4 * g] * fs, acc[kb][db][4 * g + 1] * fs,
                       acc[kb][db][4 * g + 2] * fs, acc[kb][db][4 * g + 3] * fs);
          }
      }
    }
  };
  if (role == 0) body(std::integral_constant<int, 0>{});
  else body(std::integral_constant<int, 1>{});
  if (mine != kClaimBlocks) break;
  // on to the next block; the stores of the epilogue are not waited for here
  int nb = 0;
  if (wave == 0) {
    const DkvParams p = fresh(args);
    if (!CUT && p.side_by_side != 0 && lane == 0) __hip_atomic_fetch_add(p.ended + (blk & 7), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    nb = block_claim_finish(p.taken, p.num_blocks, xcd, pending_claim);
    start_in_step(p, nb);
  }
  blk = broadcast_from_wave0(next_block, nb);
  }
  clock_log_stamp(fresh(args).clock_log, 1);
}

// The rows of dK or dV that a wave holds as N transposed blocks of 32 keys, times `scale`, as bf16 through LDS of its own (`stage`, N x 32 rows): the lane that
// holds four values of a row puts them there, and whole rows leave, 16 bytes per lane.  Stored by their holders, 8 bytes each, the rows of a block of 256 keys took
// 10 us; backward before -> now: 1024 queries on 32768 keys, 32/8 heads, 1503 -> 1484 us, 3662 causal tokens, 16/16, 202.4 -> 198.6, head_dim 256, 2668, 8/8, 141.7 ->
// 139.0.  Rows from `rows` on are not stored.
template <int D, int N>
__device__ __forceinline__ void store_key_rows(lds_bf16* stage, const f32x16 (&x)[N][D / 32], float scale, __bf16* out, int64_t stride, int rows) {
  constexpr int KC = D / 8;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int kb = 0; kb < N; ++kb)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(__attribute__((address_space(3))) bf16x4*)(stage + tile_elem<KC>(32 * kb + (lane & 31), 4 * db + g) + 4 * (lane >> 5)) =
            pack4(x[kb][db][4 * g] * scale, x[kb][db][4 * g + 1] * scale, x[kb][db][4 * g + 2] * scale, x[kb][db][4 * g + 3] * scale);
#pragma unroll 4
  for (int i = 0; i < N * 32 * KC / 64; ++i) {
    const int y = i * 64 + lane, row = y / KC, c = unswz<KC>(row, y % KC);
    const bf16x8 v = lds_load8(stage + y * 8);
    if (row < rows) *reinterpret_cast<bf16x8*>(out + row * stride + c * 8) = v;
  }
}

// ------------------------------------------------------------------------------------------------
// dkv_tall_blocks (head_dim 128, 96 and 64): the dK/dV blocks of bwd_pipe_kernel where they end sooner than those of dkv_pipe_blocks (tall_pays) or, at 64, than
// those of bwd_dkv_narrow_pipe_kernel in a launch behind that of dQ (narrow_tall_pays)
//
// A workgroup covers 256 keys, each of its four waves all four contractions of 64 of them: no wave roles, no hand-over, half the barriers, and a stage that
// has been copied to LDS serves twice the keys.  Stage n is the n-th (head, 32-row query tile) of the walk, as in dkv_pipe_blocks; step g is
//     S(g) = Q K^T     dK^T += Q^T dS(g-1)     dP(g) = dO V^T - D     dV^T += dO^T P(g)             (matrix pipe, in this order)
//     dS(g-1) = P(g-1) dP(g-1)  until dK^T needs it,  P(g) = exp2(S(g) c - LSE)  until dV^T needs it,  dS(g) from dP(g)'s end on   (vector)
// as 4 D / 16 mini-steps of one LDS operand fragment and the two MFMAs it feeds (one per 32-key block), each MFMA with its even share of the vector
// work behind it.  That order keeps one tile each of S, dP, P and dS alive, 80 registers at most: with K and V fragments (128 at head_dim 128) and the
// accumulators (256, all the accumulation registers there are) a wave has no room for a second one.  -D is what the sum of dP starts from, and one copy
// of a stage is issued every NF / PER mini-steps (behind each other they hold the wave up).  What few registers are left decides: two of them reloaded
// from scratch in every step, each time with a wait for all copies in flight, made a step 2800 -> 3330 cycles (a test looks for that).
// Bound by the issue of MFMAs at the clock that the chip's power leaves: 8192 queries on 32768 keys, 32/8 heads, the matrix pipes are busy 73 % of the cycles of these blocks, at 1.78 GHz (MFMAs alone: 96 % at 1.79), where
// dkv_pipe_blocks' were busy 59 % at 1.95 GHz (head_dim 96: 63 % at 1.88, 50 % at 2.09); cycles per 64 MFMAs of a wave 3470 -> 2800, time of these blocks 6.38 -> 5.63
// ms (96: 5.26 -> 4.66), of the backward 10.75 -> 10.18 (8.76 -> 8.40); at 64, 8192 queries on 16384 keys, 3.00 -> 2.72.  What a step could still save is little: twice the row fragments' reads cost 2.7
// % of its time, 96 more vector instructions 6 %, twice the copies 2.2 %.  Head_dim 64 has registers for P in float32, which dS then takes (32 instructions less).
// ------------------------------------------------------------------------------------------------
// LDS instructions of one step in program order and the waits that follow from it: mini-step m issues the read of fragment m + AHEAD (two instructions
// for a transposed one; past the end the next step's first), then extra(m) reads of row values after its first MFMA.  What extra(m) reads is there at
// the wait of mini-step m + AHEAD + 1.
template <int DK, int AHEAD>
struct TallOrder {
  static constexpr int NF = 4 * DK;
  static constexpr int EXP0 = DK + 2, DS0 = 3 * DK + 2;  // mini-steps in which the vector work of P and of dS starts; each lasts 2 DK of them
  static constexpr int cost(int k) { return (k % NF) / DK % 2 == 1 ? 2 : 1; }
  static constexpr int exps(int m) { return spread(32, EXP0, EXP0 + 2 * DK, m); }  // scores done by the end of mini-step m
  static constexpr int dss(int m) { return spread(32, DS0, DS0 + 2 * DK, m); }     // (m < 2 NF: the work goes on in the next step)
  static constexpr int lse_use(int quad) {  // first mini-step that needs the LSE of rows 8 quad + 4 hh ..+3
    int m = EXP0;
    while (exps(m) <= 8 * quad) ++m;
    return m;
  }
  static constexpr int lse_read(int quad) { return lse_use(quad) - AHEAD - 1; }
  static constexpr int d_use() { return 2 * DK; }  // the -D tile: four reads, two in each of two mini-steps
  static constexpr int extra(int m) {
    int n = 0;
    for (int q = 0; q < 4; ++q) n += lse_read(q) == m ? 1 : 0;
    return n + (m == d_use() - AHEAD - 2 || m == d_use() - AHEAD - 1 ? 2 : 0);
  }
  static constexpr int wait(int m) {
    int n = extra((m - AHEAD + NF) % NF);
    for (int i = m - AHEAD + 1; i < m; ++i) n += cost((i + AHEAD + NF) % NF) + extra((i + NF) % NF);
    return n;
  }
  // P and dS of the rows of a k-step are packed before the first product that reads them (pair 7 when element 16 has been done)
  static_assert(exps(3 * DK - 1) >= 17 && exps(3 * DK + DK / 2 - 1) == 32 && dss(NF + DK - 1) >= 16 && dss(NF + DK + DK / 2 - 1) == 32, "the order of a step");
};
static_assert(TallOrder<8, 4>::lse_read(0) == 5 && TallOrder<8, 4>::lse_read(3) == 17 && TallOrder<8, 4>::exps(25) == 32 && TallOrder<8, 4>::dss(41) == 32 &&
              TallOrder<8, 4>::wait(0) == 3 && TallOrder<8, 4>::wait(5) == 4 && TallOrder<8, 4>::wait(14) == 9, "worked out by hand");

template <int D>
__device__ __forceinline__ void dkv_tall_blocks(const ArgsPtr<DkvParams> args, const int mine) {
  constexpr int NW = 4;        // waves
  constexpr int BM = 32;       // query rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per operand row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dK^T / dV^T
  constexpr int QT = BM * D;   // elements per operand tile
  constexpr int DIST = 6;      // stages copied ahead
  constexpr int NS = DIST + 2; // ring slots: stages g - 1 and g in use, g + 1 .. g + DIST on their way
  constexpr int NF = 4 * DK;   // fragments (mini-steps) per step: Q rows, Q^T, dO rows, dO^T
  constexpr int AHEAD = D == 96 ? 5 : 4, RING = 8;   // fragments in flight, names of the fragment ring
  constexpr int NP = BM * KC / 64;     // 64-slot pieces per tile
  constexpr int PER = 2 * NP / NW;     // pieces per wave and stage
  constexpr int RV = 64;               // floats per slot of the LSE / D rows (32 used; a whole wave copies them)
  constexpr int BOOK = NF - 2;
  constexpr bool KEEP_P = D == 64;     // P stays in float32 for dS (32 registers more, 32 instructions of a step less)
  using Order = TallOrder<DK, AHEAD>;
  constexpr int COPY_EVERY = NF / PER;  // mini-steps from one copy of a stage to the next
  static_assert(NF % RING == 0 && AHEAD <= DK && 2 * DB == DK && NP % 2 == 0 && NF % PER == 0 && NF - 3 <= BOOK, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int R_OFF = NS * 2 * QT;       // slot n % NS holds stage n: [QT] Q rows, then [QT] dO rows (chunk-major); behind the ring
  lds_f32* const lse_s = (lds_f32*)(L + R_OFF);   // [NS][RV] LSE rows, then [NS][RV] D rows
  lds_f32* const dsum_s = lse_s + NS * RV;
  int* const next_block = (int*)((__bf16*)smem + R_OFF + 2 * NS * RV * 2);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the lane is counted anew where it is needed: held in registers, it and what follows from it would take those of the steps)
  auto lane_id = []() __attribute__((always_inline)) {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
  };

  // Persistent, and long equal walks start in groups, as in dkv_pipe_blocks.  (At 64 none do, by side_by_side: compiled without them, these blocks were 0.3 - 0.8 % slower.)
  const int xcd = xcd_of_this_wave();
  clock_log_stamp(fresh(args).clock_log, 0);
  int blk = mine;
  auto start_in_step = [&](const DkvParams& p, int b) __attribute__((always_inline)) {
    if (p.side_by_side == 0 || b < 0) return;
    const DkvItem it = load_uniform(p.items, b / p.num_kv_heads);
    if (it.j0 + it.kv_rows <= it.ctx && (int64_t)it.n_qt * p.group >= kStepsInStep) wait_for_earlier_groups(p.ended, b, p.side_by_side);
  };
  if (mine == kClaimBlocks) {
    if (wave == 0) {
      const DkvParams p = fresh(args);
      blk = block_claim_finish(p.taken, p.num_blocks, xcd, block_claim_issue(p.taken, xcd));
      start_in_step(p, blk);
    }
    blk = broadcast_from_wave0(next_block, blk);
  }
  while (blk >= 0) {
  int pending_claim = 0;
  const DkvParams p = fresh(args);
  const int kvh = blk % p.num_kv_heads;
  const DkvItem it = load_uniform(p.items, blk / p.num_kv_heads);
  const int G = p.group;
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const float c = p.scale_log2;

  // the Q tile of the slot before the first one, which step 0 reads as stage -1's (dS(-1) = 0)
  {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    for (int x = wave * 64 + lane_id(); x < QT / 8; x += NW * 64) lds_store8(L + (NS - 1) * 2 * QT + x * 8, z);
  }

  const int nqt = it.n_qt - it.qt_first;
  const int n_iter = nqt * G;

  // ---- staging (see dkv_pipe_blocks): copy i of a wave is piece i * 4 + wave of the stage's 2 NP, those of Q first; waves 0 and 1 also copy the
  // stage's LSE and D rows.  Rows past the segment's last query repeat it (their P is 0) ----
  // (piece p is chunks 2 p and 2 p + 1 of the rows; p is odd for all copies of a wave or for none, so that they share their rows' order)
  unsigned v_off;  // byte offset of the lane's chunk of piece 0 or 1 from the tile's first row, but for the piece's own 32 bytes
  const int last_row = it.q_len - 1 - (it.n_qt - 1) * BM;
  auto set_offsets = [&](int max_row) __attribute__((always_inline)) {
    const int lane = lane_id(), hh = lane >> 5, row = (lane & 31) ^ ((2 * (wave & 1) + hh) << 2);
    v_off = (unsigned)(min(row, max_row) * (int)q_stride + 8 * hh) * 2u;
  };
  const bool down = it.reverse != 0;
  const int qt_start = down ? it.n_qt - 1 : it.qt_first;
  const int64_t roff0 = (int64_t)(it.q_row_seg + qt_start * BM) * q_stride + (int64_t)(kvh * G) * D;
  const int64_t rv_first = ((int64_t)(kvh * G) * p.total_q_tiles + it.q_tile0) * 64 + qt_start * BM;
  const char* d_q = reinterpret_cast<const char*>(p.q + roff0);
  const char* d_g = reinterpret_cast<const char*>(p.d_o + roff0);
  const char* d_r = reinterpret_cast<const char*>((wave & 1 ? p.dsp : p.lse2p) + rv_first);
  const int64_t head_bytes = (int64_t)D * 2;
  const int64_t head_rows_bytes = p.total_q_tiles * 64 * 4;
  const int64_t tile_bytes = (down ? -1 : 1) * (int64_t)BM * q_stride * 2 - (G - 1) * head_bytes;
  const int64_t tile_rows_bytes = (down ? -1 : 1) * (int64_t)BM * 4 - (G - 1) * head_rows_bytes;
  int d_heads = G, d_tiles = nqt;
  const int d_ragged = down ? nqt : 1;  // d_tiles while the segment's last query tile is the one to copy
  unsigned d_slot = 0;
  lds_f32* const rows_dst = wave & 1 ? dsum_s : lse_s;
  set_offsets(d_tiles == d_ragged ? last_row : BM - 1);
  auto dma_rows = [&]() __attribute__((always_inline)) {
    if (wave < 2) dma4(d_r + (unsigned)lane_id() * 4u, rows_dst + d_slot * RV);
  };
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const int piece = i * NW + wave;
    const bool of_q = NP % NW == 0 ? i < NP / NW : piece < NP;
    asm volatile("" : "+v"(v_off));  // (widened here, not in registers held for it)
    dma16((of_q ? d_q + piece * 32 : d_g + (piece - NP) * 32) + v_off, L + d_slot * (2 * QT) + piece * 512);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_heads > 1) {
      --d_heads;
      d_q += head_bytes; d_g += head_bytes; d_r += head_rows_bytes;
    } else {  // on to the next query tile; after the last stage, stay on it
      const bool more = d_tiles > 1;
      d_tiles -= more ? 1 : 0;
      d_heads = more ? G : 1;
      const int64_t tb = more ? tile_bytes : 0, tr = more ? tile_rows_bytes : 0;
      d_q += tb; d_g += tb; d_r += tr;
      if (__builtin_expect(more && (d_tiles == d_ragged || d_tiles + 1 == d_ragged), 0)) set_offsets(d_tiles == d_ragged ? last_row : BM - 1);
    }
    d_slot = d_slot == NS - 1 ? 0u : d_slot + 1;
  };

  // byte addresses of this lane's operand reads in the Q tile of slot 0; the dO tile is a constant further
  // (odd k-steps: chunk 2 + hh instead of hh is 1024 bytes further with bit 3 of the row turned over; rows r0 + 8: the same bit)
  constexpr unsigned ROW8 = 8 * 16;
  unsigned ev0, lo0, lse0;
  {
    const int lane = lane_id(), l32 = lane & 31, hh = lane >> 5;
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    ev0 = lds_addr(L + cm_elem(l32, hh));
    lo0 = lds_addr(L + cm_elem(r0, cl) + 4 * (j & 1));
    lse0 = lds_addr(lse_s + 4 * hh);
  }
  constexpr unsigned SLOT = 2 * QT * 2;           // bytes per ring slot
  constexpr int DO_TILE = QT * 2;                 // bytes from the Q tile to the dO tile
  constexpr int D_ROWS = NS * RV * 4;             // bytes from the LSE rows to the D rows
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c, auto tile_c) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value;
    constexpr int off = (ks >> 1) * (4 * 32 * 8) * 2 + (ks & 1) * 1024 + decltype(tile_c)::value;
    return lds_asm_read16<off>((ks & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c, auto tile_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2 + decltype(tile_c)::value;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  constexpr std::integral_constant<int, 0> in_q{};
  constexpr std::integral_constant<int, DO_TILE> in_do{};

  // K and V fragments (B operands): lane holds X[key = 64 wave + 32 kb + l32][16 ks + 8 hh ..+7]
  bf16x8 kf[2][DK], vf[2][DK];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int lane = lane_id();
    const int64_t grow = it.kv_row0 + min(64 * wave + 32 * kb + (lane & 31), it.kv_rows - 1);
    const int64_t off = grow * kv_stride + (int64_t)kvh * D + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      kf[kb][ks] = *reinterpret_cast<const bf16x8*>(p.k + off + 16 * ks);
      vf[kb][ks] = *reinterpret_cast<const bf16x8*>(p.v + off + 16 * ks);
    }
  }
  // prologue: the copies of stages 0 .. DIST - 1
#pragma unroll
  for (int s = 0; s < DIST; ++s) {
    dma_rows();
#pragma unroll
    for (int i = 0; i < PER; ++i) dma_piece(i);
    dma_advance();
  }
  // stages 0 and 1 have landed (a wait the compiler can see, for the fragments).  (Waves 0 and 1 have a copy more per stage and wait for up to
  // DIST - 2 copies more than they need; so do the waits at the end of a step.)
  wait_all_but<(DIST - 2) * PER>();
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dk[2][DB], dv[2][DB];  // dK^T, dV^T: [D] x [32 keys of block kb]
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[kb][db] = dv[kb][db] = zero16;
  f32x16 s[2], dp[2];           // S (then P, packed into pw) and dP - D: [key block]
  f32x16 ps[2];                 // KEEP_P: P
  if constexpr (KEEP_P) ps[0] = ps[1] = zero16;
  u32x4 pw[2][2], sw[2][2];     // P and dS as B operands: [key block][k-step], pairs of bf16
  dp[0] = dp[1] = zero16;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) pw[kb][ks] = sw[kb][ks] = u32x4{0, 0, 0, 0};
  bf16x8 fr[RING];
  static_for<0, AHEAD>([&](auto k_c) __attribute__((always_inline)) { fr[decltype(k_c)::value] = load_rows(ev0, ev0 ^ ROW8, k_c, in_q); });

  // key index of this lane's column of block 0 relative to the context: query i of the segment sees the column of block kb
  // iff i >= jrel + l32 + 32 kb
  const int jrel = it.j0 + 64 * wave - it.ctx;          // (lane 0)
  const int jrel_hi = it.j0 + 64 * wave + 63 - it.ctx;  // of the wave's last key
  int s_cur = 0;        // slot of stage g
  int s_qt = qt_start;  // query tile of stage g
  int s_heads = G;      // heads of that tile still to come, counting stage g's

  auto step = [&](int g) __attribute__((always_inline)) {
    const int s_nxt = s_cur == NS - 1 ? 0 : s_cur + 1, s_prv = s_cur == 0 ? NS - 1 : s_cur - 1;
    const unsigned c_ev = ev0 + s_cur * SLOT, c_od = c_ev ^ ROW8, n_ev = ev0 + s_nxt * SLOT, n_od = n_ev ^ ROW8;
    const unsigned c_lo = lo0 + s_cur * SLOT, c_hi = c_lo ^ ROW8, p_lo = lo0 + s_prv * SLOT, p_hi = p_lo ^ ROW8;
    const unsigned r_cur = lse0 + s_cur * (RV * 4);
    f32x4 rl[4];          // LSE of rows 8 g4 + 4 hh + 0..3
    f32x4 rd[4];          // -D of the same rows
    f32x16 rd16;
    float e_hold;         // the first exponential (or dS) of a pair, until the second one is there
    // Element x of the vector work: rows in the order in which the products need them, 4 g4 + (x % 4) of block (x / 4) % 2, g4 = x / 8.
    auto exp_one = [&](auto x_c) __attribute__((always_inline)) {
      constexpr int x = decltype(x_c)::value, g4 = x / 8, kb = x / 4 % 2, i = 4 * g4 + x % 4;
      float e = __builtin_amdgcn_exp2f(s[kb][i] * c - rl[g4][i & 3]);
      asm volatile("" : "+v"(e));
      (KEEP_P ? ps : s)[kb][i] = e;
    };
    auto pack_p = [&](auto y_c) __attribute__((always_inline)) {  // pair y: elements 2 y and 2 y + 1
      constexpr int y = decltype(y_c)::value, kb = y / 2 % 2, w = 2 * (y / 4) + y % 2;
      bf16x2 v;
      v[0] = (__bf16)(KEEP_P ? ps : s)[kb][2 * w]; v[1] = (__bf16)(KEEP_P ? ps : s)[kb][2 * w + 1];
      unsigned u = __builtin_bit_cast(unsigned, v);
      asm volatile("" : "+v"(u));
      pw[kb][w / 4][w % 4] = u;
    };
    auto ds_one = [&](auto x_c) __attribute__((always_inline)) {
      constexpr int x = decltype(x_c)::value, kb = x / 4 % 2, i = 4 * (x / 8) + x % 4, w = i / 2;
      const unsigned pu = pw[kb][w / 4][w % 4];
      float e = (KEEP_P ? ps[kb][i] : __uint_as_float(i % 2 == 0 ? pu << 16 : pu & 0xffff0000u)) * dp[kb][i];
      if constexpr (i % 2 == 0) {
        asm volatile("" : "+v"(e));
        e_hold = e;
      } else {
        bf16x2 v;
        v[0] = (__bf16)e_hold; v[1] = (__bf16)e;
        unsigned u = __builtin_bit_cast(unsigned, v);
        asm volatile("" : "+v"(u));
        sw[kb][w / 4][w % 4] = u;
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      constexpr int lgkm = Order::wait(m);
      static_assert(lgkm >= 0 && lgkm <= 15, "lgkmcnt is a 4-bit counter");
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(lgkm));
      if constexpr (m == Order::lse_use(0)) asm volatile("" : "+v"(rl[0]));  // (the row values that this wait covers)
      if constexpr (m == Order::lse_use(1)) asm volatile("" : "+v"(rl[1]));
      if constexpr (m == Order::lse_use(2)) asm volatile("" : "+v"(rl[2]));
      if constexpr (m == Order::lse_use(3)) asm volatile("" : "+v"(rl[3]));
      if constexpr (m == Order::d_use()) {
        asm volatile("" : "+v"(rd[0]), "+v"(rd[1]), "+v"(rd[2]), "+v"(rd[3]));
#pragma unroll
        for (int i = 0; i < 16; ++i) rd16[i] = rd[i >> 2][i & 3];
      }
      if constexpr (m == Order::EXP0) {  // scores that a query does not see, and whole stages past the end of the walk
        const bool valid = g < n_iter;
        if (__builtin_expect(!valid || s_qt * BM < jrel_hi, 0)) {
          const int lane = lane_id();
          const int lim0 = valid ? jrel - s_qt * BM + (lane & 31) - 4 * (lane >> 5) : 0x40000000, lim1 = lim0 + 32;
          const float none = -INFINITY;
          asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s[0]), "+v"(s[1]));  // S(g) has been written
          // (a compare and a select at a time: 32 masks at once take scalar registers that the steps then miss)
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
            static_for<0, 16>([&](auto i_c) __attribute__((always_inline)) {
              constexpr int i = decltype(i_c)::value;
              float x = s[kb][i];
              const int lim = kb ? lim1 : lim0;
              asm volatile("v_cmp_lt_i32 vcc, %1, %2\n\ts_nop 1\n\tv_cndmask_b32 %0, %0, %3, vcc" : "+v"(x) : "n"(8 * (i >> 2) + (i & 3)), "v"(lim), "v"(none) : "vcc");
              s[kb][i] = x;
            });
        }
      }
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's Q rows)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < DK) fr[mm % RING] = load_rows(c_ev, c_od, std::integral_constant<int, mm>{}, in_q);
        else if constexpr (mm < 2 * DK) fr[mm % RING] = load_t(p_lo, p_hi, std::integral_constant<int, mm - DK>{}, in_q);
        else if constexpr (mm < 3 * DK) fr[mm % RING] = load_rows(c_ev, c_od, std::integral_constant<int, mm - 2 * DK>{}, in_do);
        else if constexpr (mm < NF) fr[mm % RING] = load_t(c_lo, c_hi, std::integral_constant<int, mm - 3 * DK>{}, in_do);
        else fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{}, in_q);
      }
      const bf16x8 fa = fr[m % RING];
      auto mma = [&](auto kb_c) __attribute__((always_inline)) {
        constexpr int kb = decltype(kb_c)::value;
        const bf16x8& a_ = fa;  // (named references: variables used only inside an asm statement are not captured)
        if constexpr (m < DK) {
          f32x16& d_ = s[kb];
          const bf16x8& b_ = kf[kb][m];
          if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "v"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "v"(b_));
        } else if constexpr (m < 2 * DK) {
          constexpr int ks = (m - DK) / DB, db = (m - DK) % DB;
          dk[kb][db] = mfma32(fa, __builtin_bit_cast(bf16x8, sw[kb][ks]), dk[kb][db]);
        } else if constexpr (m < 3 * DK) {
          constexpr int ks = m - 2 * DK;
          f32x16& d_ = dp[kb];
          const bf16x8& b_ = vf[kb][ks];
          const f32x16& c_ = rd16;
          if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d_) : "v"(a_), "v"(b_), "v"(c_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "v"(b_));
        } else {
          constexpr int ks = (m - 3 * DK) / DB, db = (m - 3 * DK) % DB;
          dv[kb][db] = mfma32(fa, __builtin_bit_cast(bf16x8, pw[kb][ks]), dv[kb][db]);
        }
      };
      // exponentials, then pairs packed one element late (an exponential cannot be used by the next instruction)
      constexpr int e0 = Order::exps(m - 1), e1 = Order::exps(m), em = e0 + (e1 - e0 + 1) / 2;
      constexpr int n0 = Order::dss(m - 1), n1 = Order::dss(m), nm = n0 + (n1 - n0 + 1) / 2;
      constexpr int l0 = Order::dss(m + NF - 1), l1 = Order::dss(m + NF), lm = l0 + (l1 - l0 + 1) / 2;  // of the stage before
      mma(std::integral_constant<int, 0>{});
      if constexpr (m >= Order::EXP0) {
        static_for<e0, em>(exp_one);
        static_for<(e0 > 0 ? (e0 - 1) / 2 : 0), (em > 0 ? (em - 1) / 2 : 0)>(pack_p);
        if constexpr (m >= Order::DS0) static_for<n0, nm>(ds_one);
      } else {
        static_for<l0, lm>(ds_one);
      }
      static_for<0, 4>([&](auto q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(q_c)::value;
        if constexpr (m == Order::lse_read(q)) rl[q] = lds_asm_read16f<32 * q>(r_cur);
        if constexpr (m == Order::d_use() - AHEAD - 2 + q / 2) rd[q] = lds_asm_read16f<D_ROWS + 32 * q>(r_cur);
      });
      __builtin_amdgcn_sched_barrier(0);
      mma(std::integral_constant<int, 1>{});
      if constexpr (m >= Order::EXP0) {
        static_for<em, e1>(exp_one);
        static_for<(em > 0 ? (em - 1) / 2 : 0), (e1 == 32 && e0 < 32 ? 16 : e1 > 0 ? (e1 - 1) / 2 : 0)>(pack_p);
        if constexpr (m >= Order::DS0) static_for<nm, n1>(ds_one);
      } else {
        static_for<lm, l1>(ds_one);
      }
      if constexpr (m == Order::d_use() + 1) asm volatile("" ::"v"(rd16));  // (its registers stay: the first MFMAs of dP read them late)
      if constexpr (m == 1) dma_rows();
      if constexpr (m % COPY_EVERY == COPY_EVERY - 3) dma_piece(m / COPY_EVERY);
      if constexpr (m == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        dma_advance();
        s_cur = s_nxt;
        if (--s_heads == 0) {
          s_heads = G;
          s_qt += down ? -1 : 1;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // stage g + 2 must have landed; the copies of the DIST - 2 stages after it may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 2) * PER) : "memory");
    wg_barrier();
  };
  // the last product is dK^T of stage n - 1 in step n
  const int claim_at = max(0, n_iter - 2);  // the step before which wave 0 claims the next block
  for (int g = 0; g <= n_iter; ++g) {
    if (g == claim_at && wave == 0 && mine == kClaimBlocks) pending_claim = block_claim_issue(fresh(args).taken, xcd);
    step(g);
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  // every copy of this wave has landed: once all waves have met at the barrier that hands out the next block, the ring may be filled again
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)

  {
    const DkvParams p = fresh(args);
    const int64_t kv_stride = (int64_t)p.num_kv_heads * D;
    if (!p.accumulate && !p.out_f32) {
      wg_barrier();  // nobody reads the ring any more
      lds_bf16* const stage = L + wave * (64 * D);
      const int64_t off = ((int64_t)it.kv_row0 + 64 * wave) * kv_stride + (int64_t)kvh * D;
      store_key_rows<D, 2>(stage, dv, 1.0f, p.dv + off, kv_stride, it.kv_rows - 64 * wave);
      store_key_rows<D, 2>(stage, dk, p.scale, p.dk + off, kv_stride, it.kv_rows - 64 * wave);
    } else {
    const int lane = lane_id(), l32 = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int kr = 64 * wave + 32 * kb + l32;
      if (kr < it.kv_rows) {
        const int64_t off = ((int64_t)it.kv_row0 + kr) * kv_stride + (int64_t)kvh * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int64_t e = off + 32 * db + 8 * g + 4 * hh;
            dkv_store4(p, p.dv, e, dv[kb][db][4 * g], dv[kb][db][4 * g + 1], dv[kb][db][4 * g + 2], dv[kb][db][4 * g + 3]);
            dkv_store4(p, p.dk, e, dk[kb][db][4 * g] * p.scale, dk[kb][db][4 * g + 1] * p.scale, dk[kb][db][4 * g + 2] * p.scale,
                       dk[kb][db][4 * g + 3] * p.scale);
          }
      }
    }
    }
  }
  if (mine != kClaimBlocks) break;
  // on to the next block; the stores of the epilogue are not waited for here
  int nb = 0;
  if (wave == 0) {
    const DkvParams p = fresh(args);
    if (p.side_by_side != 0 && lane_id() == 0) __hip_atomic_fetch_add(p.ended + (blk & 7), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    nb = block_claim_finish(p.taken, p.num_blocks, xcd, pending_claim);
    start_in_step(p, nb);
  }
  blk = broadcast_from_wave0(next_block, nb);
  }
  clock_log_stamp(fresh(args).clock_log, 1);
}

// ------------------------------------------------------------------------------------------------
// bwd_dkv_narrow_pipe (head_dim 64)
//
// With half the head dimension a wave has the registers for all four contractions of its 64 keys (K and V fragments, dK^T and
// dV^T accumulators: 192 accumulation registers), so there are no wave roles and no hand-over: a workgroup is two waves,
// 128 keys, two workgroups per CU, one wave per SIMD.  Stage n is the n-th (head, 32-row query tile) of the walk, as in
// dkv_pipe_blocks; in step g a wave runs
//     dP(g) = dO V^T     dV^T += dO^T P(g-1)     dK^T += Q^T dS(g-1)     S(g+1) = Q K^T        (matrix pipe)
//     P(g) = exp2(S(g) c - LSE)  and, once dP(g) is complete,  dS(g) = P(g) (dP(g) - D)         (vector)
// as 16 mini-steps of one LDS operand fragment and the two MFMAs it feeds (one per 32-key block), each MFMA followed by its
// share of the vector work.  Stages live in a ring of DIST + 3 slots (3 in use, DIST on their way).  Scores that a query
// does not see, and whole stages past the end of the walk, are set to -inf in a rarely taken branch before their step.
// The step is bound by what a single wave can issue: 32 MFMAs hold the matrix pipe for 1024 cycles, next to about 770
// cycles of vector work and 32 LDS reads.  Against bwd_dkv_kernel (32 keys per wave, two roles, one MFMA per fragment):
// packed 64K chunk, 32/8 heads, 6.28 -> 3.99 ms.
// ------------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(128, 1) void bwd_dkv_narrow_pipe_kernel(DkvParams p, int num_blocks) {
  constexpr int NW = 2;        // waves
  constexpr int BM = 32;       // query rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per operand row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dK^T / dV^T
  constexpr int QT = BM * D;   // elements per operand tile
  constexpr int DIST = 3;      // stages copied ahead
  constexpr int NS = DIST + 3; // ring slots: stages g - 1 .. g + 1 in use, g + 2 .. g + 1 + DIST on their way
  constexpr int NF = 2 * DK + 4 * DB;  // fragments (mini-steps) per step: dO rows, dO^T, Q^T, Q rows
  constexpr int T0 = DK, T1 = DK + 4 * DB;  // of which transposed
  constexpr int AHEAD = 4, RING = 8;   // fragments in flight, registers of the fragment ring
  constexpr int NP = BM * KC / 64;     // 64-slot pieces per tile
  constexpr int PER = 2 * NP / NW;     // pieces per wave and stage
  constexpr int CPS = PER + 1;         // copies per wave and stage: its pieces and one set of row values (LSE or D)
  constexpr int RV = 64;               // floats per slot of the LSE / D rows (32 used; a whole wave copies them)
  constexpr int EXP0 = 0, EXP1 = 9, DS0 = 7;  // mini-steps of the vector work (spread); dP(g) is complete after mini-step 3
  constexpr int D_READ = 2, LSE_READ = NF - 3;  // mini-steps that read the D rows of this stage / the LSE rows of the next
  constexpr int BOOK = NF - 2;
  static_assert(D == 64 && NF == 16 && NF % RING == 0 && PER % 2 == 0 && 3 + 2 * PER < BOOK, "the schedule of a step");
  // LDS instructions issued between the read of fragment m and the start of mini-step m (fragment_wait and the row values)
  auto lds_wait = [](int m) constexpr {
    int n = fragment_wait(NF, T0, T1, m);
    for (int i = m - 4; i < m; ++i) {
      const int k = (i + NF) % NF;
      if (k == D_READ || k == LSE_READ) n += 4;
    }
    return m == 0 && n > 2 ? 2 : n;  // mini-step 0 also waits for the LSE rows: two fragments have been read since
  };
  static_assert(LSE_READ == NF - 3 && DS0 >= D_READ + 5, "the row values have arrived when they are first used");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int Q_OFF = 0;                 // [NS][QT]  Q rows of stage n in slot n % NS (chunk-major)
  constexpr int G_OFF = Q_OFF + NS * QT;   // [NS][QT]  dO rows
  constexpr int R_OFF = G_OFF + NS * QT;   // [NS][RV] floats LSE rows, then [NS][RV] floats D rows
  lds_f32* const lse_s = (lds_f32*)(L + R_OFF);
  lds_f32* const dsum_s = lse_s + NS * RV;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;

  // Persistent, as dkv_pipe_blocks.
  __shared__ int next_block;
  const int xcd = xcd_of_this_wave();
  int blk = 0;
  if (wave == 0) blk = block_claim_finish(p.taken, num_blocks, xcd, block_claim_issue(p.taken, xcd));
  blk = broadcast_from_wave0(&next_block, blk);
  while (blk >= 0) {
  const int kvh = blk % p.num_kv_heads;
  const DkvItem it = p.items[blk / p.num_kv_heads];
  const int G = p.group;
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const float c = p.scale_log2;

  // the slots the prologue does not fill: slot NS - 1 (stage -1) is read in step 0
  {
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    for (int x = tid; x < (NS - DIST - 1) * QT / 8; x += NW * 64) {
      lds_store8(L + Q_OFF + (DIST + 1) * QT + x * 8, z);
      lds_store8(L + G_OFF + (DIST + 1) * QT + x * 8, z);
    }
  }

  const int nqt = it.n_qt - it.qt_first;
  const int n_iter = nqt * G;

  // ---- staging (see dkv_pipe_blocks): copy i of a wave is piece (i % (PER / 2)) * 2 + wave of Q (i < PER / 2) or of dO ----
  unsigned v_full[PER / 2], v_last[PER / 2];
  {
    const int last_row = it.q_len - 1 - (it.n_qt - 1) * BM;
#pragma unroll
    for (int i = 0; i < PER / 2; ++i) {
      const int x = (i * NW + wave) * 64 + lane;
      const int off = (x >> 5) * 8, row = (x & 31) ^ (((x >> 5) & 3) << 2);
      v_full[i] = (unsigned)(row * (int)q_stride + off) * 2u;
      v_last[i] = (unsigned)(min(row, last_row) * (int)q_stride + off) * 2u;
    }
  }
  const bool down = it.reverse != 0;
  const int qt_start = down ? it.n_qt - 1 : it.qt_first;
  const int64_t roff0 = (int64_t)(it.q_row_seg + qt_start * BM) * q_stride + (int64_t)(kvh * G) * D;
  const int64_t rv_first = ((int64_t)(kvh * G) * p.total_q_tiles + it.q_tile0) * 64 + qt_start * BM;
  const char* d_q = reinterpret_cast<const char*>(p.q + roff0);
  const char* d_g = reinterpret_cast<const char*>(p.d_o + roff0);
  const char* d_r = reinterpret_cast<const char*>((wave ? p.dsp : p.lse2p) + rv_first);
  const int64_t head_bytes = (int64_t)D * 2;
  const int64_t head_rows_bytes = p.total_q_tiles * 64 * 4;
  const int64_t tile_bytes = (down ? -1 : 1) * (int64_t)BM * q_stride * 2 - (G - 1) * head_bytes;
  const int64_t tile_rows_bytes = (down ? -1 : 1) * (int64_t)BM * 4 - (G - 1) * head_rows_bytes;
  int d_heads = G, d_tiles = nqt;
  const int d_ragged = down ? nqt : 1;
  unsigned d_slot = 0;  // element offset of the ring slot inside the Q / dO rings (slot index x QT)
  const unsigned lane4 = (unsigned)lane * 4u;
  lds_f32* const rows_dst = wave ? dsum_s : lse_s;
  auto dma_rows = [&]() __attribute__((always_inline)) { dma4(d_r + lane4, rows_dst + d_slot / (QT / RV)); };
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const bool of_q = i < PER / 2;
    const int k = i % (PER / 2);
    const unsigned voff = d_tiles == d_ragged ? v_last[k] : v_full[k];
    lds_bf16* dst = L + (of_q ? Q_OFF : G_OFF) + (k * NW + wave) * 512 + d_slot;
    dma16((of_q ? d_q : d_g) + voff, dst);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_heads > 1) {
      --d_heads;
      d_q += head_bytes; d_g += head_bytes; d_r += head_rows_bytes;
    } else {  // on to the next query tile; after the last stage, stay on it
      const bool more = d_tiles > 1;
      d_tiles -= more ? 1 : 0;
      d_heads = more ? G : 1;
      const int64_t tb = more ? tile_bytes : 0, tr = more ? tile_rows_bytes : 0;
      d_q += tb; d_g += tb; d_r += tr;
    }
    d_slot = d_slot == (unsigned)((NS - 1) * QT) ? 0u : d_slot + (unsigned)QT;
  };

  // byte addresses of this lane's operand reads inside slot 0 of the Q ring; the dO ring is a constant further
  unsigned ev0, od0, lo0, hi0;
  {
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    ev0 = lds_addr(L + Q_OFF + cm_elem(l32, hh));
    od0 = lds_addr(L + Q_OFF + cm_elem(l32, 2 + hh));
    lo0 = lds_addr(L + Q_OFF + cm_elem(r0, cl) + 4 * (j & 1));
    hi0 = lds_addr(L + Q_OFF + cm_elem(r0 + 8, cl) + 4 * (j & 1));
  }
  const unsigned lse0 = lds_addr(lse_s + 4 * hh);
  constexpr unsigned SLOT = QT * 2;               // bytes per ring slot
  constexpr int DO_RING = (G_OFF - Q_OFF) * 2;    // bytes from the Q ring to the dO ring
  constexpr int D_ROWS = NS * RV * 4;             // bytes from the LSE rows to the D rows
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c, auto ring_c) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value;
    constexpr int off = (ks >> 1) * (4 * 32 * 8) * 2 + decltype(ring_c)::value;
    return lds_asm_read16<off>((ks & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c, auto ring_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2 + decltype(ring_c)::value;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  constexpr std::integral_constant<int, 0> in_q{};
  constexpr std::integral_constant<int, DO_RING> in_do{};

  // K and V fragments (B operands): lane holds X[key = 64 wave + 32 kb + l32][16 ks + 8 hh ..+7]
  bf16x8 kf[2][DK], vf[2][DK];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int64_t grow = it.kv_row0 + min(64 * wave + 32 * kb + l32, it.kv_rows - 1);
    const int64_t off = grow * kv_stride + (int64_t)kvh * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      kf[kb][ks] = *reinterpret_cast<const bf16x8*>(p.k + off + 16 * ks);
      vf[kb][ks] = *reinterpret_cast<const bf16x8*>(p.v + off + 16 * ks);
    }
  }
  // prologue: the copies of stages 0 .. DIST
#pragma unroll
  for (int s = 0; s <= DIST; ++s) {
    dma_rows();
#pragma unroll
    for (int i = 0; i < PER; ++i) dma_piece(i);
    dma_advance();
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0), visible to the compiler
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dk[2][DB], dv[2][DB];  // dK^T, dV^T: [D] x [32 keys of block kb]
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int db = 0; db < DB; ++db) dk[kb][db] = dv[kb][db] = zero16;
  f32x16 x[2][2];       // S: [buffer][key block]
  f32x16 dp[2];         // dP: [key block]
  bf16x8 fp[2][2][2], fs[2][2][2];  // P and dS as B operands: [buffer][key block][k-step]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) fp[b][kb][ks][i] = fs[b][kb][ks][i] = (__bf16)0.0f;
  bf16x8 fr[RING];
  f32x4 rl[4], rd[4];   // LSE and -D of rows 8 g4 + 4 hh + 0..3

  // S(0), then the LSE rows of stage 0 and the first fragments of step 0 (dO rows of stage 0)
  {
    bf16x8 a[DK];
    static_for<0, DK>([&](auto k_c) __attribute__((always_inline)) { a[decltype(k_c)::value] = load_rows(ev0, od0, k_c, in_q); });
    static_for<0, 4>([&](auto g_c) __attribute__((always_inline)) { rl[decltype(g_c)::value] = lds_asm_read16f<32 * decltype(g_c)::value>(lse0); });
    static_for<0, AHEAD>([&](auto k_c) __attribute__((always_inline)) { fr[decltype(k_c)::value] = load_rows(ev0, od0, k_c, in_do); });
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(AHEAD) : "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(a[ks]));  // (after the wait, in this order)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) asm volatile("" : "+v"(rl[g4]));
#pragma unroll
    for (int ks = 0; ks < DK; ++ks)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        f32x16& d_ = x[0][kb];
        const bf16x8& b_ = kf[kb][ks];
        if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a[ks]), "a"(b_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a[ks]), "a"(b_));
      }
    mfma_settle();
  }

  // key index of this lane's column of block 0 relative to the context: query i of the segment sees the column of block kb
  // iff i >= jrel + 32 kb
  const int jrel = it.j0 + 64 * wave + l32 - it.ctx;
  const int jrel_hi = it.j0 + 64 * wave + 63 - it.ctx;  // of the wave's last key
  int s_cur = 0;        // slot of stage g
  int s_qt = qt_start;  // query tile of stage g
  int s_heads = G;      // heads of that tile still to come, counting stage g's

  auto step = [&](int g, f32x16 (&cur)[2], f32x16 (&nxt)[2], bf16x8 (&p_old)[2][2], bf16x8 (&p_new)[2][2], bf16x8 (&s_old)[2][2],
                  bf16x8 (&s_new)[2][2]) __attribute__((always_inline)) {
    const int s_nxt = s_cur == NS - 1 ? 0 : s_cur + 1, s_prv = s_cur == 0 ? NS - 1 : s_cur - 1;
    const unsigned c_ev = ev0 + s_cur * SLOT, c_od = od0 + s_cur * SLOT, n_ev = ev0 + s_nxt * SLOT, n_od = od0 + s_nxt * SLOT;
    const unsigned t_lo = lo0 + s_prv * SLOT, t_hi = hi0 + s_prv * SLOT;
    const unsigned r_cur = lse0 + s_cur * (RV * 4), r_nxt = lse0 + s_nxt * (RV * 4);
    // entry (query 8 (i / 4) + 4 hh + i % 4 of the tile, column of block kb) is visible iff 8 (i / 4) + i % 4 >= lim + 32 kb
    const bool valid = g < n_iter;
    if (__builtin_expect(!valid || s_qt * BM < jrel_hi, 0)) {
      const int lim = valid ? jrel - s_qt * BM - 4 * hh : 0x40000000;
      asm volatile("s_nop 15\n\ts_nop 7" : "+v"(cur[0]), "+v"(cur[1]));  // S(g) has been written
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + (i & 3) < lim + 32 * kb) cur[kb][i] = -INFINITY;
    }
    float pf[2][16];             // P(g)
    unsigned pw[2][8], sw[2][8]; // P(g), dS(g), packed pairs
    auto pack_p = [&](int j) __attribute__((always_inline)) {  // (one pair late: an exponential cannot be used by the next instruction)
      bf16x2 w;
      w[0] = (__bf16)pf[j >> 3][2 * (j & 7)]; w[1] = (__bf16)pf[j >> 3][2 * (j & 7) + 1];
      unsigned wu = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(wu));
      pw[j >> 3][j & 7] = wu;
    };
    auto exp_half = [&](auto x_c) __attribute__((always_inline)) {
      constexpr int j = decltype(x_c)::value / 2, q = decltype(x_c)::value % 2, kb = j >> 3, i = 2 * (j & 7) + q;
      if constexpr (j > 0 && q == 0) pack_p(j - 1);
      pf[kb][i] = __builtin_amdgcn_exp2f(cur[kb][i] * c - rl[i >> 2][i & 3]);
      asm volatile("" : "+v"(pf[kb][i]));
    };
    auto ds_pair = [&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, kb = j >> 3, i = 2 * (j & 7);
      bf16x2 w;
      w[0] = (__bf16)(pf[kb][i] * (dp[kb][i] + rd[i >> 2][i & 3]));
      w[1] = (__bf16)(pf[kb][i + 1] * (dp[kb][i + 1] + rd[i >> 2][(i & 3) + 1]));
      unsigned wu = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(wu));
      sw[kb][j & 7] = wu;
    };
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      if constexpr (m == 0)
        asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(fr[0]), "+v"(rl[0]), "+v"(rl[1]), "+v"(rl[2]), "+v"(rl[3]) : "n"(lds_wait(0)));
      else if constexpr (m == DS0)
        asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(fr[m % RING]), "+v"(rd[0]), "+v"(rd[1]), "+v"(rd[2]), "+v"(rd[3]) : "n"(lds_wait(m)));
      else
        asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(lds_wait(m)));
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's dO rows)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < T0) fr[mm % RING] = load_rows(c_ev, c_od, std::integral_constant<int, mm>{}, in_do);
        else if constexpr (mm < T0 + 2 * DB) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm - T0>{}, in_do);
        else if constexpr (mm < T1) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm - T0 - 2 * DB>{}, in_q);
        else if constexpr (mm < NF) fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - T1>{}, in_q);
        else fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{}, in_do);
      }
      const bf16x8 fa = fr[m % RING];
      auto mma = [&](auto kb_c) __attribute__((always_inline)) {
        constexpr int kb = decltype(kb_c)::value;
        const bf16x8& a_ = fa;  // (named references: variables used only inside an asm statement are not captured)
        if constexpr (m < T0) {
          f32x16& d_ = dp[kb];
          const bf16x8& b_ = vf[kb][m];
          if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
        } else if constexpr (m < T0 + 2 * DB) {
          constexpr int ks = (m - T0) / DB, db = (m - T0) % DB;
          dv[kb][db] = mfma32(fa, p_old[kb][ks], dv[kb][db]);
        } else if constexpr (m < T1) {
          constexpr int ks = (m - T0 - 2 * DB) / DB, db = (m - T0 - 2 * DB) % DB;
          dk[kb][db] = mfma32(fa, s_old[kb][ks], dk[kb][db]);
        } else {
          constexpr int ks = m - T1;
          f32x16& d_ = nxt[kb];
          const bf16x8& b_ = kf[kb][ks];
          if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
        }
      };
      constexpr int e0 = 2 * spread(16, EXP0, EXP1, m - 1), e1 = 2 * spread(16, EXP0, EXP1, m), em = e0 + (e1 - e0 + 1) / 2;
      constexpr int s0 = spread(16, DS0, NF, m - 1), s1 = spread(16, DS0, NF, m), sm = s0 + (s1 - s0 + 1) / 2;
      static_assert(2 * s1 <= e0 || e0 == 32, "a pair's exponentials come before its dS");
      mma(std::integral_constant<int, 0>{});
      static_for<e0, em>(exp_half);
      static_for<s0, sm>(ds_pair);
      if constexpr (m == D_READ) {
        rd[0] = lds_asm_read16f<D_ROWS>(r_cur);
        rd[1] = lds_asm_read16f<D_ROWS + 32>(r_cur);
        rd[2] = lds_asm_read16f<D_ROWS + 64>(r_cur);
        rd[3] = lds_asm_read16f<D_ROWS + 96>(r_cur);
      }
      if constexpr (m == LSE_READ) {
        rl[0] = lds_asm_read16f<0>(r_nxt);
        rl[1] = lds_asm_read16f<32>(r_nxt);
        rl[2] = lds_asm_read16f<64>(r_nxt);
        rl[3] = lds_asm_read16f<96>(r_nxt);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(std::integral_constant<int, 1>{});
      static_for<em, e1>(exp_half);
      static_for<sm, s1>(ds_pair);
      if constexpr (m == EXP1 - 1) pack_p(15);
      if constexpr (m >= 3 && m < 3 + 2 * PER && ((m - 3) & 1) == 0) dma_piece((m - 3) >> 1);
      if constexpr (m == 3 + 2 * PER) dma_rows();
      if constexpr (m == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        dma_advance();
        s_cur = s_nxt;
        if (--s_heads == 0) {
          s_heads = G;
          s_qt += down ? -1 : 1;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 pv = {pw[kb][4 * ks], pw[kb][4 * ks + 1], pw[kb][4 * ks + 2], pw[kb][4 * ks + 3]};
        const u32x4 sv = {sw[kb][4 * ks], sw[kb][4 * ks + 1], sw[kb][4 * ks + 2], sw[kb][4 * ks + 3]};
        p_new[kb][ks] = __builtin_bit_cast(bf16x8, pv);
        s_new[kb][ks] = __builtin_bit_cast(bf16x8, sv);
      }
    // stage g + 2 must have landed; the copies of the DIST - 1 stages after it may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 1) * CPS) : "memory");
    wg_barrier();
  };
  // the last products are those of stage n - 1 in step n; a pair of steps may run one past that, which contributes nothing
  int pending_claim = 0;
  const int claim_at = max(0, n_iter - 3) & ~1;  // the step pair before which wave 0 claims the next block
  for (int g = 0; g <= n_iter; g += 2) {
    if (g == claim_at && wave == 0) pending_claim = block_claim_issue(p.taken, xcd);
    step(g, x[0], x[1], fp[0], fp[1], fs[0], fs[1]);
    step(g + 1, x[1], x[0], fp[1], fp[0], fs[1], fs[0]);
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]), "+v"(rl[i]));
  // every copy of this wave has landed: once both waves have met at the barrier that hands out the next block, the ring
  // may be filled again
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)

#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int kr = 64 * wave + 32 * kb + l32;
    if (kr < it.kv_rows) {
      const int64_t off = ((int64_t)it.kv_row0 + kr) * kv_stride + (int64_t)kvh * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t e = off + 32 * db + 8 * g + 4 * hh;
          dkv_store4(p, p.dv, e, dv[kb][db][4 * g], dv[kb][db][4 * g + 1], dv[kb][db][4 * g + 2], dv[kb][db][4 * g + 3]);
          dkv_store4(p, p.dk, e, dk[kb][db][4 * g] * p.scale, dk[kb][db][4 * g + 1] * p.scale, dk[kb][db][4 * g + 2] * p.scale,
                     dk[kb][db][4 * g + 3] * p.scale);
        }
    }
  }
  // on to the next block; the stores of the epilogue are not waited for here
  int nb = 0;
  if (wave == 0) nb = block_claim_finish(p.taken, num_blocks, xcd, pending_claim);
  blk = broadcast_from_wave0(&next_block, nb);
  }
}

// ------------------------------------------------------------------------------------------------
// dkv_wide_blocks (head_dim 256): the dK/dV blocks of bwd_pipe_kernel
//
// One wave per SIMD, no wave roles, as dkv_tall_blocks: a workgroup covers 128 keys, each of its four waves all four contractions of 32 of them, whose
// accumulators fill the accumulation registers and whose K and V fragments take half of the others.  Stage n is the n-th (head, 32-row query tile) of
// the walk; step g is
//     S(g) = Q K^T     dP(g) = dO V^T - D     dV^T += dO^T P(g)     dK^T += Q^T dS(g)               (matrix pipe, in this order)
//     P(g) = exp2(S(g) c - LSE)  until dV^T needs it,  dS(g) = P(g) dP(g)  until dK^T needs it        (vector)
// as 64 mini-steps of one LDS operand fragment and the MFMA it feeds.  There is half the vector work per MFMA of head_dim 128, so that it fits under the
// products of dP and dV, and nothing but fragments lives from one step to the next: a stage leaves LDS with its step, and four slots of Q and dO
// are enough for copies to have a step to land.  P stays in float32 for dS.
// A step is bound by its LDS reads (96, and 8 of row values, 16 cycles each to issue; the CU reads 256 KB of LDS per step): its 64 MFMAs take 2048 of 2680 cycles,
// at 1.74 GHz.  Against two score waves that handed P and dS to two gradient waves, for 64 keys, in a launch behind that of dQ: packed
// 64K chunk, 32/8 heads, forward and backward, 35.3 -> 32.0 ms; backward of 7307 causal tokens 3.6 -> 2.5.
// ------------------------------------------------------------------------------------------------
// The schedule of a step, as TallOrder.
template <int DK, int AHEAD>
struct WideOrder {
  static constexpr int NF = 4 * DK;
  static constexpr int EXP0 = DK + 3, DS0 = 2 * DK + 3;
  static constexpr int cost(int k) { return (k % NF) / DK >= 2 ? 2 : 1; }
  static constexpr int exps(int m) { return spread(16, EXP0, 2 * DK + 5, m); }  // scores done by the end of mini-step m
  static constexpr int dss(int m) { return spread(16, DS0, 3 * DK + 5, m); }
  static constexpr int lse_use(int quad) {  // first mini-step that needs the LSE of rows 8 quad + 4 hh ..+3
    int m = EXP0;
    while (exps(m) <= 4 * quad) ++m;
    return m;
  }
  static constexpr int lse_read(int quad) { return lse_use(quad) - AHEAD - 1; }
  static constexpr int d_use() { return DK; }  // the -D tile
  static constexpr int d_read(int quad) { return DK - AHEAD - 4 + quad; }
  static constexpr int extra(int m) {
    int n = 0;
    for (int q = 0; q < 4; ++q) n += (lse_read(q) == m ? 1 : 0) + (d_read(q) == m ? 1 : 0);
    return n;
  }
  static constexpr int wait(int m) {
    int n = extra((m - AHEAD + NF) % NF);
    for (int i = m - AHEAD + 1; i < m; ++i) n += cost((i + AHEAD + NF) % NF) + extra((i + NF) % NF);
    return n;
  }
  static_assert(exps(2 * DK - 1) >= 9 && exps(2 * DK + DK / 2 - 1) == 16 && dss(3 * DK - 1) >= 8 && dss(3 * DK + DK / 2 - 1) == 16, "the order of a step");
};
template <int D>
__device__ __forceinline__ void dkv_wide_blocks(const ArgsPtr<DkvParams> args, const int mine) {
  constexpr int NW = 4;        // waves
  constexpr int BM = 32;       // query rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per operand row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dK^T / dV^T
  constexpr int QT = BM * D;   // elements per operand tile
  constexpr int DIST = 3;      // stages copied ahead
  constexpr int NS = DIST + 1; // ring slots: stage g in use, g + 1 .. g + DIST on their way
  constexpr int NF = 4 * DK;   // fragments (mini-steps) per step: Q rows, dO rows, dO^T, Q^T
  constexpr int AHEAD = 6, RING = 8;   // fragments in flight, names of the fragment ring
  constexpr int NP = BM * KC / 64;     // 64-slot pieces per tile
  constexpr int PER = 2 * NP / NW;     // pieces per wave and stage
  constexpr int RV = 64;               // floats per slot of the LSE / D rows (32 used; a whole wave copies them)
  constexpr int BOOK = NF - 2;
  using Order = WideOrder<DK, AHEAD>;
  constexpr int COPY_EVERY = NF / PER;  // mini-steps from one copy of a stage to the next
  static_assert(D == 256 && NF % RING == 0 && 2 * DB == DK && NF % PER == 0 && NF - 3 <= BOOK, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int R_OFF = NS * 2 * QT;       // slot n % NS holds stage n: [QT] Q rows, then [QT] dO rows (chunk-major); behind the ring
  lds_f32* const lse_s = (lds_f32*)(L + R_OFF);   // [NS][RV] LSE rows, then [NS][RV] D rows
  lds_f32* const dsum_s = lse_s + NS * RV;
  int* const next_block = (int*)((__bf16*)smem + R_OFF + 2 * NS * RV * 2);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the lane is counted anew where it is needed: held in registers, it and what follows from it would take those of the steps)
  auto lane_id = []() __attribute__((always_inline)) {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
  };

  // Persistent, as dkv_pipe_blocks.
  const int xcd = xcd_of_this_wave();
  clock_log_stamp(fresh(args).clock_log, 0);
  int blk = mine;
  if (mine == kClaimBlocks) {
    if (wave == 0) {
      const DkvParams p = fresh(args);
      blk = block_claim_finish(p.taken, p.num_blocks, xcd, block_claim_issue(p.taken, xcd));
    }
    blk = broadcast_from_wave0(next_block, blk);
  }
  while (blk >= 0) {
  int pending_claim = 0;
  const DkvParams p = fresh(args);
  const int kvh = blk % p.num_kv_heads;
  const DkvItem it = load_uniform(p.items, blk / p.num_kv_heads);
  const int G = p.group;
  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const float c = p.scale_log2;

  const int nqt = it.n_qt - it.qt_first;
  const int n_iter = nqt * G;

  // ---- staging (see dkv_pipe_blocks): copy i of a wave is piece i * 4 + wave of the stage's 2 NP, those of Q first; waves 0 and 1 also copy the
  // stage's LSE and D rows.  Rows past the segment's last query repeat it (their P is 0) ----
  // (piece p is chunks 2 p and 2 p + 1 of the rows; p is odd for all copies of a wave or for none, so that they share their rows' order)
  unsigned v_off;  // byte offset of the lane's chunk of piece 0 or 1 from the tile's first row, but for the piece's own 32 bytes
  const int last_row = it.q_len - 1 - (it.n_qt - 1) * BM;
  auto set_offsets = [&](int max_row) __attribute__((always_inline)) {
    const int lane = lane_id(), hh = lane >> 5, row = (lane & 31) ^ ((2 * (wave & 1) + hh) << 2);
    v_off = (unsigned)(min(row, max_row) * (int)q_stride + 8 * hh) * 2u;
  };
  const bool down = it.reverse != 0;
  const int qt_start = down ? it.n_qt - 1 : it.qt_first;
  const int64_t roff0 = (int64_t)(it.q_row_seg + qt_start * BM) * q_stride + (int64_t)(kvh * G) * D;
  const int64_t rv_first = ((int64_t)(kvh * G) * p.total_q_tiles + it.q_tile0) * 64 + qt_start * BM;
  const char* d_q = reinterpret_cast<const char*>(p.q + roff0);
  const char* d_g = reinterpret_cast<const char*>(p.d_o + roff0);
  const char* d_r = reinterpret_cast<const char*>((wave & 1 ? p.dsp : p.lse2p) + rv_first);
  const int64_t head_bytes = (int64_t)D * 2;
  const int64_t head_rows_bytes = p.total_q_tiles * 64 * 4;
  const int64_t tile_bytes = (down ? -1 : 1) * (int64_t)BM * q_stride * 2 - (G - 1) * head_bytes;
  const int64_t tile_rows_bytes = (down ? -1 : 1) * (int64_t)BM * 4 - (G - 1) * head_rows_bytes;
  int d_heads = G, d_tiles = nqt;
  const int d_ragged = down ? nqt : 1;  // d_tiles while the segment's last query tile is the one to copy
  unsigned d_slot = 0;
  lds_f32* const rows_dst = wave & 1 ? dsum_s : lse_s;
  set_offsets(d_tiles == d_ragged ? last_row : BM - 1);
  auto dma_rows = [&]() __attribute__((always_inline)) {
    if (wave < 2) dma4(d_r + (unsigned)lane_id() * 4u, rows_dst + d_slot * RV);
  };
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const int piece = i * NW + wave;
    const bool of_q = NP % NW == 0 ? i < NP / NW : piece < NP;
    asm volatile("" : "+v"(v_off));  // (widened here, not in registers held for it)
    dma16((of_q ? d_q + piece * 32 : d_g + (piece - NP) * 32) + v_off, L + d_slot * (2 * QT) + piece * 512);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_heads > 1) {
      --d_heads;
      d_q += head_bytes; d_g += head_bytes; d_r += head_rows_bytes;
    } else {  // on to the next query tile; after the last stage, stay on it
      const bool more = d_tiles > 1;
      d_tiles -= more ? 1 : 0;
      d_heads = more ? G : 1;
      const int64_t tb = more ? tile_bytes : 0, tr = more ? tile_rows_bytes : 0;
      d_q += tb; d_g += tb; d_r += tr;
      if (__builtin_expect(more && (d_tiles == d_ragged || d_tiles + 1 == d_ragged), 0)) set_offsets(d_tiles == d_ragged ? last_row : BM - 1);
    }
    d_slot = d_slot == NS - 1 ? 0u : d_slot + 1;
  };

  // byte addresses of this lane's operand reads in the Q tile of slot 0; the dO tile is a constant further
  // (odd k-steps: chunk 2 + hh instead of hh is 1024 bytes further with bit 3 of the row turned over; rows r0 + 8: the same bit)
  constexpr unsigned ROW8 = 8 * 16;
  unsigned ev0, lo0, lse0;
  {
    const int lane = lane_id(), l32 = lane & 31, hh = lane >> 5;
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    ev0 = lds_addr(L + cm_elem(l32, hh));
    lo0 = lds_addr(L + cm_elem(r0, cl) + 4 * (j & 1));
    lse0 = lds_addr(lse_s + 4 * hh);
  }
  constexpr unsigned SLOT = 2 * QT * 2;           // bytes per ring slot
  constexpr int DO_TILE = QT * 2;                 // bytes from the Q tile to the dO tile
  constexpr int D_ROWS = NS * RV * 4;             // bytes from the LSE rows to the D rows
  auto load_rows = [&](unsigned ev_addr, unsigned od_addr, auto ks_c, auto tile_c) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_c)::value;
    constexpr int off = (ks >> 1) * (4 * 32 * 8) * 2 + (ks & 1) * 1024 + decltype(tile_c)::value;
    return lds_asm_read16<off>((ks & 1) ? od_addr : ev_addr);
  };
  auto load_t = [&](unsigned lo_addr, unsigned hi_addr, auto m_c, auto tile_c) __attribute__((always_inline)) {
    constexpr int m = decltype(m_c)::value;  // ks2 * DB + db
    constexpr int off = ((m / DB) * (16 * 8) + (m % DB) * (4 * 32 * 8)) * 2 + decltype(tile_c)::value;
    const s16x4 lo = lds_asm_read_tr<off>(lo_addr);
    const s16x4 hi = lds_asm_read_tr<off>(hi_addr);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  constexpr std::integral_constant<int, 0> in_q{};
  constexpr std::integral_constant<int, DO_TILE> in_do{};

  // K and V fragments (B operands): lane holds X[key = 32 wave + l32][16 ks + 8 hh ..+7]
  bf16x8 kf[DK], vf[DK];
  {
    const int lane = lane_id();
    const int64_t grow = it.kv_row0 + min(32 * wave + (lane & 31), it.kv_rows - 1);
    const int64_t off = grow * kv_stride + (int64_t)kvh * D + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8*>(p.k + off + 16 * ks);
      vf[ks] = *reinterpret_cast<const bf16x8*>(p.v + off + 16 * ks);
    }
  }
  // prologue: the copies of stages 0 .. DIST - 1
#pragma unroll
  for (int s = 0; s < DIST; ++s) {
    dma_rows();
#pragma unroll
    for (int i = 0; i < PER; ++i) dma_piece(i);
    dma_advance();
  }
  // stages 0 and 1 have landed (a wait the compiler can see, for the fragments).  (Waves 0 and 1 have a copy more per stage and wait for up to
  // DIST - 2 copies more than they need; so do the waits at the end of a step.)
  wait_all_but<(DIST - 2) * PER>();
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dk[1][DB], dv[1][DB];  // dK^T, dV^T: [D] x [32 keys]
#pragma unroll
  for (int db = 0; db < DB; ++db) dk[0][db] = dv[0][db] = zero16;
  f32x16 s, dp;           // S, then P, and dP - D
  u32x4 pw[2], sw[2];     // P and dS as B operands: [k-step], pairs of bf16
  bf16x8 fr[RING];
  static_for<0, AHEAD>([&](auto k_c) __attribute__((always_inline)) { fr[decltype(k_c)::value] = load_rows(ev0, ev0 ^ ROW8, k_c, in_q); });

  // index of the wave's first key relative to the context: query i of the segment sees the column of this lane iff i >= jrel + l32
  const int jrel = it.j0 + 32 * wave - it.ctx;
  int s_cur = 0;        // slot of stage g
  int s_qt = qt_start;  // query tile of stage g
  int s_heads = G;      // heads of that tile still to come, counting stage g's

  auto step = [&]() __attribute__((always_inline)) {
    const int s_nxt = s_cur == NS - 1 ? 0 : s_cur + 1;
    const unsigned c_ev = ev0 + s_cur * SLOT, c_od = c_ev ^ ROW8, n_ev = ev0 + s_nxt * SLOT, n_od = n_ev ^ ROW8;
    const unsigned c_lo = lo0 + s_cur * SLOT, c_hi = c_lo ^ ROW8;
    const unsigned r_cur = lse0 + s_cur * (RV * 4);
    f32x4 rl[4];          // LSE of rows 8 g4 + 4 hh + 0..3
    f32x4 rd[4];          // -D of the same rows
    f32x16 rd16;
    float e_hold;         // the first exponential (or dS) of a pair, until the second one is there
    auto exp_one = [&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value;
      float e = __builtin_amdgcn_exp2f(s[i] * c - rl[i / 4][i & 3]);
      asm volatile("" : "+v"(e));
      s[i] = e;
    };
    auto pack_p = [&](auto w_c) __attribute__((always_inline)) {  // pair w: scores 2 w and 2 w + 1
      constexpr int w = decltype(w_c)::value;
      bf16x2 v;
      v[0] = (__bf16)s[2 * w]; v[1] = (__bf16)s[2 * w + 1];
      unsigned u = __builtin_bit_cast(unsigned, v);
      asm volatile("" : "+v"(u));
      pw[w / 4][w % 4] = u;
    };
    auto ds_one = [&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value, w = i / 2;
      float e = s[i] * dp[i];
      if constexpr (i % 2 == 0) {
        asm volatile("" : "+v"(e));
        e_hold = e;
      } else {
        bf16x2 v;
        v[0] = (__bf16)e_hold; v[1] = (__bf16)e;
        unsigned u = __builtin_bit_cast(unsigned, v);
        asm volatile("" : "+v"(u));
        sw[w / 4][w % 4] = u;
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      constexpr int lgkm = Order::wait(m);
      static_assert(lgkm >= 0 && lgkm <= 15, "lgkmcnt is a 4-bit counter");
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(lgkm));
      if constexpr (m == Order::lse_use(0)) asm volatile("" : "+v"(rl[0]));  // (the row values that this wait covers)
      if constexpr (m == Order::lse_use(1)) asm volatile("" : "+v"(rl[1]));
      if constexpr (m == Order::lse_use(2)) asm volatile("" : "+v"(rl[2]));
      if constexpr (m == Order::lse_use(3)) asm volatile("" : "+v"(rl[3]));
      if constexpr (m == Order::d_use()) {
        asm volatile("" : "+v"(rd[0]), "+v"(rd[1]), "+v"(rd[2]), "+v"(rd[3]));
#pragma unroll
        for (int i = 0; i < 16; ++i) rd16[i] = rd[i >> 2][i & 3];
      }
      if constexpr (m == Order::EXP0) {  // scores that a query does not see
        if (__builtin_expect(s_qt * BM < jrel + 31, 0)) {
          const int lane = lane_id();
          const int lim = jrel - s_qt * BM + (lane & 31) - 4 * (lane >> 5);
          const float none = -INFINITY;
          asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s));  // S(g) has been written
          // (a compare and a select at a time: 16 masks at once take scalar registers that the steps then miss)
          static_for<0, 16>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            float x = s[i];
            asm volatile("v_cmp_lt_i32 vcc, %1, %2\n\ts_nop 1\n\tv_cndmask_b32 %0, %0, %3, vcc" : "+v"(x) : "n"(8 * (i >> 2) + (i & 3)), "v"(lim), "v"(none) : "vcc");
            s[i] = x;
          });
        }
      }
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's Q rows)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < DK) fr[mm % RING] = load_rows(c_ev, c_od, std::integral_constant<int, mm>{}, in_q);
        else if constexpr (mm < 2 * DK) fr[mm % RING] = load_rows(c_ev, c_od, std::integral_constant<int, mm - DK>{}, in_do);
        else if constexpr (mm < 3 * DK) fr[mm % RING] = load_t(c_lo, c_hi, std::integral_constant<int, mm - 2 * DK>{}, in_do);
        else if constexpr (mm < NF) fr[mm % RING] = load_t(c_lo, c_hi, std::integral_constant<int, mm - 3 * DK>{}, in_q);
        else fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{}, in_q);
      }
      const bf16x8 fa = fr[m % RING];
      if constexpr (m < DK) {
        if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(fa), "v"(kf[m]));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(fa), "v"(kf[m]));
      } else if constexpr (m < 2 * DK) {
        constexpr int ks = m - DK;
        if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(dp) : "v"(fa), "v"(vf[ks]), "v"(rd16));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(dp) : "v"(fa), "v"(vf[ks]));
      } else if constexpr (m < 3 * DK) {
        constexpr int ks = (m - 2 * DK) / DB, db = (m - 2 * DK) % DB;
        dv[0][db] = mfma32(fa, __builtin_bit_cast(bf16x8, pw[ks]), dv[0][db]);
      } else {
        constexpr int ks = (m - 3 * DK) / DB, db = (m - 3 * DK) % DB;
        dk[0][db] = mfma32(fa, __builtin_bit_cast(bf16x8, sw[ks]), dk[0][db]);
      }
      // exponentials, pairs packed one element late (an exponential cannot be used by the next instruction), and dS
      constexpr int e0 = Order::exps(m - 1), e1 = Order::exps(m), n0 = Order::dss(m - 1), n1 = Order::dss(m);
      static_for<e0, e1>(exp_one);
      static_for<(e0 == 16 ? 8 : e0 > 0 ? (e0 - 1) / 2 : 0), (e0 == 16 ? 8 : e1 == 16 ? 8 : e1 > 0 ? (e1 - 1) / 2 : 0)>(pack_p);
      static_for<n0, n1>(ds_one);
      static_for<0, 4>([&](auto q_c) __attribute__((always_inline)) {
        constexpr int q = decltype(q_c)::value;
        if constexpr (m == Order::lse_read(q)) rl[q] = lds_asm_read16f<32 * q>(r_cur);
        if constexpr (m == Order::d_read(q)) rd[q] = lds_asm_read16f<D_ROWS + 32 * q>(r_cur);
      });
      if constexpr (m == Order::d_use() + 3) asm volatile("" ::"v"(rd16));  // (its registers stay: the first MFMA of dP reads them late)
      if constexpr (m == 1) dma_rows();
      if constexpr (m % COPY_EVERY == COPY_EVERY - 3) dma_piece(m / COPY_EVERY);
      if constexpr (m == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        dma_advance();
        s_cur = s_nxt;
        if (--s_heads == 0) {
          s_heads = G;
          s_qt += down ? -1 : 1;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // stage g + 2 must have landed; the copies of the DIST - 2 stages after it may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 2) * PER) : "memory");
    wg_barrier();
  };
  const int claim_at = max(0, n_iter - 3);  // the step before which wave 0 claims the next block
  for (int g = 0; g < n_iter; ++g) {
    if (g == claim_at && wave == 0 && mine == kClaimBlocks) pending_claim = block_claim_issue(fresh(args).taken, xcd);
    step();
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  // every copy of this wave has landed: once all waves have met at the barrier that hands out the next block, the ring may be filled again
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)

  {
    const DkvParams p = fresh(args);
    const int64_t kv_stride = (int64_t)p.num_kv_heads * D;
    const int lane = lane_id(), hh = lane >> 5;
    const int kr = 32 * wave + (lane & 31);
    if (!p.accumulate && !p.out_f32) {
      wg_barrier();  // nobody reads the ring any more
      lds_bf16* const stage = L + wave * (32 * D);
      const int64_t off = ((int64_t)it.kv_row0 + 32 * wave) * kv_stride + (int64_t)kvh * D;
      store_key_rows<D, 1>(stage, dv, 1.0f, p.dv + off, kv_stride, it.kv_rows - 32 * wave);
      store_key_rows<D, 1>(stage, dk, p.scale, p.dk + off, kv_stride, it.kv_rows - 32 * wave);
    } else if (kr < it.kv_rows) {
      const int64_t off = ((int64_t)it.kv_row0 + kr) * kv_stride + (int64_t)kvh * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t e = off + 32 * db + 8 * g + 4 * hh;
          dkv_store4(p, p.dv, e, dv[0][db][4 * g], dv[0][db][4 * g + 1], dv[0][db][4 * g + 2], dv[0][db][4 * g + 3]);
          dkv_store4(p, p.dk, e, dk[0][db][4 * g] * p.scale, dk[0][db][4 * g + 1] * p.scale, dk[0][db][4 * g + 2] * p.scale, dk[0][db][4 * g + 3] * p.scale);
        }
    }
  }
  if (mine != kClaimBlocks) break;
  // on to the next block; the stores of the epilogue are not waited for here
  int nb = 0;
  if (wave == 0) {
    const DkvParams p = fresh(args);
    nb = block_claim_finish(p.taken, p.num_blocks, xcd, pending_claim);
  }
  blk = broadcast_from_wave0(next_block, nb);
  }
  clock_log_stamp(fresh(args).clock_log, 1);
}

// ------------------------------------------------------------------------------------------------
// dq_pipe_blocks: the dQ blocks of bwd_pipe_kernel (head_dim 128 and 96) and, with long walks, of head_dim 64
//
// dQ in the style of dkv_pipe_blocks: one wave per SIMD, a workgroup of 4 waves, each wave
// owning two 32-row query blocks ("units": the workgroup's 8 units are the same (head, row block) pairs the
// 8 waves of bwd_dq_kernel take), so that every K / V fragment read from LDS feeds two MFMAs.  Stage t is
// the t-th 32-key tile of the segment; in step t a wave runs
//     dP^T(t) = V(t) dO^T        S^T(t+1) = K(t+1) Q^T        dQ^T += K(t-1)^T dS^T(t-1)      (matrix pipe)
//     P^T(t) = exp2(S^T(t) c - LSE)  and, once dP^T(t) is complete,  dS^T(t) = P^T(t) (dP^T(t) - D)   (vector)
// as 24 (head_dim 96: 18, 64: 12) mini-steps of one LDS operand fragment and the two MFMAs it feeds (one per unit), each MFMA followed
// by its share of the vector work.  K^T is read from the K tile itself with the LDS transpose read (tiles
// are stored chunk-major as in the dK/dV kernels), so no transposed image of K is needed.  K and V tiles
// live in a ring of DIST + 3 slots.  Steps whose tile needs the causal mask (the last one or two of the
// walk) or lies past the end run a second variant of the step that masks in the vector work.
// ------------------------------------------------------------------------------------------------
// (CUT: some items are pieces; see fwd_pipe_kernel)
template <int D, bool CUT>
__device__ __forceinline__ void dq_pipe_blocks(const ArgsPtr<DqParams> args, const int mine) {
  constexpr int NW = 4;        // waves
  constexpr int BN = 32;       // key rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dQ^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int DIST = DQ_PIPE_DIST;  // stages copied ahead
  constexpr int NS = DIST + 3; // ring slots: stages t - 1 .. t + 1 in use, t + 2 .. t + 1 + DIST on their way
  constexpr int NF = 2 * DK + 2 * DB;  // operand fragments (mini-steps) per step: V rows, K rows, K^T
  constexpr int AHEAD = 4;             // fragments in flight
  constexpr int RING = NF % 8 == 0 ? 8 : 6;  // registers of the fragment ring: a step starts where the ring does
  constexpr int NP = BN * KC / 64;     // 64-slot pieces per tile
  constexpr int PER = 2 * NP / NW;     // global->LDS copies per wave and stage
  constexpr int BOOK = D == 64 ? 8 : 12;  // mini-step of the bookkeeping, behind the last copy
  // Vector work of a step: the 16 pairs' exponentials in mini-steps EXP0 .. EXP1 - 1, their dS from DS0 on (dP^T is
  // complete two mini-steps before), spread evenly.  head_dim 128: one pair of exponentials per mini-step from 6 on (the first
  // six are left to the MFMAs alone: measured 1 % faster than starting with 0, and faster than starting with 2, 4 or
  // 8), dS one pair per mini-step from 10 on and two in the last two.
  constexpr int EXP0 = D == 128 ? 6 : D == 96 ? 4 : 2, EXP1 = D == 128 ? 22 : D == 96 ? 16 : 9, DS0 = DK + 2;
  auto exp_done = [](int m) constexpr { return spread(16, EXP0, EXP1, m); };
  auto ds_done = [](int m) constexpr { return D == 128 && m < 22 ? spread(12, DS0, 22, m) : D == 128 ? 12 + 2 * (m - 21) : spread(16, DS0, NF, m); };
  static_assert(2 * NP % NW == 0 && NF % RING == 0 && RING > AHEAD && 3 + 2 * (PER - 1) < BOOK && BOOK < NF, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int K_OFF = 0;               // [NS][KT]  K rows of stage n in slot n % NS (chunk-major)
  constexpr int V_OFF = K_OFF + NS * KT; // [NS][KT]  V rows
  // [NW][64][D] staging of a wave's 64 rows of dQ on their way out, rows of 16-byte chunks, swizzled (tile_elem<KC>):
  // global memory is then written in whole rows (four per instruction) instead of 32 rows with 16 bytes each, which
  // costs the address unit several times as long.  Its first word doubles as the slot through which wave 0 announces
  // the next block, between the last read of one block and the first write of the next.
  constexpr int ST_OFF = V_OFF + NS * KT;

  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  int* const next_block = (int*)((__bf16*)smem + ST_OFF);

  // The workgroup is persistent: it claims one block (work item x key/value head x head split) after the other
  // (device_common.hpp) until none is left.  The next block is claimed before the current one's last few steps: early
  // enough for the answer to arrive by the time it is needed, and not earlier (that would fix the order of the blocks
  // before it is known which workgroup is free first).
  const int xcd = xcd_of_this_wave();
  clock_log_stamp(fresh(args).clock_log, 0);
  int blk = mine;
  if (mine == kClaimBlocks) {
    const DqParams p = fresh(args);
    if (wave == 0) blk = block_claim_finish(p.taken, p.num_blocks, xcd, block_claim_issue(p.taken, xcd));
    blk = broadcast_from_wave0(next_block, blk);
  }
  while (blk >= 0) {
  wg_barrier();  // every wave has read the announcement: the staging area may be written again
  const DqParams p = fresh(args);
  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = __builtin_amdgcn_readfirstlane(blk % inner_n);
  const DqItem it = load_uniform(p.items, __builtin_amdgcn_readfirstlane(blk / inner_n));
  const int kvh = __builtin_amdgcn_readfirstlane(inner % p.num_kv_heads), hs = inner / p.num_kv_heads;
  int head[2], row0[2];  // of the wave's two units
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int unit = 2 * wave + u;
    head[u] = kvh * p.group + hs * p.heads_per_wg + unit % p.heads_per_wg;
    row0[u] = (unit / p.heads_per_wg) * 32;
  }

  const int n_last = it.n0 + it.q_rows - 1;                // keys the last valid row sees ...
  const int n_wg = CUT ? min(n_last, it.keys) : n_last;  // ... of the item's range
  const int nt = (n_wg + BN - 1) / BN;       // stages

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  // the ring slots the prologue does not fill are read before anything is copied into them (K(-1) in step 0)
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
  // copied again (into a slot nobody reads for anything that counts). ----
  unsigned v_full[PER], v_last[PER];  // byte offset of the lane's chunk from the tile's first row: full tile, last tile
  {
    const int last_row = n_wg - 1 - (nt - 1) * BN;  // rows past the last key repeat it (masked)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int x = ((i * NW + wave) % NP) * 64 + lane;
      const int off = (x >> 5) * 8, row = (x & 31) ^ (((x >> 5) & 3) << 2);
      v_full[i] = (unsigned)(row * (int)kv_stride + off) * 2u;
      v_last[i] = (unsigned)(min(row, last_row) * (int)kv_stride + off) * 2u;
    }
  }
  int d_t = 0, d_slot = 0;   // stage to copy next (clamped to the last one) and its slot
  const char* d_k = reinterpret_cast<const char*>(Kg);  // its first row in K and in V (running pointers stay in scalar registers)
  const char* d_v = reinterpret_cast<const char*>(Vg);
  auto dma_piece = [&](int i) __attribute__((always_inline)) {
    const int piece = i * NW + wave;  // wave-uniform; the first NP are pieces of K, the others of V
    const bool of_k = NP % NW == 0 ? i < NP / NW : piece < NP;
    const unsigned voff = d_t == nt - 1 ? v_last[i] : v_full[i];
    const char* base = of_k ? d_k : d_v;
    lds_bf16* dst = L + (of_k ? K_OFF + piece * 512 : V_OFF + (piece - NP) * 512) + d_slot * KT;
    dma16(base + voff, dst);
  };
  auto dma_advance = [&]() __attribute__((always_inline)) {
    if (d_t + 1 < nt) {
      ++d_t;
      d_k += BN * kv_stride * 2;
      d_v += BN * kv_stride * 2;
    }
    d_slot = d_slot == NS - 1 ? 0 : d_slot + 1;
  };

  // per-lane operand addresses inside a tile (as in the dK/dV kernels)
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
  const unsigned v_ev0 = lds_addr(L + V_OFF + x_off[0]), v_od0 = lds_addr(L + V_OFF + x_off[1]);
  const unsigned t_lo0 = lds_addr(L + K_OFF + t_off[0]), t_hi0 = lds_addr(L + K_OFF + t_off[1]);
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

  // prologue: the copies of stages 0 and 1 first, then the fragments, so that both travel at the same time, then the later
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
  // Q and dO fragments (B operands): lane holds X[row = l32 of the unit][16 ks + 8 hh ..+7]; LSE and D of that row
  bf16x8 qf[2][DK], gf[2][DK];
  float lse2[2], dsum[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int r_own = min(row0[u] + l32, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
    const int64_t off = (int64_t)(it.q_row0 + r_own) * q_stride + (int64_t)head[u] * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      qf[u][ks] = *reinterpret_cast<const bf16x8*>(p.q + off + 16 * ks);
      gf[u][ks] = *reinterpret_cast<const bf16x8*>(p.d_o + off + 16 * ks);
    }
    const int64_t slot = (int64_t)head[u] * p.total_q_tiles * 64 + it.q_slot0 + r_own;
    lse2[u] = p.lse2p[slot];
    dsum[u] = p.dsp[slot];
  }
  // -D of the unit's row in every element of a tile: the accumulation of dP^T starts from it, so that the vector work
  // gets dP - D straight from the matrix pipe (a column of dP^T belongs to one query row)
  f32x16 dneg[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 16; ++i) dneg[u][i] = dsum[u];
  copy_stages(DIST - 1);
  // One wait the compiler can see for the fragments (and the copies before them), so that it puts no full waits for outstanding
  // loads into the loop
  wait_all_but<(DIST - 1) * PER>();
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dq[2][DB];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int db = 0; db < DB; ++db) dq[u][db] = zero16;
  f32x16 x[2][2];   // S^T: [buffer][unit]
  f32x16 dp[2];     // dP^T: [unit]
  bf16x8 f[2][2][2];  // dS^T as B operands: [buffer][unit][k-step]
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

  // S^T(0) = K(0) Q^T, then the first fragments of step 0 (V rows of stage 0)
  {
    bf16x8 a[DK];
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) { a[decltype(ks_c)::value] = load_rows(k_ev0, k_od0, ks_c); });
    static_for<0, AHEAD>([&](auto ks_c) __attribute__((always_inline)) { fr[decltype(ks_c)::value] = load_rows(v_ev0, v_od0, ks_c); });
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(AHEAD) : "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(a[ks]));  // (after the wait, in this order)
#pragma unroll
    for (int ks = 0; ks < DK; ++ks)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(x[0][u]) : "v"(a[ks]), "a"(qf[u][ks]));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(x[0][u]) : "v"(a[ks]), "a"(qf[u][ks]));
      }
    mfma_settle();
  }

  // In program order mini-step m reads fragment m + 4: one instruction for the rows fragments (0 .. 2 DK - 1 of this step,
  // 0 .. 3 of the next), two for the transposed ones.
  int sV = 0;  // slot of stage t
  auto step = [&](int t, f32x16 (&cur)[2], f32x16 (&nxt)[2], bf16x8 (&f_old)[2][2], bf16x8 (&f_new)[2][2],
                  auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int sK = sV == NS - 1 ? 0 : sV + 1;   // stage t + 1
    const int sM = sV == 0 ? NS - 1 : sV - 1;   // stage t - 1
    const unsigned v_ev = v_ev0 + sV * SLOT, v_od = v_od0 + sV * SLOT, k_ev = k_ev0 + sK * SLOT, k_od = k_od0 + sK * SLOT;
    const unsigned t_lo = t_lo0 + sM * SLOT, t_hi = t_hi0 + sM * SLOT, n_ev = v_ev0 + sK * SLOT, n_od = v_od0 + sK * SLOT;
    // MASKED: element i (key 8 (i / 4) + 4 hh + i % 4 of the tile) of unit u is visible iff 8 (i / 4) + i % 4 < lim[u]
    int lim[2];
    if (MASKED) {
#pragma unroll
      for (int u = 0; u < 2; ++u) lim[u] = t < nt ? it.n0 + row0[u] + l32 - BN * t - 4 * hh : -0x40000000;
    }
    float pf[2][16];   // P^T(t)
    unsigned pw[2][8]; // dS^T(t), packed pairs
    auto exp_half = [&](auto j_c, auto q_c) __attribute__((always_inline)) {  // P of element 2 dw + q of unit u (pair j = 8 u + dw)
      constexpr int j = decltype(j_c)::value, q = decltype(q_c)::value;
      constexpr int u = j >> 3, i = 2 * (j & 7) + q;
      float tt = cur[u][i] * c - lse2[u];
      if (MASKED) {
        if (8 * (i >> 2) + (i & 3) >= lim[u]) tt = -INFINITY;
      }
      pf[u][i] = __builtin_amdgcn_exp2f(tt);
      asm volatile("" : "+v"(pf[u][i]));  // pinned here (the compiler would gather the vector work elsewhere)
    };
    auto ds_pair = [&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value;
      constexpr int u = j >> 3, dw = j & 7;
      bf16x2 w;
      w[0] = (__bf16)(pf[u][2 * dw] * dp[u][2 * dw]);  // dp holds dP - D: its accumulation starts from -D
      w[1] = (__bf16)(pf[u][2 * dw + 1] * dp[u][2 * dw + 1]);
      unsigned wu = __builtin_bit_cast(unsigned, w);
      asm volatile("" : "+v"(wu));
      pw[u][dw] = wu;
    };
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[m % RING]) : "n"(fragment_wait(NF, 2 * DK, NF, m)));
      {  // read the fragment of mini-step m + AHEAD (past the end: the next step's first V fragments)
        constexpr int mm = m + AHEAD;
        if constexpr (mm < DK) fr[mm % RING] = load_rows(v_ev, v_od, std::integral_constant<int, mm>{});
        else if constexpr (mm < 2 * DK) fr[mm % RING] = load_rows(k_ev, k_od, std::integral_constant<int, mm - DK>{});
        else if constexpr (mm < NF) fr[mm % RING] = load_t(t_lo, t_hi, std::integral_constant<int, mm - 2 * DK>{});
        else fr[mm % RING] = load_rows(n_ev, n_od, std::integral_constant<int, mm - NF>{});
      }
      const bf16x8 fa = fr[m % RING];
      // dP^T and S^T are kept in vector registers, the Q / dO fragments in accumulation registers (opaque MFMAs, see
      // dkv_pipe_blocks); dP^T is first read three mini-steps after its last MFMA, S^T in the next step
      auto mma = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        const bf16x8& a_ = fa;  // (named references: variables used only inside an asm statement are not captured)
        if constexpr (m < DK) {
          f32x16& d_ = dp[u];
          const bf16x8& b_ = gf[u][m];
          const f32x16& n_ = dneg[u];
          if (m == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d_) : "v"(a_), "a"(b_), "v"(n_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
        } else if constexpr (m < 2 * DK) {
          constexpr int ks = m - DK;
          f32x16& d_ = nxt[u];
          const bf16x8& b_ = qf[u][ks];
          if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
          else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
        } else {
          constexpr int ks = (m - 2 * DK) / DB, db = (m - 2 * DK) % DB;
          dq[u][db] = mfma32(fa, f_old[u][ks], dq[u][db]);
        }
      };
      constexpr std::integral_constant<int, 0> c0{};
      constexpr std::integral_constant<int, 1> c1{};
      // scores e0 .. e1 - 1 (two per pair) and pairs s0 .. s1 - 1 of dS belong to this mini-step, the first half of each
      // after its first MFMA
      constexpr int e0 = 2 * exp_done(m - 1), e1 = 2 * exp_done(m), em = e0 + (e1 - e0 + 1) / 2;
      constexpr int s0 = ds_done(m - 1), s1 = ds_done(m), sm = s0 + (s1 - s0 + 1) / 2;
      static_assert(s1 <= exp_done(m - 1), "a pair's exponentials come before its dS");
      auto exp_range = [&](auto lo_c, auto hi_c) __attribute__((always_inline)) {
        static_for<decltype(lo_c)::value, decltype(hi_c)::value>([&](auto i_c) __attribute__((always_inline)) {
          constexpr int i = decltype(i_c)::value;
          exp_half(std::integral_constant<int, i / 2>{}, std::integral_constant<int, i % 2>{});
        });
      };
      mma(c0);
      exp_range(std::integral_constant<int, e0>{}, std::integral_constant<int, em>{});
      static_for<s0, sm>(ds_pair);
      __builtin_amdgcn_sched_barrier(0);
      mma(c1);
      exp_range(std::integral_constant<int, em>{}, std::integral_constant<int, e1>{});
      if constexpr (m >= 3 && m < 3 + 2 * PER && ((m - 3) & 1) == 0) dma_piece((m - 3) >> 1);
      static_for<sm, s1>(ds_pair);
      if constexpr (m == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        dma_advance();
        sV = sK;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        u32x4 v = {pw[u][4 * ks], pw[u][4 * ks + 1], pw[u][4 * ks + 2], pw[u][4 * ks + 3]};
        f_new[u][ks] = __builtin_bit_cast(bf16x8, v);
      }
    // stage t + 2 must have landed; the copies of the DIST - 1 stages after it may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DIST - 1) * PER) : "memory");
    wg_barrier();
  };

  // Steps are taken two at a time (the two S^T buffers and the two dS^T buffers swap roles without a copy): first the
  // pairs whose tiles every row of the wave sees completely, then the rest with the mask, up to step nt (whose only
  // real work is the dQ^T product of the last tile); a pair may run one step past that, which contributes nothing.
  const int t_full = min(nt, (it.n0 + min(row0[0], row0[1])) / BN) & ~1;
  int t = 0;
  for (; t < t_full; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::false_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::false_type{});
  }
  int pending_claim = 0;
  if (wave == 0 && mine == kClaimBlocks) pending_claim = block_claim_issue(fresh(args).taken, xcd);
  for (; t <= nt; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::true_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::true_type{});
  }

  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  // every copy of this wave has landed (the last ones rewrote a slot nobody reads): after the barrier below the next
  // block may fill the ring again
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  // ---- epilogue: dQ = scale * dQ^T, through the wave's staging tile (one unit after the other) ----
  lds_bf16* const stage = L + ST_OFF + wave * (64 * D);
  // (the lane index is made opaque here: the addresses below depend on nothing else, and computed ahead of the loop
  // they would take registers the loop has no room for)
  int lane_e = lane;
  asm volatile("" : "+v"(lane_e));
  const int l32_e = lane_e & 31, hh_e = lane_e >> 5;
  const DqParams pe = fresh(args);
  const int64_t q_stride_e = (int64_t)pe.num_q_heads * D;
  if (CUT && it.part >= 0) {  // a piece: dQ^T as it is, put together by bwd_merge_kernel
    float* const out = pe.parts + ((int64_t)it.part * (pe.num_kv_heads * pe.head_splits) + inner) * kPartRowFloats + wave * (2 * 4096) + lane_e * 4;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(out + u * 4096 + (db * 4 + g) * 256) =
              f32x4{dq[u][db][4 * g], dq[u][db][4 * g + 1], dq[u][db][4 * g + 2], dq[u][db][4 * g + 3]};
  } else
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const bf16x4 v = pack4(dq[u][db][4 * g] * pe.scale, dq[u][db][4 * g + 1] * pe.scale, dq[u][db][4 * g + 2] * pe.scale,
                               dq[u][db][4 * g + 3] * pe.scale);
        *(__attribute__((address_space(3))) bf16x4*)(stage + tile_elem<KC>(32 * u + l32_e, 4 * db + g) + 4 * hh_e) = v;
      }
    __bf16* obase = pe.dq + (int64_t)(it.q_row0 + row0[u]) * q_stride_e + (int64_t)head[u] * D;
#pragma unroll 2
    for (int i = 0; i < 32 * KC / 64; ++i) {
      const int x = (u * 32 * KC / 64 + i) * 64 + lane_e;
      const int row = x / KC, c = unswz<KC>(row, x % KC);  // row of the staging tile: 32 u + row of the unit
      const bf16x8 v = lds_load8(stage + x * 8);
      const int ru = row - 32 * u;
      if (row0[u] + ru < it.q_rows) *reinterpret_cast<bf16x8*>(obase + (int64_t)ru * q_stride_e + c * 8) = v;
    }
  }
  if (mine != kClaimBlocks) break;
  // on to the next block; the stores above are not waited for here
  int nb = 0;
  if (wave == 0) {
    const DqParams pc = fresh(args);
    nb = block_claim_finish(pc.taken, pc.num_blocks, xcd, pending_claim);
  }
  blk = broadcast_from_wave0(next_block, nb);
  }
  clock_log_stamp(fresh(args).clock_log, 1);
}

// ------------------------------------------------------------------------------------------------
// bwd_dq_wide (head_dim 256)
//
// dQ in the style of dq_pipe_blocks with 32 query rows per wave (Q and dO fragments and dQ^T take all 256 accumulation registers): in step t
// a wave runs
//     dP^T(t) = V(t) dO^T        S^T(t+1) = K(t+1) Q^T        dQ^T += K(t-1)^T dS^T(t-1)      (matrix pipe)
//     P^T(t) = exp2(S^T(t) c - LSE)  and, once dP^T(t) is complete,  dS^T(t) = P^T(t) (dP^T(t) - D)   (vector)
// as 48 mini-steps of one operand fragment and the MFMA it feeds.  dP^T and S^T are one accumulator each, so their MFMAs are kept
// apart: 16 of dP^T alternate with 8 of S^T and 8 of dQ^T, then the other 8 of S^T with the other 8 of dQ^T, next to which dS^T is formed.
// LDS is full: six stages of K (t - 1, t, t + 1 and, read ahead over the end of the step, t + 2 in use; t + 3 and t + 4 on their way) and
// four of V (t and t + 1 in use, t + 2 and t + 3 on their way); a copy has more than a step to land.  dQ goes out through the V
// ring.  As in fwd_wide_kernel every fragment feeds one MFMA, so a step is bound by its 64 LDS reads and 48 MFMAs.
// Packed 64K chunk, 32/8 heads, backward: 29.4 ms with bwd_dq_kernel, 27.2 with this; 8192 queries on 32768 keys 25.9 -> 24.0 (dq_wide_pays: more).
// ------------------------------------------------------------------------------------------------
// mini-step k: what its MFMA adds to (0: dP^T, 1: S^T, 2: dQ^T) and the index of its fragment
constexpr int wide_kind(int k) { return k < 32 ? (k % 2 == 0 ? 0 : k % 4 == 1 ? 1 : 2) : 1 + k % 2; }
constexpr int wide_index(int k) { return k < 32 ? (k % 2 == 0 ? k / 2 : k / 4) : 8 + (k - 32) / 2; }
// LDS instructions issued between the read of fragment k and the start of mini-step k (a transposed fragment takes two)
constexpr int wide_wait(int k, int ahead) {
  int n = 0;
  for (int i = k + 1; i < k + ahead; ++i) n += wide_kind(i % 48) == 2 ? 2 : 1;
  return n;
}
static_assert(wide_kind(0) == 0 && wide_kind(1) == 1 && wide_kind(3) == 2 && wide_kind(30) == 0 && wide_kind(32) == 1 && wide_kind(47) == 2 &&
              wide_index(1) == 0 && wide_index(3) == 0 && wide_index(5) == 1 && wide_index(29) == 7 && wide_index(30) == 15 && wide_index(31) == 7 &&
              wide_index(32) == 8 && wide_index(47) == 15 && wide_wait(0, 6) == 6 && wide_wait(32, 6) == 8, "worked out by hand");

__device__ __forceinline__ void dq_wide_blocks(ArgsPtr<DqParams> args, int mine) {
  constexpr int D = 256;
  constexpr int NW = 4;        // waves
  constexpr int BN = 32;       // key rows per stage
  constexpr int KC = D / 8;    // 16-byte chunks per K / V row
  constexpr int DK = D / 16;   // k-steps over the head dimension
  constexpr int DB = D / 32;   // 32-row blocks of dQ^T
  constexpr int KT = BN * D;   // elements per tile
  constexpr int KS = 6, VS = 4;           // ring slots of K and of V
  constexpr int NF = 3 * DK;              // mini-steps per step
  constexpr int AHEAD = 6, RING = 8;      // fragments in flight, registers of the fragment ring
  constexpr int PER = BN * KC / 64 / NW;  // global->LDS copies per wave, tile and stage
  constexpr int EXP0 = 3, DS0 = 33;       // score i's exponential next to MFMA EXP0 + 2 i, pair j of dS next to MFMA DS0 + 2 j
  constexpr int BOOK = 40;                // mini-step of the bookkeeping, behind the last copy
  static_assert(NF == 48 && 2 * DB == DK && NF % RING == 0 && RING > AHEAD && 2 + 5 * (2 * PER - 1) < BOOK, "the schedule of a step");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  lds_bf16* const L = (lds_bf16*)smem;
  constexpr int K_OFF = 0;               // [KS][KT]  K rows of stage n in slot n % KS (chunk-major)
  constexpr int V_OFF = K_OFF + KS * KT; // [VS][KT]  V rows
  // the V ring is also the [NW][32][D] staging of dQ on its way out (rows of swizzled 16-byte chunks), whose first word
  // doubles as the slot through which wave 0 announces the next block
  constexpr int ST_OFF = V_OFF;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  int* const next_block = (int*)((__bf16*)smem + ST_OFF);

  const int xcd = xcd_of_this_wave();
  const bool direct = mine != kClaimBlocks;
  int blk = mine;
  if (!direct) {
    const DqParams p = fresh(args);
    if (wave == 0) blk = block_claim_finish(p.taken, p.num_blocks, xcd, block_claim_issue(p.taken, xcd));
    blk = broadcast_from_wave0(next_block, blk);
  }
  int pending_claim = 0;
  while (blk >= 0) {
  wg_barrier();  // every wave has read the announcement: the V ring may be written again
  const DqParams p = fresh(args);
  const int inner_n = p.num_kv_heads * p.head_splits;
  const int inner = __builtin_amdgcn_readfirstlane(blk % inner_n);
  const DqItem it = load_uniform(p.items, __builtin_amdgcn_readfirstlane(blk / inner_n));
  const int kvh = __builtin_amdgcn_readfirstlane(inner % p.num_kv_heads), hs = inner / p.num_kv_heads;
  const int head = kvh * p.group + hs * p.heads_per_wg + wave % p.heads_per_wg;
  const int row0 = (wave / p.heads_per_wg) * 32;
  const int n_wg = it.n0 + it.q_rows - 1;  // keys the last valid row sees
  const int nt = (n_wg + BN - 1) / BN;     // stages

  const int64_t q_stride = (int64_t)p.num_q_heads * D, kv_stride = (int64_t)p.num_kv_heads * D;
  const __bf16* __restrict__ Kg = p.k + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;
  const __bf16* __restrict__ Vg = p.v + (int64_t)it.kv_row0 * kv_stride + (int64_t)kvh * D;

  {  // K(-1), read in step 0 before anything is copied into its slot
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    for (int x = tid; x < KT / 8; x += NW * 64) lds_store8(L + K_OFF + (KS - 1) * KT + x * 8, z);
  }

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
  struct Stream {  // the next stage to copy, its slot, its first row
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
  const unsigned v_ev0 = lds_addr(L + V_OFF + x_off[0]), v_od0 = lds_addr(L + V_OFF + x_off[1]);
  const unsigned t_lo0 = lds_addr(L + K_OFF + t_off[0]), t_hi0 = lds_addr(L + K_OFF + t_off[1]);
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

  // prologue: K of stages 0 .. 2 and V of stages 0 and 1 first, then the fragments, so that all travel at the same time, then
  // K(3) and V(2), which step 0 waits for at its end
  auto copy_tile = [&](Stream& st, int ring, int slots) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PER; ++i) copy_piece(st, ring, i);
    advance(st, slots);
  };
#pragma unroll
  for (int n = 0; n < 3; ++n) copy_tile(ks, K_OFF, KS);
#pragma unroll
  for (int n = 0; n < 2; ++n) copy_tile(vs, V_OFF, VS);
  // Q and dO fragments (B operands): lane holds X[row = l32][16 ks + 8 hh ..+7]; LSE and D of that row
  bf16x8 qf[DK], gf[DK];
  float lse2, dsum;
  {
    const int r_own = min(row0 + l32, it.q_rows - 1);  // rows past the tile repeat the last one (never stored)
    const int64_t off = (int64_t)(it.q_row0 + r_own) * q_stride + (int64_t)head * D + 8 * hh;
#pragma unroll
    for (int k = 0; k < DK; ++k) {
      qf[k] = *reinterpret_cast<const bf16x8*>(p.q + off + 16 * k);
      gf[k] = *reinterpret_cast<const bf16x8*>(p.d_o + off + 16 * k);
    }
    const int64_t slot = (int64_t)head * p.total_q_tiles * 64 + it.q_slot0 + r_own;
    lse2 = p.lse2p[slot];
    dsum = p.dsp[slot];
  }
  f32x16 dneg;  // -D of the lane's row in every element: the accumulation of dP^T starts from it (as in dq_pipe_blocks)
#pragma unroll
  for (int i = 0; i < 16; ++i) dneg[i] = dsum;
  copy_tile(ks, K_OFF, KS);
  copy_tile(vs, V_OFF, VS);
  // One wait the compiler can see for the fragments (and the copies before them), so that it puts no full waits for outstanding
  // loads into the loop
  wait_all_but<2 * PER>();
  // (the fragments settle in their accumulation registers here: an opaque MFMA must not follow a write to one of its operands)
#pragma unroll
  for (int k = 0; k < DK; ++k) {
    asm volatile("" : "+a"(qf[k]));
    asm volatile("" : "+a"(gf[k]));
  }
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16;
  f32x16 x[2], dp;   // S^T (two buffers), dP^T
  bf16x8 f[2][2];    // dS^T as B operands: [buffer][k-step]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < 8; ++i) f[b][k][i] = (__bf16)0.0f;
  const float c = p.scale_log2;
  bf16x8 fr[RING];  // ring of operand fragments

  {  // S^T(0) = K(0) Q^T
    bf16x8 a[DK];
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) { a[decltype(ks_c)::value] = load_rows(k_ev0, k_od0, ks_c); });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int k = 0; k < DK; ++k) asm volatile("" : "+v"(a[k]));  // (after the wait, in this order)
#pragma unroll
    for (int k = 0; k < DK; ++k) {
      f32x16& d_ = x[0];
      const bf16x8& b_ = qf[k];
      if (k == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a[k]), "a"(b_));
      else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a[k]), "a"(b_));
    }
    mfma_settle();
  }

  // the fragment of mini-step k of a step whose V(t), K(t + 1) and K(t - 1) lie in slots sV, sK and sT
  auto load_fragment = [&](auto k_c, int sV, int sK, int sT) __attribute__((always_inline)) {
    constexpr int k = decltype(k_c)::value, kind = wide_kind(k);
    constexpr std::integral_constant<int, wide_index(k)> i{};
    if constexpr (kind == 0) return load_rows(v_ev0 + sV * SLOT, v_od0 + sV * SLOT, i);
    else if constexpr (kind == 1) return load_rows(k_ev0 + sK * SLOT, k_od0 + sK * SLOT, i);
    else return load_t(t_lo0 + sT * SLOT, t_hi0 + sT * SLOT, i);
  };
  static_for<0, AHEAD>([&](auto k_c) __attribute__((always_inline)) { fr[decltype(k_c)::value] = load_fragment(k_c, 0, 1, KS - 1); });

  int sV = 0, sK = 1, sT = KS - 1;  // slots of V(t), K(t + 1), K(t - 1)
  auto step = [&](int t, f32x16& cur, f32x16& nxt, bf16x8 (&f_old)[2], bf16x8 (&f_new)[2], auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int nV = sV == VS - 1 ? 0 : sV + 1, nK = sK == KS - 1 ? 0 : sK + 1, nT = sT == KS - 1 ? 0 : sT + 1;  // of the next step
    // MASKED: element i (key 8 (i / 4) + 4 hh + i % 4 of the tile) is visible iff 8 (i / 4) + i % 4 < lim
    int lim = 0;
    if (MASKED) lim = t < nt ? it.n0 + row0 + l32 - BN * t - 4 * hh : -0x40000000;
    float pf[16];   // P^T(t)
    unsigned pw[8]; // dS^T(t), packed pairs
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NF>([&](auto k_c) __attribute__((always_inline)) {
      constexpr int k = decltype(k_c)::value, kind = wide_kind(k), idx = wide_index(k);
      static_assert(wide_wait(k, AHEAD) <= 15, "lgkmcnt is a 4-bit counter");
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[k % RING]) : "n"(wide_wait(k, AHEAD)));
      {  // read the fragment of mini-step k + AHEAD (past the end: the next step's first ones)
        constexpr int kk = k + AHEAD;
        if constexpr (kk < NF) fr[kk % RING] = load_fragment(std::integral_constant<int, kk>{}, sV, sK, sT);
        else fr[kk % RING] = load_fragment(std::integral_constant<int, kk - NF>{}, nV, nK, nT);
      }
      const bf16x8& a_ = fr[k % RING];
      if constexpr (kind == 0) {
        f32x16& d_ = dp;
        const bf16x8& b_ = gf[idx];
        const f32x16& n_ = dneg;
        if (idx == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d_) : "v"(a_), "a"(b_), "v"(n_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
      } else if constexpr (kind == 1) {
        f32x16& d_ = nxt;
        const bf16x8& b_ = qf[idx];
        if (idx == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d_) : "v"(a_), "a"(b_));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d_) : "v"(a_), "a"(b_));
      } else {
        dq[idx % DB] = mfma32(a_, f_old[idx / DB], dq[idx % DB]);
      }
      if constexpr (k >= EXP0 && (k - EXP0) % 2 == 0 && (k - EXP0) / 2 < 16) {
        constexpr int i = (k - EXP0) / 2;
        float tt = cur[i] * c - lse2;
        if (MASKED) {
          if (8 * (i >> 2) + (i & 3) >= lim) tt = -INFINITY;
        }
        pf[i] = __builtin_amdgcn_exp2f(tt);
        asm volatile("" : "+v"(pf[i]));  // pinned here (the compiler would gather the vector work elsewhere)
      }
      if constexpr (k >= DS0 && (k - DS0) % 2 == 0 && (k - DS0) / 2 < 8) {
        constexpr int j = (k - DS0) / 2;
        static_assert(EXP0 + 2 * (2 * j + 1) < k, "a pair's exponentials come before its dS");
        bf16x2 w;
        w[0] = (__bf16)(pf[2 * j] * dp[2 * j]);  // dp holds dP - D: its accumulation starts from -D
        w[1] = (__bf16)(pf[2 * j + 1] * dp[2 * j + 1]);
        unsigned wu = __builtin_bit_cast(unsigned, w);
        asm volatile("" : "+v"(wu));
        pw[j] = wu;
      }
      // V(t + 3) and K(t + 4)
      if constexpr (k >= 2 && (k - 2) % 5 == 0 && (k - 2) / 5 < 2 * PER) {
        constexpr int i = (k - 2) / 5;
        if constexpr (i < PER) copy_piece(vs, V_OFF, i);
        else copy_piece(ks, K_OFF, i - PER);
      }
      if constexpr (k == BOOK) {  // bookkeeping for the next step (this step's copies have been issued)
        advance(ks, KS);
        advance(vs, VS);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    sV = nV;
    sK = nK;
    sT = nT;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      u32x4 v = {pw[4 * k], pw[4 * k + 1], pw[4 * k + 2], pw[4 * k + 3]};
      f_new[k] = __builtin_bit_cast(bf16x8, v);
    }
    // the copies of the step before (V(t + 2), K(t + 3)) must have landed; this step's may still be in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
    wg_barrier();
  };

  // (as in dq_pipe_blocks)
  const int t_full = min(nt, (it.n0 + row0) / BN) & ~1;
  int t = 0;
  for (; t < t_full; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::false_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::false_type{});
  }
  if (wave == 0 && !direct) pending_claim = block_claim_issue(fresh(args).taken, xcd);
  for (; t <= nt; t += 2) {
    step(t, x[0], x[1], f[0], f[1], std::true_type{});
    step(t + 1, x[1], x[0], f[1], f[0], std::true_type{});
  }
  // the last step's reads ahead are nobody's operands; their registers stay taken until they have arrived
#pragma unroll
  for (int i = 0; i < RING; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(fr[i]));
  // every copy of this wave has landed (the last ones rewrote slots nobody reads)
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  wg_barrier();  // nobody reads the rings, and nobody copies into them, any more: dQ may be staged there

  // ---- epilogue: dQ = scale * dQ^T, through the wave's staging tile (as in dq_pipe_blocks) ----
  {
    const DqParams pe = fresh(args);
    const int64_t q_stride_e = (int64_t)pe.num_q_heads * D;
    lds_bf16* const stage = L + ST_OFF + wave * KT;
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int l32_e = lane_e & 31, hh_e = lane_e >> 5;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const bf16x4 v = pack4(dq[db][4 * g] * pe.scale, dq[db][4 * g + 1] * pe.scale, dq[db][4 * g + 2] * pe.scale, dq[db][4 * g + 3] * pe.scale);
        *(__attribute__((address_space(3))) bf16x4*)(stage + tile_elem<KC>(l32_e, 4 * db + g) + 4 * hh_e) = v;
      }
    __bf16* obase = pe.dq + (int64_t)(it.q_row0 + row0) * q_stride_e + (int64_t)head * D;
#pragma unroll 4
    for (int i = 0; i < 32 * KC / 64; ++i) {
      const int y = i * 64 + lane_e;
      const int row = y / KC, ch = unswz<KC>(row, y % KC);
      const bf16x8 v = lds_load8(stage + y * 8);
      if (row0 + row < it.q_rows) *reinterpret_cast<bf16x8*>(obase + (int64_t)row * q_stride_e + ch * 8) = v;
    }
  }
  if (direct) break;
  // on to the next block; the stores above are not waited for here
  int nb = 0;
  if (wave == 0) {
    const DqParams pc = fresh(args);
    nb = block_claim_finish(pc.taken, pc.num_blocks, xcd, pending_claim);
  }
  blk = broadcast_from_wave0(next_block, nb);
  }
}

__global__ __launch_bounds__(256, 1) void bwd_dq_wide_kernel(DqParams) {
  const ArgsPtr<DqParams> args = (ArgsPtr<DqParams>)__builtin_amdgcn_kernarg_segment_ptr();
  dq_wide_blocks(args, args->num_blocks <= (int)gridDim.x ? (int)blockIdx.x : kClaimBlocks);
}

// ------------------------------------------------------------------------------------------------
// bwd_pipe (head_dim 128 and 96, 256 where wide_pays and 64 where narrow_tall_pays): the dQ and the dK/dV blocks of a chunk in one launch
//
// The two kinds of block need nothing of each other, so a workgroup that finds no more blocks of one kind goes on to the other:
// small chunks run both kinds side by side on compute units that one kind alone would leave idle, and no chunk ends twice.  The kind
// with the longer walks goes first (`dq_phase`: the phase of dQ), so that long blocks do not start last.  Both kinds fill
// the LDS and a wave's registers, whatever the order.  Forward and backward, two launches -> one: 557 causal tokens, 32/8 heads,
// 123 -> 96 us; two slices of 3193 and 4999 queries (backwards only) 1886 -> 1801; packed 64K chunk, 8192 queries on 32768 keys within 0.3 %;
// 16384 queries on 131072 keys, 64/8, 230.8 -> 232.5 ms at most (four comparisons, 0.1 - 0.7 %): dQ blocks start as dK/dV blocks end, no longer together,
// and fetch K and V more often.  Head_dim 256, 250 queries on 4730 keys, 16/8 heads, backward, 236 -> 168 us; 512 on 8704, 8/8, 384 -> 281.
// ------------------------------------------------------------------------------------------------
struct BwdPipeParams {
  DqParams dq;
  DkvParams dkv;
  int32_t dq_phase;
};
template <int D, bool CUT, bool TALL>
__global__ __launch_bounds__(256, 1) void bwd_pipe_kernel(BwdPipeParams) {
  static_assert(D != 256 || (!CUT && TALL), "head_dim 256: dq_wide_blocks and dkv_wide_blocks");
  typedef const __attribute__((address_space(4))) BwdPipeParams* args_ptr;
  for (int phase = 0; phase < 2; ++phase) {
    if (phase > 0) wg_barrier();  // every wave has read that no block of the other kind is left: the LDS may be written again
    args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const bool is_dq = phase == args->dq_phase;
    if ((is_dq ? args->dq.num_blocks : args->dkv.num_blocks) == 0) continue;  // (this launch has blocks of the other kind only)
    int mine = kClaimBlocks;
    if (args->dq.num_blocks + args->dkv.num_blocks <= (int)gridDim.x) {  // a workgroup per block: nothing to claim
      const int first = args->dq_phase == 0 ? args->dq.num_blocks : args->dkv.num_blocks;
      mine = phase == 0 ? ((int)blockIdx.x < first ? (int)blockIdx.x : -1) : (int)blockIdx.x - first;
    }
    if constexpr (D == 256) {
      if (is_dq) dq_wide_blocks(&args->dq, mine);
      else dkv_wide_blocks<D>(&args->dkv, mine);
    } else if (is_dq) dq_pipe_blocks<D, CUT>(&args->dq, mine);
    else if constexpr (TALL) dkv_tall_blocks<D>(&args->dkv, mine);
    else dkv_pipe_blocks<D, CUT>(&args->dkv, mine);
    if (mine >= 0) break;
  }
}

// The same for chunks of head_dim 64 and 256 that are too small or too short for the pipelined dK/dV kernels, a workgroup per block.  Each kind by
// itself is a launch, first copies and walks that leave compute units idle at their end; neither waits for the other here.  At 64 a
// dQ block takes four of the eight waves; the others end at once (a barrier waits for the waves that are left).  Figures: short_joins.
template <int D, int KB, bool CUT, bool WIDE>
__global__ __launch_bounds__(KB * 128, D > 128 ? 1 : 4 / KB) void bwd_short_kernel(BwdPipeParams p) {
  const int first = p.dq_phase == 0 ? p.dq.num_blocks : p.dkv.num_blocks;
  const bool second = (int)blockIdx.x >= first;
  const int blk = second ? (int)blockIdx.x - first : (int)blockIdx.x;
  if (second == (p.dq_phase == 0)) {
    dkv_block<D, KB, CUT>(p.dkv, blk);
  } else if constexpr (WIDE) {
    dq_wide_blocks(&((ArgsPtr<BwdPipeParams>)__builtin_amdgcn_kernarg_segment_ptr())->dq, blk);
  } else if (threadIdx.x < 256) {
    dq_block<D, 4>(p.dq, blk);
  }
}

// head_dim 64, where dQ is pipelined
__global__ __launch_bounds__(256, 1) void bwd_dq_pipe_kernel(DqParams) {
  dq_pipe_blocks<64, false>((ArgsPtr<DqParams>)__builtin_amdgcn_kernarg_segment_ptr(), kClaimBlocks);
}

// Puts the pieces of cut walks together: dQ rows = scale x the sum of their partial results in the order of the pieces, dK and dV
// rows likewise.  A workgroup takes one unit of 32 rows of a whole item (the layout in which the pipelined kernel held it), each of
// its 4 waves a quarter of the accumulator; first the dQ units, then the dK/dV units.  Bound by the latency of reading the partial
// results (128 KB per block and piece, most of it written on another XCD).  A workgroup per whole block, its 8 waves a unit
// each, and a launch per kind took 8 - 26 us each: 557 causal tokens, 32/8 heads, 10.3 us, now 5.0; 918 queries on 4182 keys,
// 8/2 heads, 11.8 (dQ) and 26 (dK/dV), now 12.6 together.
template <int D>
__global__ __launch_bounds__(256) void bwd_merge_kernel(DqParams pq, const DqItem* __restrict__ dq_cut, int dq_units, DkvParams pk,
                                                        const DkvItem* __restrict__ dkv_cut) {
  constexpr int NQ = D / 8 / 4;  // accumulator quarters per wave
  constexpr int UNITS = D > 128 ? 4 : 8, KEY_UNITS = UNITS / 2;  // units per block, units of dV (then as many of dK)
  const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool is_dq = (int)blockIdx.x < dq_units;
  const int x = is_dq ? blockIdx.x : blockIdx.x - dq_units;
  const int unit = x % UNITS, block = x / UNITS;
  const int inner_n = is_dq ? pq.num_kv_heads * pq.head_splits : pk.num_kv_heads, inner = block % inner_n;
  int part, pieces, row, rows, head = 0;
  int64_t row0;
  if (is_dq) {
    const DqItem it = dq_cut[block / inner_n];
    part = it.part;
    pieces = it.pieces;
    head = inner % pq.num_kv_heads * pq.group + inner / pq.num_kv_heads * pq.heads_per_wg + unit % pq.heads_per_wg;
    row = (unit / pq.heads_per_wg) * 32 + l32;
    rows = it.q_rows;
    row0 = it.q_row0;
  } else {
    const DkvItem it = dkv_cut[block / inner_n];
    part = it.part;
    pieces = it.pieces;
    row = unit % KEY_UNITS * 32 + l32;
    rows = it.kv_rows;
    row0 = it.kv_row0;
  }
  if (row >= rows) return;
  const int64_t step = (int64_t)inner_n * kPartRowFloats;
  const float* src = (is_dq ? pq.parts : pk.parts) + part * step + (int64_t)inner * kPartRowFloats + unit * part_unit_floats(D) + wave * (NQ * 256) + lane * 4;
  f32x4 s[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) s[i] = *reinterpret_cast<const f32x4*>(src + i * 256);
#pragma unroll 4
  for (int k = 1; k < pieces; ++k) {
#pragma unroll
    for (int i = 0; i < NQ; ++i) s[i] += *reinterpret_cast<const f32x4*>(src + k * step + i * 256);
  }
  const int col = wave * (NQ * 8) + 4 * hh;
  if (is_dq) {
    __bf16* op = pq.dq + ((row0 + row) * pq.num_q_heads + head) * D + col;
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      *reinterpret_cast<bf16x4*>(op + 8 * i) = pack4(s[i][0] * pq.scale, s[i][1] * pq.scale, s[i][2] * pq.scale, s[i][3] * pq.scale);
  } else {
    __bf16* const out = unit < KEY_UNITS ? pk.dv : pk.dk;
    const float f = unit < KEY_UNITS ? 1.0f : pk.scale;
    const int64_t off = ((row0 + row) * pk.num_kv_heads + inner) * D + col;
#pragma unroll
    for (int i = 0; i < NQ; ++i) dkv_store4(pk, out, off + 8 * i, s[i][0] * f, s[i][1] * f, s[i][2] * f, s[i][3] * f);
  }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
size_t up256(size_t x) { return (x + 255) / 256 * 256; }
size_t n_dkv_blocks(const chunk_attn_desc* d) {
  size_t n = 0;
  for (int t = 0; t < d->num_segments; ++t) n += (d->segments[t].kv_len + dkv_keys(d->head_dim) - 1) / dkv_keys(d->head_dim);
  return n;
}

// Whether head_dim 64 runs its pipelined dK/dV kernel, given the walks of one key/value head.  Its blocks start and end more slowly than
// bwd_dkv_kernel's, which has several of them on a CU, so it needs two blocks per CU, 24 stages for each of the 512 workgroups that run at a time, and
// below three blocks per CU walks that are nearly equal or belong to several sequences, none with more than a quarter of the blocks (one or two long causal
// sequences put long walks on the same CU, which then ends last).
// Measured backward, bwd_dkv_kernel / pipelined (stages per workgroup): 64 sequences of 64, 8/8 heads (2) 28 / 38
// us; 64 of 128, 32/8 (16) 83 / 86; 64 of 256, 8/8 (12) 77 / 78; 32 of 256, 32/8 (24) 106 / 101; 128 of 128, 32/8 (32) 170 /
// 175; 64 of 256 (48) 217 / 202; 16 of 1024 (144) 478 / 390; 128 queries on 16384 keys (32) 325 / 320, 512 (126) 450 / 407.
// Causal sequences with 512 blocks, 32/8 heads: eight of 1024 265 / 215, four of 2048 438 / 365, two of 4096 604 / 647, one of
// 8192 1099 / 1222; 8/2: four of 8192 1554 / 1233, two of 16384 2256 / 2414; with 768 blocks: three of 4096 1028 / 811.
bool dkv_pipe_pays(const chunk_attn_desc* d, const Walks& w) {
  const int64_t blocks = w.items * d->num_kv_heads, stages = w.stages * d->num_kv_heads;
  if (blocks < 2 * kCus) return false;
  return stages >= 24 * 2 * kCus && (blocks >= 3 * kCus || 4 * w.largest <= w.items || 10 * stages >= 9 * 2 * kCus * w.longest);
}

// The walks of bwd_dkv_kernel's blocks (head_dim 64 and 256) are cut like those of 96 and 128 (choose_tile_split; its step is 0.6 us at 64,
// 1.4 at 256).  Backward, uncut / cut: head_dim 64, 1185 tokens behind 52, 32/8 heads, 134 / 71 us; 500 tokens, 64/8, 102 / 41; 4096
// tokens 460 / 329; 6000 741 / 700; 24000 tokens, 8/2, 2829 / 2541; head_dim 256, 2412 tokens, 8/2, 541 / 228; 1024 tokens, 32/8, 246 / 143;
// 3000 805 / 754.  What the estimate leaves alone (6500 tokens at 64, 3500 at 256) runs as before.
constexpr int64_t kMaxShortParts = 2 * kCus;  // partial results of such a chunk (64 MB at most)

// Whether a chunk of head_dim 64 or 256 runs its dQ and dK/dV blocks in one launch (bwd_short_kernel): where neither kind is pipelined with
// blocks of its own shape, as long as one grid holds both.  The kind with the longer walks goes first; at 64, dQ if they are equal.  (A dQ block
// of 64 holds the place of eight waves in that launch, which the other kind going on under it outweighs.)
// Backward, two launches / one: head_dim 64, four sequences of 256, 8/8 heads, 22.7 / 16.5 us; 1024 tokens 49.4 / 30.9; 3000 tokens 102 / 72; 1185
// tokens behind 52, 32/8, 67 / 48; 24 sequences of 200, 64/8, 142 / 125; 64 of 256, 8/8, 77.9 / 75.7 (dK/dV first 79.5); 128 of 256 143.5 / 143.4; 16
// times 64 queries on 2000 keys 91 / 67 (dK/dV first 99); head_dim 256, 512 tokens, 8/8, 65 / 38; 148 queries on 595 keys, 8/2, 71 / 42; 1500
// tokens, 64/8, 394 / 366; 300 queries on 3000 keys, 32/8, 231 / 162; 128 sequences of 128, 32/8, 733 / 700; 40 of 150, 8/8, 122 / 109 (dQ first 113).
bool short_joins(const BwdPlan& P, int64_t blocks, int threads) { return !P.dq_pipe && !P.dkv_pipe && blocks * threads < (int64_t)1 << 32; }

// workgroups of the pipelined dK/dV kernels on a CU
constexpr int dkv_per_cu(int head_dim) { return head_dim == 64 ? 2 : 1; }

// Raises a kernel's dynamic-LDS limit; callers keep the result in a function-local static, so that it happens once per
// process and is safe from several threads.
template <class K>
hipError_t raise_smem_limit(K kernel, size_t smem) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
}

template <int D>
hipError_t launch_bwd_t(const chunk_attn_desc* d, const BwdArgs& a, const BwdPlan& P, const std::vector<char>& blob, hipStream_t stream) {
  char* ws = a.workspace;
  float* lse2p = reinterpret_cast<float*>(ws + P.lse2p_off);
  float* dsp = reinterpret_cast<float*>(ws + P.dsp_off);
  hipError_t e;

  // pre-pass: D, scaled LSE
  {
    const int64_t blocks = (int64_t)P.qjobs.size() * d->num_q_heads;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const bool carry = blob.size() <= kInlineBlob;
    BwdPreArgs p;
    p.o = a.o; p.d_o = a.d_o; p.lse = a.lse;
    p.jobs = carry ? nullptr : reinterpret_cast<const TileJob*>(ws + P.qjobs_off);
    p.lse2p = lse2p; p.dsp = dsp;
    p.total_q_tiles = P.q_tiles; p.total_q = d->total_q; p.num_q_heads = d->num_q_heads;
    p.blob_dst = reinterpret_cast<u32x4*>(ws);
    p.blob_n16 = carry ? (int)(blob.size() / 16) : 0;
    p.jobs_off = (int)P.qjobs_off;
    if (carry) std::memcpy(p.blob, blob.data(), blob.size());
    static_assert(kInlineBlob <= 256 * 16, "one workgroup copies it");
    hipLaunchKernelGGL((bwd_pre_kernel<D>), dim3((unsigned)blocks), dim3(256), 0, stream, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = zero_uncovered(d, a, stream)) != hipSuccess) return e;

  const int group = d->num_q_heads / d->num_kv_heads;
  if constexpr (D == 128) {
    if (P.fused) return launch_bwd_fused(d, a, P, lse2p, dsp, stream);
  }
  DqParams pq;
  pq.q = a.q; pq.k = a.k; pq.v = a.v; pq.d_o = a.d_o; pq.lse2p = lse2p; pq.dsp = dsp; pq.dq = a.dq;
  pq.items = reinterpret_cast<const DqItem*>(ws + P.dq_items_off);
  pq.total_q_tiles = P.q_tiles;
  pq.num_q_heads = d->num_q_heads; pq.num_kv_heads = d->num_kv_heads; pq.group = group;
  pq.heads_per_wg = heads_per_wg(group, P.dq_waves); pq.head_splits = group / pq.heads_per_wg;
  pq.scale = d->softmax_scale; pq.scale_log2 = d->softmax_scale * kLog2e;
  pq.parts = reinterpret_cast<float*>(ws + P.dq_parts_off);
  pq.taken = reinterpret_cast<int32_t*>(ws + P.queues_off);
  pq.clock_log = clock_log(1);
  const int64_t dq_blocks = (int64_t)P.dq_items.size() * d->num_kv_heads * pq.head_splits;
  DkvParams pk;
  pk.q = a.q; pk.k = a.k; pk.v = a.v; pk.d_o = a.d_o; pk.lse2p = lse2p; pk.dsp = dsp;
  pk.dk = a.dk; pk.dv = a.dv;
  pk.items = reinterpret_cast<const DkvItem*>(ws + P.dkv_items_off);
  pk.total_q_tiles = P.q_tiles;
  pk.num_q_heads = d->num_q_heads; pk.num_kv_heads = d->num_kv_heads; pk.group = group;
  pk.scale = d->softmax_scale; pk.scale_log2 = d->softmax_scale * kLog2e;
  pk.accumulate = a.accumulate ? 1 : 0;
  pk.out_f32 = a.dkv_f32 ? 1 : 0;
  pk.taken = reinterpret_cast<int32_t*>(ws + P.queues_off) + kBlockQueues;
  pk.ended = pk.taken + kBlockQueues;
  pk.side_by_side = P.dkv_in_step ? persistent_grid(0x7fffffff) / kBlockQueues : 0;
  pk.parts = reinterpret_cast<float*>(ws + P.fdq_off);
  pk.clock_log = clock_log(2);
  static_assert(DKV_KEYS == 128, "the head_dim 64 and 128 kernels cover 128 keys per workgroup");
  const int64_t dkv_blocks = (int64_t)P.dkv_items.size() * d->num_kv_heads;
  if (dq_blocks > 0x7fffffff || dkv_blocks > 0x7fffffff) return hipErrorInvalidValue;
  pq.num_blocks = (int)dq_blocks;
  pk.num_blocks = (int)dkv_blocks;
  ProfileEvents pe = profile_events();
  profile_events() = ProfileEvents{};

  if constexpr (pipelined(D)) {
    // dQ: ring slots of a K and a V tile, then the staging tiles of the four waves (64 rows each).  dK/dV: ring slots of two 32-row
    // operand tiles, 2 P hand-over slots, one slot of LSE and D rows per ring slot, the word that announces the next block
    constexpr int NS = DKV_PIPE_DIST + 5;
    constexpr size_t dq_smem = (size_t)2 * (DQ_PIPE_DIST + 3) * 32 * D * 2 + (size_t)4 * 64 * D * 2;
    constexpr size_t dkv_smem = (size_t)2 * NS * 32 * D * 2 + 2 * 4096 * 2 + 2 * NS * 64 * sizeof(float) + 16;
    constexpr size_t smem = dq_smem > dkv_smem ? dq_smem : dkv_smem;
    if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return e;
    // the blocks of one kind or of both, then their pieces put together
    auto run = [&](bool dq, bool dkv) {
      BwdPipeParams p;
      p.dq = pq;
      p.dkv = pk;
      p.dq_phase = P.dq_first ? 0 : 1;
      if (!dq) p.dq.num_blocks = 0;
      if (!dkv) p.dkv.num_blocks = 0;
      const size_t n_dq_cut = dq ? P.n_dq_cut : 0, n_dkv_cut = dkv ? P.n_dkv_cut : 0;
      const dim3 grid((unsigned)persistent_grid((int64_t)p.dq.num_blocks + p.dkv.num_blocks));
      if (P.dkv_tall) {
        static const hipError_t attr = raise_smem_limit(&bwd_pipe_kernel<D, false, true>, smem);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((bwd_pipe_kernel<D, false, true>), grid, dim3(256), smem, stream, p);
        return hipGetLastError();
      }
      if (n_dq_cut == 0 && n_dkv_cut == 0) {
        static const hipError_t attr = raise_smem_limit(&bwd_pipe_kernel<D, false, false>, smem);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((bwd_pipe_kernel<D, false, false>), grid, dim3(256), smem, stream, p);
        return hipGetLastError();
      }
      static const hipError_t attr = raise_smem_limit(&bwd_pipe_kernel<D, true, false>, smem);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL((bwd_pipe_kernel<D, true, false>), grid, dim3(256), smem, stream, p);
      const hipError_t err = hipGetLastError();
      if (err != hipSuccess) return err;
      const int64_t dq_units = 8 * (int64_t)n_dq_cut * d->num_kv_heads * pq.head_splits, dkv_units = 8 * (int64_t)n_dkv_cut * d->num_kv_heads;
      // (cut chunks have few blocks: choose_key_split, choose_tile_split)
      hipLaunchKernelGGL((bwd_merge_kernel<D>), dim3((unsigned)(dq_units + dkv_units)), dim3(256), 0, stream, pq,
                         reinterpret_cast<const DqItem*>(ws + P.dq_cut_off), (int)dq_units, pk,
                         reinterpret_cast<const DkvItem*>(ws + P.dkv_cut_off));
      return hipGetLastError();
    };
    if (P.in_turn) {
      if ((e = run(true, false)) != hipSuccess || (e = run(false, true)) != hipSuccess) return e;
    } else if ((e = run(true, true)) != hipSuccess) {
      return e;
    }
  } else {
    constexpr int KB = (D > 128 ? 64 : DKV_KEYS) / 32;  // as dkv_keys(D)
    // 4 ring slots of two 32-row operand tiles, 2 P hand-over slots, 4 slots of LSE and D rows
    constexpr size_t dkv_smem = (size_t)8 * 32 * D * 2 + 2 * KB * 1024 * 2 + 2 * 4 * 64 * sizeof(float);
    const bool joint = short_joins(P, dq_blocks + dkv_blocks, KB * 128);
    if (joint) {
      BwdPipeParams p;
      p.dq = pq;
      p.dkv = pk;
      p.dq_phase = P.dq_first ? 0 : 1;
      const dim3 grid((unsigned)(dq_blocks + dkv_blocks));
      auto run = [&](auto cut_c, auto wide_c) {
        constexpr bool CUT = decltype(cut_c)::value, WIDE = decltype(wide_c)::value;
        constexpr size_t dq_smem = (size_t)(WIDE ? 10 : 6) * 32 * D * 2, smem = dq_smem > dkv_smem ? dq_smem : dkv_smem;  // (as below)
        static const hipError_t attr = raise_smem_limit(&bwd_short_kernel<D, KB, CUT, WIDE>, smem);
        if (attr != hipSuccess) return attr;
        hipError_t err;
        if (pe.start && (err = hipEventRecord(pe.start, stream)) != hipSuccess) return err;
        hipLaunchKernelGGL((bwd_short_kernel<D, KB, CUT, WIDE>), grid, dim3(KB * 128), smem, stream, p);
        return hipGetLastError();
      };
      const std::bool_constant<D == 256> wide;
      if (P.n_dkv_cut == 0) e = P.dq_wide ? run(std::false_type{}, wide) : run(std::false_type{}, std::false_type{});
      else e = P.dq_wide ? run(std::true_type{}, wide) : run(std::true_type{}, std::false_type{});
      if (e != hipSuccess) return e;
    } else if ((D == 256 && P.dkv_pipe) || (D == 64 && P.dkv_tall)) {
      BwdPipeParams p;
      p.dq = pq;
      p.dkv = pk;
      p.dq_phase = P.dq_first ? 0 : 1;
      // 256: six ring slots of K and four of V, and as many of two 32-row operand tiles and of their LSE and D rows as dkv_wide_blocks has; 64: as at 96 and 128
      constexpr int kSlots = D == 256 ? 4 : 8;
      constexpr size_t dq_smem = D == 256 ? (size_t)10 * 32 * D * 2 : (size_t)2 * (DQ_PIPE_DIST + 3) * 32 * D * 2 + (size_t)4 * 64 * D * 2;
      constexpr size_t dkv_smem = (size_t)2 * kSlots * 32 * D * 2 + 2 * kSlots * 64 * sizeof(float) + 16, smem = dq_smem > dkv_smem ? dq_smem : dkv_smem;
      static const hipError_t attr = raise_smem_limit(&bwd_pipe_kernel<D, false, true>, smem);
      if (attr != hipSuccess) return attr;
      if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return e;
      hipLaunchKernelGGL((bwd_pipe_kernel<D, false, true>), dim3((unsigned)persistent_grid(dq_blocks + dkv_blocks)), dim3(256), smem, stream, p);
    } else if (D == 256 && P.dq_wide) {
      const size_t smem = (size_t)10 * 32 * D * 2;  // six slots of K and four of V
      static const hipError_t attr = raise_smem_limit(&bwd_dq_wide_kernel, smem);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL(bwd_dq_wide_kernel, dim3((unsigned)persistent_grid(dq_blocks)), dim3(256), smem, stream, pq);
    } else if (D == 64 && P.dq_pipe) {
      const size_t smem = (size_t)2 * (DQ_PIPE_DIST + 3) * 32 * D * 2 + (size_t)4 * 64 * D * 2;
      static const hipError_t attr = raise_smem_limit(&bwd_dq_pipe_kernel, smem);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL(bwd_dq_pipe_kernel, dim3((unsigned)persistent_grid(dq_blocks)), dim3(256), smem, stream, pq);
    } else {
      const size_t smem = (size_t)6 * 32 * D * 2;  // 3 stages of K and V tiles
      constexpr int DQW = 4;
      static const hipError_t attr = raise_smem_limit(&bwd_dq_kernel<D, DQW>, smem);
      if (attr != hipSuccess) return attr;
      hipLaunchKernelGGL((bwd_dq_kernel<D, DQW>), dim3((unsigned)dq_blocks), dim3(DQW * 64), smem, stream, pq);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if constexpr (D == 64) {
      if (P.dkv_pipe && !P.dkv_tall) {
        // 6 ring slots of two 32-row operand tiles and their LSE and D rows
        const size_t smem = (size_t)2 * 6 * 32 * D * 2 + 2 * 6 * 64 * sizeof(float);
        static const hipError_t attr = raise_smem_limit(&bwd_dkv_narrow_pipe_kernel<D>, smem);
        if (attr != hipSuccess) return attr;
        if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return e;
        hipLaunchKernelGGL((bwd_dkv_narrow_pipe_kernel<D>), dim3((unsigned)persistent_grid(dkv_blocks, dkv_per_cu(D))), dim3(128), smem, stream, pk,
                           (int)dkv_blocks);
      }
    }
    if (!joint && !P.dkv_pipe) {
      if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return e;
      if (P.n_dkv_cut == 0) {
        static const hipError_t attr = raise_smem_limit(&bwd_dkv_kernel<D, KB, false>, dkv_smem);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((bwd_dkv_kernel<D, KB, false>), dim3((unsigned)dkv_blocks), dim3(KB * 128), dkv_smem, stream, pk);
      } else {
        static const hipError_t attr = raise_smem_limit(&bwd_dkv_kernel<D, KB, true>, dkv_smem);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((bwd_dkv_kernel<D, KB, true>), dim3((unsigned)dkv_blocks), dim3(KB * 128), dkv_smem, stream, pk);
      }
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (P.n_dkv_cut > 0)
      hipLaunchKernelGGL((bwd_merge_kernel<D>), dim3((unsigned)(2 * KB * P.n_dkv_cut * d->num_kv_heads)), dim3(256), 0, stream, pq,
                         static_cast<const DqItem*>(nullptr), 0, pk, reinterpret_cast<const DkvItem*>(ws + P.dkv_cut_off));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (pe.stop && (e = hipEventRecord(pe.stop, stream)) != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace

hipError_t zero_uncovered(const chunk_attn_desc* d, const BwdArgs& a, hipStream_t stream) {
  if (a.accumulate) return hipSuccess;
  for (const auto& gap : uncovered_kv_ranges(d)) {
    const int64_t row = (int64_t)d->num_kv_heads * d->head_dim * (a.dkv_f32 ? 4 : 2);  // bytes
    const int64_t n16 = (gap.second - gap.first) * row / 16;
    for (__bf16* base : {a.dk, a.dv})
      hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, stream,
                         reinterpret_cast<u32x4*>(reinterpret_cast<char*>(base) + gap.first * row), n16);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

int dkv_block_keys(const BwdPlan& P, int head_dim) { return P.dkv_tall ? kTallKeys : head_dim == 256 && P.dkv_pipe ? kWideKeys : dkv_keys(head_dim); }

void bwd_layout(const chunk_attn_desc* d, BwdPlan& P, bool with_plan, Cut cut, int share_dim) {
  P = BwdPlan{};
  const int group = d->num_q_heads / d->num_kv_heads;
  const bool pipe = d->head_dim == 128;
  P.dq_waves = pipe ? 8 : 4;
  P.dq_pipe = P.dkv_pipe = pipe;
  if (d->head_dim == 64) {
    P.dq_pipe = pipe_pays(count_walks(d, tile_rows(group, 8)), d->num_kv_heads * (group / heads_per_wg(group, 8)));
    if (P.dq_pipe) P.dq_waves = 8;
  }
  const int dq_rows = tile_rows(group, P.dq_waves);
  if (d->head_dim == 64) P.dkv_pipe = dkv_pipe_pays(d, count_dkv_walks(d, dkv_keys(64)));
  if (d->head_dim == 256) P.dkv_pipe = wide_pays(d, dq_rows, d->num_kv_heads * (group / heads_per_wg(group, P.dq_waves)), dkv_keys(256), kCus);
  if (d->head_dim == 256) P.dq_wide = P.dkv_pipe || dq_wide_pays(count_walks(d, dq_rows));
  if (d->head_dim == 64 && P.dq_pipe && P.dkv_pipe) P.dkv_tall = narrow_tall_pays(group, count_dkv_walks(d, dkv_keys(64)));
  P.q_tiles = count_tiles(d, false, 64);
  P.qt32_tiles = count_tiles(d, false, 32);
  // head_dim 128: room for dQ tiles in float32, for the one-pass backward or for the partial results of cut dQ walks
  const size_t dq_tile_bytes = pipe ? (size_t)fused_num_bufs(d, dkv_keys(128)) * d->num_q_heads * P.qt32_tiles * 4096 * sizeof(float) : 0;
  P.fused = d->head_dim == 128 && bwd_mode() == 2;
  size_t n_dq = 0, n_dkv = 0;
  if (pipe && cut > kCutNone) {  // (in either mode: the pieces are part of the layout, whose size must not depend on the mode)
    const int inner = d->num_kv_heads * (group / heads_per_wg(group, P.dq_waves));
    // Whether walks are cut is decided for as many partial results as the float32 dQ tiles have room for; into how many pieces, for
    // all blocks of the launch together and with room for two partial results per compute unit.  Forward + backward, one decision / two: 439
    // tokens, 8/2 heads, 67 / 56 us; 557 tokens, 32/8, 73 / 68; slices of 918 and 3264 queries, 8/2, 255 / 240; a hybrid chunk of 1742
    // queries behind 23348 keys with 3732 packed tokens, 8/8, 996 / 945.  (Finer pieces of each kind by itself: 1144 tokens, 32/8, 110 / 122.)
    const int64_t room = (int64_t)(dq_tile_bytes / ((size_t)kPartRowFloats * sizeof(float)));
    P.split = choose_key_split(d, dq_rows, inner, kCus, room / inner);
    P.dkv_split = choose_tile_split(d, dkv_keys(d->head_dim), kCus, room / d->num_kv_heads);
    if (cut == kCutFine) refine_bwd_split(d, dq_rows, inner, dkv_keys(d->head_dim), kCus, std::max(room, kMaxShortParts), &P.split, &P.dkv_split);
  }
  if (!pipe && !P.dkv_pipe && cut == kCutFine)
    P.dkv_split = choose_tile_split(d, dkv_keys(d->head_dim), kCus, kMaxShortParts / d->num_kv_heads);
  if (share_dim > 0 && (pipe || (d->head_dim == 64 && !P.dq_pipe)) && shared_backward_fits(d))  // (before walks are counted)
    P.share_waves = choose_shared_waves(d, share_dim, count_walks(d, dq_rows), d->num_kv_heads * (group / heads_per_wg(group, P.dq_waves)),
                                        count_dkv_walks(d, dkv_keys(d->head_dim)), P.split, P.dkv_split);
  // (kCutFine: what runs where a workspace is too small for a chunk's cut keeps to the blocks of the cut run, whose sums it repeats but for their order)
  if (pipe && cut == kCutFine && !P.fused && P.share_waves == 0 && P.split.target == 0 && P.dkv_split.target == 0)
    P.dkv_tall = tall_pays(d, dq_rows, d->num_kv_heads * (group / heads_per_wg(group, P.dq_waves)), dkv_keys(d->head_dim), kCus);
  if (with_plan && P.share_waves == 0) {
    if (P.fused) {
      P.fplan = plan_fused(d, dkv_keys(d->head_dim), kNumXcd, fused_num_bufs(d, dkv_keys(d->head_dim)));
    } else {
      P.dq_items = plan_dq(d, dq_rows);
      if (P.split.target > 0) P.dq_items = cut_items(P.dq_items, P.split.target, &P.dq_cut);
      // the pipelined kernels walk either way; the key blocks of one key/value head that run at the same time are the
      // workgroups of the launch over the number of key/value heads
      const int side_by_side = P.dkv_pipe ? std::max(1, persistent_grid(0x7fffffff, P.dkv_tall ? 1 : dkv_per_cu(d->head_dim)) / d->num_kv_heads) : 0;
      P.dkv_items = plan_dkv(d, dkv_block_keys(P, d->head_dim), P.dkv_split.target > 0 ? 0 : side_by_side);
      if (P.dkv_split.target > 0) P.dkv_items = cut_items(P.dkv_items, P.dkv_split.target, &P.dkv_cut);
    }
    P.qjobs = query_tile_jobs(d, 64);
    int dq_longest = 0, dkv_longest = 0;
    for (const DqItem& it : P.dq_items) dq_longest = std::max(dq_longest, (std::min(it.n0 + it.q_rows - 1, it.keys) + kStageKeys - 1) / kStageKeys);
    for (const DkvItem& it : P.dkv_items) dkv_longest = std::max(dkv_longest, (it.n_qt - it.qt_first) * group);
    P.dq_first = dq_longest > dkv_longest || (d->head_dim == 64 && dq_longest == dkv_longest);  // (64: short_joins)
    P.dkv_in_step = pipe && !P.dq_first && dkv_longest >= kStepsInStep;
  }
  // the layout does not depend on which backward runs: item and piece counts follow from the segment table
  for (int t = 0; t < d->num_segments; ++t) {
    n_dq += (d->segments[t].q_len + dq_rows - 1) / dq_rows;
    n_dkv += (d->segments[t].kv_len + dkv_keys(d->head_dim) - 1) / dkv_keys(d->head_dim);
  }
  // (cut walks: the pieces, then the whole items that were cut)
  auto up16 = [](size_t x) { return (x + 15) / 16 * 16; };
  P.n_dq_cut = n_dq - (size_t)(P.split.target > 0 ? P.split.pieces - P.split.parts : (int64_t)n_dq);
  P.n_dkv_cut = n_dkv - (size_t)(P.dkv_split.target > 0 ? P.dkv_split.pieces - P.dkv_split.parts : (int64_t)n_dkv);
  P.dq_items_off = 0;
  P.dq_cut_off = up16((P.split.target > 0 ? (size_t)P.split.pieces : n_dq) * sizeof(DqItem));
  P.dkv_items_off = P.dq_cut_off + up16(P.n_dq_cut * sizeof(DqItem));
  P.dkv_cut_off = P.dkv_items_off + up16((P.dkv_split.target > 0 ? (size_t)P.dkv_split.pieces : n_dkv) * sizeof(DkvItem));
  P.qjobs_off = P.dkv_cut_off + up16(P.n_dkv_cut * sizeof(DkvItem));
  // block-queue counters of the dQ and of the dK/dV kernel (zero in the blob): dQ queues, dK/dV queues, dK/dV blocks ended
  P.queues_off = P.qjobs_off + up16((size_t)P.q_tiles * sizeof(TileJob));
  P.fitems_off = P.queues_off + up16(3 * kBlockQueues * sizeof(int32_t));
  // the workspace is sized for either backward (the mode may change between the size query and the call): the one-pass
  // backward has one item per (key block, key/value head) and at most 8 x that many workgroup slots
  const size_t n_fused = d->head_dim == 128 ? n_dkv_blocks(d) * (size_t)d->num_kv_heads : 0;
  P.forder_off = P.fitems_off + up16(n_fused * sizeof(FusedItem));
  P.q32jobs_off = P.forder_off + up16(n_fused * kNumXcd * sizeof(int32_t));
  P.blob_bytes = up256(P.q32jobs_off + (d->head_dim == 128 ? (size_t)P.qt32_tiles * sizeof(DqTileJob) : 0));
  P.upload_bytes = P.fused ? P.blob_bytes : P.fitems_off;
  const size_t row_slots = (size_t)d->num_q_heads * P.q_tiles * 64;
  P.fprog_off = P.blob_bytes;
  // progress counters, then the status word (its own 256 bytes), then a scratch tile
  P.fprog_bytes = up256(n_fused * 4 * sizeof(unsigned)) + 256 + kFusedSinkBytes;
  P.lse2p_off = P.fprog_off + P.fprog_bytes;
  P.dsp_off = P.lse2p_off + up256(row_slots * sizeof(float));
  // (256 bytes remain: the dK/dV kernels copy the LSE / D rows 64 at a time, up to 32 past a segment's last)
  P.fdq_off = P.dsp_off + up256(row_slots * sizeof(float)) + 256;
  // partial results of cut walks: those of dK/dV, then those of dQ, as both kinds of block run in one launch; where the room is
  // that of the dQ tiles and too small for both, each kind has all of it in turn, in a launch of its own
  P.dq_parts_off = P.fdq_off + up256((size_t)P.dkv_split.parts * d->num_kv_heads * kPartRowFloats * sizeof(float));
  const size_t dq_part_bytes = P.split.parts > 0 ? (size_t)P.split.parts * d->num_kv_heads * (group / heads_per_wg(group, P.dq_waves)) * kPartRowFloats * sizeof(float) : 0;
  P.in_turn = cut == kCutInPlace && P.dkv_split.parts > 0 && P.split.parts > 0 && P.dq_parts_off + dq_part_bytes > P.fdq_off + dq_tile_bytes;
  if (P.in_turn) P.dq_parts_off = P.fdq_off;
  P.total = std::max(P.fdq_off + dq_tile_bytes, P.dq_parts_off + dq_part_bytes);
}

std::vector<char> bwd_blob(const BwdPlan& P) {
  std::vector<char> blob(P.upload_bytes);
  std::memcpy(blob.data() + P.dq_items_off, P.dq_items.data(), P.dq_items.size() * sizeof(DqItem));
  std::memcpy(blob.data() + P.dq_cut_off, P.dq_cut.data(), P.dq_cut.size() * sizeof(DqItem));
  std::memcpy(blob.data() + P.dkv_items_off, P.dkv_items.data(), P.dkv_items.size() * sizeof(DkvItem));
  std::memcpy(blob.data() + P.dkv_cut_off, P.dkv_cut.data(), P.dkv_cut.size() * sizeof(DkvItem));
  std::memcpy(blob.data() + P.qjobs_off, P.qjobs.data(), P.qjobs.size() * sizeof(TileJob));
  if (P.fused) {
    std::memcpy(blob.data() + P.fitems_off, P.fplan.items.data(), P.fplan.items.size() * sizeof(FusedItem));
    std::memcpy(blob.data() + P.forder_off, P.fplan.order.data(), P.fplan.order.size() * sizeof(int32_t));
    std::memcpy(blob.data() + P.q32jobs_off, P.fplan.tiles.data(), P.fplan.tiles.size() * sizeof(DqTileJob));
  }
  return blob;
}

hipError_t launch_bwd(const chunk_attn_desc* d, const BwdArgs& a, const BwdPlan& P, const std::vector<char>& blob, hipStream_t stream) {
  return d->head_dim == 128 ? launch_bwd_t<128>(d, a, P, blob, stream)
         : d->head_dim == 96 ? launch_bwd_t<96>(d, a, P, blob, stream)
         : d->head_dim == 256 ? launch_bwd_t<256>(d, a, P, blob, stream) : launch_bwd_t<64>(d, a, P, blob, stream);
}

}  // namespace chunk_attn

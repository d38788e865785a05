// Chunk attention backward of small chunks in one launch (head_dim 64, 96 and 128): no pre-pass, no list in device memory, no merge.
//
// The W waves of a workgroup share one small output tile and divide the walk that makes it:
//   dQ      32 query rows of one head; wave w takes key stages w, w + W, ... of 32 keys:
//           S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - D), dQ^T += K^T dS^T
//   dK, dV  32 keys of one key/value head; wave w takes every W-th (query tile, head of the group) of those that see them:
//           S = Q K^T, dP = dO V^T, dV^T += dO^T P, dS = P (dP - D), dK^T += Q^T dS
// Either way a wave keeps two tiles as fragments (Q and dO, or K and V), copies its own stages of two tiles (K and V, or Q and dO) into
// its own LDS slots, so that it waits for nothing but its copies, and the waves' sums meet in LDS at the end, added in wave order.
// D_i = <dO_i, O_i> is made where it is used: by a dQ workgroup for its 32 rows, by a dK/dV wave for every stage (O comes in registers
// a stage ahead, in the order in which the copies lay out dO).
// Tiles are rows swizzled by share_swz, as in fwd_share_kernel.
//
// Why: such a chunk's backward was three or four launches one after the other (pre-pass 4 us, dQ and dK/dV blocks, merge of cut walks 5 us), each
// a serial chain of stages on few compute units.  Backward before -> now, us: head_dim 64, 8/8 heads, sequences of 256, 512, 128 and 128, 19.5 ->
// 10.4; 100 queries on 10100 keys, 32/8, 175 -> 72; head_dim 128, 8/8, 500 tokens, 33.4 -> 14.7.
// What is left is the start (arguments, first copies: 4 - 6 us), the chain of a wave (0.6 us a dQ stage and 1.1 a dK/dV stage at 64 with four waves, 1.0
// and 1.8 at 128, one wave per SIMD) and the sums.  A dK/dV stage at 128 took 2.5 us with the rows of every copy clamped (a multiplication each), 2.2
// without, 2.05 once O's loads were waited for ahead of the copies (rows_loaded), 1.84 with D by v_dot2 and copies from a scalar base.
// Four waves (64: two workgroups per compute unit) or eight: choose_shared_waves.
#include <type_traits>

#include "kernels.hpp"
#include "tiles.hpp"

namespace chunk_attn {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct ShareParams {
  const __bf16 *q, *k, *v, *o, *d_o;
  const float* lse;
  __bf16 *dq, *dk, *dv;
  int32_t total_q, num_q_heads, num_kv_heads, group;
  float scale, scale_log2;
  int32_t accumulate, out_f32;
  int32_t dq_blocks, dkv_blocks, dq_first;
};
// A block is (segment, tile of 32 rows of its queries or keys).  In the kernel arguments: 4 KB are documented for a launch.
struct ShareItem {
  uint16_t seg, tile;
};
struct ShareArgs {
  ShareParams p;
  chunk_attn_seg segs[kMaxShareSegs];
  ShareItem items[kMaxShareItems];  // dQ, then dK/dV
};
static_assert(sizeof(ShareArgs) <= 3840);

// LDS: W waves' slots (two stages of two tiles each; at the end the wave's sums), the two stationary tiles, 32 values of LSE and of -D per wave
template <int D, int W>
constexpr size_t share_bwd_smem() { return (size_t)(W * 4 + 2) * 32 * share_cols(D) * 2 + (size_t)W * 64 * sizeof(float); }

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
// sum over the C (8 or 16) consecutive lanes that hold a row's chunks, in each of them
template <int C>
__device__ __forceinline__ float sum_row(float x) {
  x = dpp_add<0xb1>(x);   // lanes 1 apart
  x = dpp_add<0x4e>(x);   // 2 apart
  x = dpp_add<0x141>(x);  // the other half of eight
  if constexpr (C == 16) x = dpp_add<0x140>(x);  // the other eight of sixteen
  return x;
}
__device__ __forceinline__ float dot8(bf16x8 a, bf16x8 b) {
  float s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), 0.f, false);
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), s, false);
  s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), s, false);
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), s, false);
}
__device__ __forceinline__ bf16x8 join(s16x4 lo, s16x4 hi) {
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// What both kinds of block use: the lane's place in copies and operand reads.
template <int D>
struct ShareLane {
  static constexpr int ROW = share_cols(D) * 2, C = ROW / 16, PT = C / 2, RPC = 64 / C, TILE = 32 * ROW;  // ROW: bytes of a row in LDS
  int lane, l32, hh, c_row, c_chunk;
  unsigned row_at, tr_at;  // byte offsets in a tile of the row reads and of the transposed reads
  __device__ __forceinline__ ShareLane() {
    lane = threadIdx.x & 63;
    l32 = lane & 31;
    hh = lane >> 5;
    c_row = lane / C;
    c_chunk = (lane % C) ^ share_swz<D>(c_row);
    row_at = (unsigned)(l32 * ROW + ((hh ^ share_swz<D>(l32)) * 16));
    const int j = lane & 15, cl = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1), r0 = 4 * hh + (j >> 2);
    tr_at = (unsigned)(r0 * ROW + ((cl ^ share_swz<D>(r0)) * 16) + 8 * (j & 1));
  }
  template <int I>
  __device__ __forceinline__ int column() const {  // of the lane's chunk in copy I of a tile
    const int chunk = c_chunk ^ share_swz<D>(RPC * I);
    return (D == 96 ? min(chunk, D / 8 - 1) : chunk) * 8;
  }
  template <int I>
  __device__ __forceinline__ bool in_row() const { return D != 96 || (c_chunk ^ share_swz<D>(RPC * I)) < D / 8; }  // it is one of the row's
  // The chunk, of rows of `stride` elements, that copy i of a tile puts at this lane's place; rows past `last` (< 31) repeat it, which costs a
  // multiplication for every copy: whole tiles find their chunks a scalar row and a constant XOR away from `c_off` = c_row * stride.
  template <int I>
  __device__ __forceinline__ const __bf16* chunk(const __bf16* src, int stride, int c_off, int last) const {
    const int col = column<I>();
    if (last >= 31)  // (bytes, so that the address is a scalar base and a 32-bit offset)
      return reinterpret_cast<const __bf16*>(reinterpret_cast<const char*>(src + (int64_t)(RPC * I) * stride) + (unsigned)(2 * c_off + 2 * col));
    return src + (int64_t)min(RPC * I + c_row, last) * stride + col;
  }
  __device__ __forceinline__ void copy_tile(const __bf16* src, int stride, int c_off, int last, lds_bf16* dst) const {
    if (last >= 31)
      static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        dma16(chunk<i>(src, stride, c_off, 31), dst + i * 512);
      });
    else
      static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        dma16(src + (int64_t)min(RPC * i + c_row, last) * stride + column<i>(), dst + i * 512);
      });
  }
};

// The waves' sums of NT tiles (f32x16 x DB each, in accumulator order) added in wave order: each wave gets NT * DB * 4 / W quarters of 8
// columns.  `use(quarter, sum)` is called for each of the wave's own.
template <int D, int W, int N, class F>
__device__ __forceinline__ void add_shares(char* smem, int wave, int lane, int parts, const f32x16 (&acc)[N], F&& use) {
  constexpr int NQ = N * 4, NQW = NQ / W, REGION = 4 * 32 * share_cols(D) * 2;
  static_assert(NQ % W == 0 && NQ * 1024 <= REGION);
  if (wave < parts) {
    lds_f32* const out = (lds_f32*)(smem + wave * REGION) + lane * 4;
#pragma unroll
    for (int x = 0; x < NQ; ++x)
      *(__attribute__((address_space(3))) f32x4*)(out + x * 256) =
          f32x4{acc[x / 4][4 * (x % 4)], acc[x / 4][4 * (x % 4) + 1], acc[x / 4][4 * (x % 4) + 2], acc[x / 4][4 * (x % 4) + 3]};
  }
  __syncthreads();
  const lds_f32* const src = (const lds_f32*)smem + wave * NQW * 256 + lane * 4;
  f32x4 s[NQW];
#pragma unroll
  for (int x = 0; x < NQW; ++x) s[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int w = 0; w < parts; ++w)
#pragma unroll
    for (int x = 0; x < NQW; ++x) s[x] += lds_load4f(src + w * (REGION / 4) + x * 256);
#pragma unroll
  for (int x = 0; x < NQW; ++x) use(wave * NQW + x, s[x]);
}

template <int D, int W>
__device__ __forceinline__ void share_dq_block(const ShareParams& p, const chunk_attn_seg seg, int tile, int inner, char* smem) {
  constexpr int DK = D / 16, DB = D / 32;
  typedef ShareLane<D> Lane;
  constexpr int TILE = Lane::TILE, PT = Lane::PT, RPC = Lane::RPC;
  const Lane L;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kvh = inner % p.num_kv_heads, head = kvh * p.group + inner / p.num_kv_heads;
  const int q_rows = min(32, seg.q_len - 32 * tile), n0 = seg.kv_len - seg.q_len + 32 * tile + 1;
  const int n_keys = n0 + q_rows - 1, nt = (n_keys + 31) / 32, n_mine = nt > wave ? (nt - wave + W - 1) / W : 0;
  const int q_stride = p.num_q_heads * D, kv_stride = p.num_kv_heads * D, kv_c = L.c_row * kv_stride, q_c = L.c_row * q_stride;
  const int64_t q_off = (int64_t)(seg.q_start + 32 * tile) * q_stride + head * D;
  const __bf16* const Kg = p.k + (int64_t)seg.kv_start * kv_stride + (int64_t)kvh * D;
  const __bf16* const Vg = p.v + (int64_t)seg.kv_start * kv_stride + (int64_t)kvh * D;
  lds_bf16* const region = (lds_bf16*)(smem + wave * 4 * TILE);
  lds_bf16* const own = (lds_bf16*)(smem + W * 4 * TILE);                // Q, dO
  lds_f32* const rows = (lds_f32*)(smem + (W * 4 + 2) * TILE);           // LSE log2(e) [32], -D [32]

  // ---- the waves together: Q and dO tiles, D and LSE of the rows ----
  float nd[PT];
  static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value;
    if (i % W == wave) {
      const float x = dot8(*reinterpret_cast<const bf16x8*>(L.template chunk<i>(p.o + q_off, q_stride, q_c, q_rows - 1)),
                           *reinterpret_cast<const bf16x8*>(L.template chunk<i>(p.d_o + q_off, q_stride, q_c, q_rows - 1)));
      nd[i] = L.template in_row<i>() ? x : 0.f;
    }
  });
  float lse2 = 0.f;
  if (wave == W - 1) lse2 = p.lse[(int64_t)head * p.total_q + seg.q_start + 32 * tile + min(L.l32, q_rows - 1)] * kLog2e;
  static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value;
    if (i % W == wave) {
      dma16(L.template chunk<i>(p.q + q_off, q_stride, q_c, q_rows - 1), own + i * 512);
      dma16(L.template chunk<i>(p.d_o + q_off, q_stride, q_c, q_rows - 1), own + TILE / 2 + i * 512);
    }
  });
  static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value;
    if (i % W == wave) {
      const float s = sum_row<Lane::C>(nd[i]);
      if (L.lane % Lane::C == 0) lds_asm_write4(lds_addr(rows + 32 + RPC * i + L.c_row), (int)__float_as_uint(-s));
    }
  });
  if (wave == W - 1 && L.lane < 32) lds_asm_write4(lds_addr(rows + L.lane), (int)__float_as_uint(lse2));
  auto copy_stage = [&](int i, int slot) __attribute__((always_inline)) {
    const int t = wave + W * min(i, n_mine - 1);
    const int64_t off = (int64_t)(32 * t) * kv_stride;
    L.copy_tile(Kg + off, kv_stride, kv_c, n_keys - 1 - 32 * t, region + slot * TILE);
    L.copy_tile(Vg + off, kv_stride, kv_c, n_keys - 1 - 32 * t, region + slot * TILE + TILE / 2);
  };
  if (n_mine > 0) {
    copy_stage(0, 0);
    copy_stage(1, 1);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * PT) : "memory");  // (all but the stages' copies)
  } else {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  }
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16;
  bf16x8 qf[DK], gf[DK];
  {
    const unsigned base = lds_addr(own) + L.row_at;
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      qf[ks] = lds_asm_read16<0>(base ^ (ks * 32));
      gf[ks] = lds_asm_read16<TILE>(base ^ (ks * 32));
    });
  }
  float row_lse, row_nd;
  asm volatile("ds_read_b32 %0, %1" : "=v"(row_lse) : "v"(lds_addr(rows + L.l32)) : "memory");
  asm volatile("ds_read_b32 %0, %1" : "=v"(row_nd) : "v"(lds_addr(rows + 32 + L.l32)) : "memory");
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(row_lse), "+v"(row_nd)::"memory");
#pragma unroll
  for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(qf[ks]), "+v"(gf[ks]));

  const float c = p.scale_log2;
  const unsigned k_base = lds_addr(region) + L.row_at, t_base = lds_addr(region) + L.tr_at;
  for (int i = 0; i < n_mine; ++i) {
    const int t = wave + W * i, slot = i & 1;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PT) : "memory");  // the stage after this one may be outstanding
    const unsigned ka = k_base + slot * (2 * TILE), ta = t_base + slot * (2 * TILE);
    bf16x8 kf[DK], vf[DK];
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      kf[ks] = lds_asm_read16<0>(ka ^ (ks * 32));
    });
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      vf[ks] = lds_asm_read16<TILE>(ka ^ (ks * 32));
    });
    f32x16 s, dp;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));
    s16x4 lo[2][DB], hi[2][DB];  // operands of dQ^T += K^T dS^T
    static_for<0, 2 * DB>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(x_c)::value / DB, db = decltype(x_c)::value % DB;
      lo[ks][db] = lds_asm_read_tr<ks * 16 * Lane::ROW>(ta ^ (db * 64));
      hi[ks][db] = lds_asm_read_tr<(ks * 16 + 8) * Lane::ROW>(ta ^ (db * 64 + share_swz<D>(8) * 16));
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {  // (two chains of products, one between the other's)
      s = mfma32(kf[ks], qf[ks], ks == 0 ? zero16 : s);
      dp = mfma32(vf[ks], gf[ks], ks == 0 ? zero16 : dp);
    }
    float pe[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) pe[e] = __builtin_amdgcn_exp2f(s[e] * c - row_lse);
    if (32 * t + 32 > n0) {
      const int lim = n0 + L.l32 - 32 * t;  // visible iff local key index < lim
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + 4 * L.hh + (e & 3) >= lim) pe[e] = 0.f;
    }
    bf16x8 f[2];
    {
      float w[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) w[e] = pe[e] * (dp[e] + row_nd);
      f[0] = pack8(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]);
      f[1] = pack8(w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int x = 0; x < 2 * DB; ++x) asm volatile("" : "+v"(lo[x / DB][x % DB]), "+v"(hi[x / DB][x % DB]));
    copy_stage(i + 2, slot);  // (every read of the slot has returned; past the end the last stage again, for nobody)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < DB; ++db) dq[db] = mfma32(join(lo[ks][db], hi[ks][db]), f[ks], dq[db]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  __bf16* const out = p.dq + q_off + (int64_t)L.l32 * q_stride + 4 * L.hh;
  const bool valid = L.l32 < q_rows;
  const float scale = p.scale;
  add_shares<D, W>(smem, wave, L.lane, min(nt, W), dq, [&](int quarter, f32x4 s) __attribute__((always_inline)) {
    if (valid) *reinterpret_cast<bf16x4*>(out + quarter * 8) = pack4(s[0] * scale, s[1] * scale, s[2] * scale, s[3] * scale);
  });
}

template <int D, int W>
__device__ __forceinline__ void share_dkv_block(const ShareParams& p, const chunk_attn_seg seg, int tile, int kvh, char* smem) {
  constexpr int DK = D / 16, DB = D / 32;
  typedef ShareLane<D> Lane;
  constexpr int TILE = Lane::TILE, PT = Lane::PT, RPC = Lane::RPC;
  const Lane L;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j0 = 32 * tile, kv_rows = min(32, seg.kv_len - j0), ctx = seg.kv_len - seg.q_len;
  const int qt_first = max(0, j0 - ctx) / 32, n_qt = (seg.q_len + 31) / 32, G = p.group;
  const int n_all = (n_qt - qt_first) * G, n_mine = n_all > wave ? (n_all - wave + W - 1) / W : 0;
  const int q_stride = p.num_q_heads * D, kv_stride = p.num_kv_heads * D, kv_c = L.c_row * kv_stride, q_c = L.c_row * q_stride;
  const int64_t kv_off = (int64_t)(seg.kv_start + j0) * kv_stride + kvh * D;
  lds_bf16* const region = (lds_bf16*)(smem + wave * 4 * TILE);
  lds_bf16* const own = (lds_bf16*)(smem + W * 4 * TILE);                       // K, V
  lds_f32* const rows = (lds_f32*)(smem + (W * 4 + 2) * TILE) + wave * 64;      // of the wave's stage: LSE log2(e) [32], -D [32]

  // a stage of the wave: query tile and head of the group (heads of a tile one after the other); `next` finds the wave's next one
  struct Stage {
    int qt, h;
  };
  const int per_qt = W / G, per_h = W % G;
  auto next = [&](Stage x) __attribute__((always_inline)) {
    x.h += per_h;
    x.qt += per_qt;
    if (x.h >= G) {
      x.h -= G;
      ++x.qt;
    }
    return x;
  };
  bf16x8 of[PT];   // O of the next stage, as the copies lay out dO
  float lse = 0.f; // and its LSE, rows 0 .. 31 in the first 32 lanes
  auto load_rows = [&](Stage x) __attribute__((always_inline)) {
    const int i0 = 32 * x.qt, head = kvh * G + x.h, last = seg.q_len - 1 - i0;
    const __bf16* const src = p.o + (int64_t)(seg.q_start + i0) * q_stride + head * D;
    lse = p.lse[(int64_t)head * p.total_q + seg.q_start + i0 + min(L.l32, last)];
    if (last >= 31)
      static_for<0, PT>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int n = decltype(x_c)::value;
        of[n] = *reinterpret_cast<const bf16x8*>(L.template chunk<n>(src, q_stride, q_c, 31));
      });
    else
      static_for<0, PT>([&](auto x_c) __attribute__((always_inline)) {
        constexpr int n = decltype(x_c)::value;
        of[n] = *reinterpret_cast<const bf16x8*>(L.template chunk<n>(src, q_stride, q_c, min(last, 30)));
      });
  };
  // Stands where the loads of load_rows have long ended and no copy has been issued since the last one that must have landed: the compiler waits for
  // a load by counting what was issued after it, and takes copies in branches for none, so that at its use it would wait for the next stage's copies.
  auto rows_loaded = [&]() __attribute__((always_inline)) {
    asm volatile("" : "+v"(lse));
#pragma unroll
    for (int x = 0; x < PT; ++x) asm volatile("" : "+v"(of[x]));
  };
  auto copy_stage = [&](Stage x, int slot) __attribute__((always_inline)) {
    const int i0 = 32 * x.qt, head = kvh * G + x.h, last = seg.q_len - 1 - i0;
    const int64_t off = (int64_t)(seg.q_start + i0) * q_stride + head * D;
    L.copy_tile(p.q + off, q_stride, q_c, last, region + slot * TILE);
    L.copy_tile(p.d_o + off, q_stride, q_c, last, region + slot * TILE + TILE / 2);
  };
  Stage cur{qt_first + wave / G, wave % G}, ahead = n_mine > 1 ? next(cur) : cur;  // of the step, and the one after it
  static_for<0, PT>([&](auto i_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value;
    if (i % W == wave) {
      dma16(L.template chunk<i>(p.k + kv_off, kv_stride, kv_c, kv_rows - 1), own + i * 512);
      dma16(L.template chunk<i>(p.v + kv_off, kv_stride, kv_c, kv_rows - 1), own + TILE / 2 + i * 512);
    }
  });
  if (n_mine > 0) {
    load_rows(cur);
    copy_stage(cur, 0);
    rows_loaded();
    copy_stage(ahead, 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * PT) : "memory");  // (all but the stages' copies)
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  wg_barrier();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 acc[2 * DB];  // dV^T, dK^T
#pragma unroll
  for (int db = 0; db < 2 * DB; ++db) acc[db] = zero16;
  bf16x8 kf[DK], vf[DK];
  {
    const unsigned base = lds_addr(own) + L.row_at;
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      kf[ks] = lds_asm_read16<0>(base ^ (ks * 32));
      vf[ks] = lds_asm_read16<TILE>(base ^ (ks * 32));
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));
  }

  const float c = p.scale_log2;
  const int jrel = j0 + L.l32 - ctx;  // query i of the segment sees the lane's key iff i >= jrel
  const unsigned r_base = lds_addr(region) + L.row_at, t_base = lds_addr(region) + L.tr_at, d_base = lds_addr(region) + TILE + L.lane * 16;
  const unsigned rv = lds_addr(rows) + 16 * L.hh;
  for (int i = 0; i < n_mine; ++i) {
    const int slot = i & 1;
    const int i0 = 32 * cur.qt;
    const int valid = seg.q_len - i0;  // rows of the tile (32 or more: all)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PT) : "memory");  // the copies of the stage after this one may be outstanding
    const unsigned ra = r_base + slot * (2 * TILE), ta = t_base + slot * (2 * TILE);
    bf16x8 qf[DK], gf[DK], g[PT];
    f32x4 r_lse[4], r_nd[4];
    f32x16 s, dp;
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      qf[ks] = lds_asm_read16<0>(ra ^ (ks * 32));
    });
    static_for<0, PT>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int x = decltype(x_c)::value;
      g[x] = lds_asm_read16<x * 1024>(d_base + slot * (2 * TILE));
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(qf[ks]));
#pragma unroll
    for (int x = 0; x < PT; ++x) asm volatile("" : "+v"(g[x]));
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) s = mfma32(qf[ks], kf[ks], ks == 0 ? zero16 : s);
    // ---- -D and LSE of the stage's rows, through LDS into the rows of the accumulators ----
    float nd[PT];
    static_for<0, PT>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int x = decltype(x_c)::value;
      const float part = dot8(of[x], g[x]);
      nd[x] = sum_row<Lane::C>(L.template in_row<x>() ? part : 0.f);
    });
    static_for<0, PT>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int x = decltype(x_c)::value;
      if (L.lane % Lane::C == 0) lds_asm_write4(lds_addr(rows + 32 + RPC * x + L.c_row), (int)__float_as_uint(RPC * x + L.c_row < valid ? -nd[x] : 0.f));
    });
    if (L.lane < 32) lds_asm_write4(lds_addr(rows + L.lane), (int)__float_as_uint(L.lane < valid ? lse * kLog2e : INFINITY));
    load_rows(ahead);
    static_for<0, 4>([&](auto g_c) __attribute__((always_inline)) {
      constexpr int x = decltype(g_c)::value;
      r_lse[x] = lds_asm_read16f<x * 32>(rv);
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, DK>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      gf[ks] = lds_asm_read16<TILE>(ra ^ (ks * 32));
    });
    static_for<0, 4>([&](auto g_c) __attribute__((always_inline)) {
      constexpr int g = decltype(g_c)::value;
      r_nd[g] = lds_asm_read16f<128 + g * 32>(rv);
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) asm volatile("" : "+v"(gf[ks]));
#pragma unroll
    for (int g = 0; g < 4; ++g) asm volatile("" : "+v"(r_lse[g]), "+v"(r_nd[g]));
    s16x4 glo[2][DB], ghi[2][DB];  // operands of dV^T += dO^T P
    static_for<0, 2 * DB>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(x_c)::value / DB, db = decltype(x_c)::value % DB;
      glo[ks][db] = lds_asm_read_tr<TILE + ks * 16 * Lane::ROW>(ta ^ (db * 64));
      ghi[ks][db] = lds_asm_read_tr<TILE + (ks * 16 + 8) * Lane::ROW>(ta ^ (db * 64 + share_swz<D>(8) * 16));
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) dp = mfma32(gf[ks], vf[ks], ks == 0 ? zero16 : dp);
    float pe[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) pe[e] = __builtin_amdgcn_exp2f(s[e] * c - r_lse[e >> 2][e & 3]);
    if (i0 < j0 + 31 - ctx) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (i0 + 8 * (e >> 2) + 4 * L.hh + (e & 3) < jrel) pe[e] = 0.f;
    }
    const bf16x8 p0 = pack8(pe[0], pe[1], pe[2], pe[3], pe[4], pe[5], pe[6], pe[7]);
    const bf16x8 p1 = pack8(pe[8], pe[9], pe[10], pe[11], pe[12], pe[13], pe[14], pe[15]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int x = 0; x < 2 * DB; ++x) asm volatile("" : "+v"(glo[x / DB][x % DB]), "+v"(ghi[x / DB][x % DB]));
    s16x4 qlo[2][DB], qhi[2][DB];  // operands of dK^T += Q^T dS
    static_for<0, 2 * DB>([&](auto x_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(x_c)::value / DB, db = decltype(x_c)::value % DB;
      qlo[ks][db] = lds_asm_read_tr<ks * 16 * Lane::ROW>(ta ^ (db * 64));
      qhi[ks][db] = lds_asm_read_tr<(ks * 16 + 8) * Lane::ROW>(ta ^ (db * 64 + share_swz<D>(8) * 16));
    });
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = mfma32(join(glo[0][db], ghi[0][db]), p0, acc[db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = mfma32(join(glo[1][db], ghi[1][db]), p1, acc[db]);
    float w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] = pe[e] * (dp[e] + r_nd[e >> 2][e & 3]);
    const bf16x8 f0 = pack8(w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]);
    const bf16x8 f1 = pack8(w[8], w[9], w[10], w[11], w[12], w[13], w[14], w[15]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int x = 0; x < 2 * DB; ++x) asm volatile("" : "+v"(qlo[x / DB][x % DB]), "+v"(qhi[x / DB][x % DB]));
    rows_loaded();
    cur = ahead;
    if (i + 2 < n_mine) ahead = next(ahead);
    copy_stage(ahead, slot);  // (every read of the slot has returned; past the end the last stage again, for nobody)
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[DB + db] = mfma32(join(qlo[0][db], qhi[0][db]), f0, acc[DB + db]);
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[DB + db] = mfma32(join(qlo[1][db], qhi[1][db]), f1, acc[DB + db]);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  const int64_t row = kv_off + (int64_t)L.l32 * kv_stride + 4 * L.hh;
  const bool valid = L.l32 < kv_rows, add = p.accumulate != 0, wide = p.out_f32 != 0;
  add_shares<D, W>(smem, wave, L.lane, min(n_all, W), acc, [&](int quarter, f32x4 s) __attribute__((always_inline)) {
    const bool is_dk = quarter >= DB * 4;
    const float f = is_dk ? p.scale : 1.0f;
    __bf16* const base = is_dk ? p.dk : p.dv;
    const int64_t at = row + (is_dk ? quarter - DB * 4 : quarter) * 8;
    f32x4 x = {s[0] * f, s[1] * f, s[2] * f, s[3] * f};
    if (!valid) return;
    if (wide) {
      f32x4* const op = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(base) + at);
      if (add) x += *op;
      *op = x;
    } else {
      bf16x4* const op = reinterpret_cast<bf16x4*>(base + at);
      if (add) {
        const bf16x4 old = *op;
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] += (float)old[r];
      }
      *op = pack4(x[0], x[1], x[2], x[3]);
    }
  });
}

template <int D, int W>
__global__ __launch_bounds__(W * 64, D == 64 ? 2 : 1) void bwd_share_kernel(ShareArgs) {
  typedef const __attribute__((address_space(4))) ShareArgs* args_ptr;
  const args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  ShareParams p;
  __builtin_memcpy(&p, (const void*)&args->p, sizeof(p));
  int blk = blockIdx.x;
  const int n_first = p.dq_first ? p.dq_blocks : p.dkv_blocks;
  const bool dq = (blk < n_first) == (p.dq_first != 0);
  if (blk >= n_first) blk -= n_first;
  const int inner_n = dq ? p.num_q_heads : p.num_kv_heads;
  const int n_dq_items = p.dq_blocks / p.num_q_heads;
  const unsigned word = ((const __attribute__((address_space(4))) unsigned*)args->items)[blk / inner_n + (dq ? 0 : n_dq_items)];
  chunk_attn_seg seg;
  __builtin_memcpy(&seg, (const void*)(args->segs + (word & 0xffff)), sizeof(seg));
  if (dq) share_dq_block<D, W>(p, seg, word >> 16, blk % inner_n, smem);
  else share_dkv_block<D, W>(p, seg, word >> 16, blk % inner_n, smem);
}

template <int D, int W>
hipError_t launch(const ShareArgs& a, hipStream_t stream) {
  constexpr size_t smem = share_bwd_smem<D, W>();
  static_assert(smem <= 160 * 1024);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_share_kernel<D, W>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((bwd_share_kernel<D, W>), dim3((unsigned)(a.p.dq_blocks + a.p.dkv_blocks)), dim3(W * 64), smem, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_share(const chunk_attn_desc* d, const BwdArgs& a, int waves, hipStream_t stream) {
  ShareArgs s;
  s.p.q = a.q; s.p.k = a.k; s.p.v = a.v; s.p.o = a.o; s.p.d_o = a.d_o; s.p.lse = a.lse;
  s.p.dq = a.dq; s.p.dk = a.dk; s.p.dv = a.dv;
  s.p.total_q = d->total_q; s.p.num_q_heads = d->num_q_heads; s.p.num_kv_heads = d->num_kv_heads;
  s.p.group = d->num_q_heads / d->num_kv_heads;
  s.p.scale = d->softmax_scale; s.p.scale_log2 = d->softmax_scale * kLog2e;
  s.p.accumulate = a.accumulate ? 1 : 0; s.p.out_f32 = a.dkv_f32 ? 1 : 0;
  // blocks of either kind, longest walk first
  const std::vector<ShareBlock> dq = share_blocks(d, false), dkv = share_blocks(d, true);
  if (dq.size() + dkv.size() > (size_t)kMaxShareItems || d->num_segments > kMaxShareSegs) return hipErrorInvalidValue;
  for (int t = 0; t < d->num_segments; ++t) s.segs[t] = d->segments[t];
  size_t n = 0;
  for (const ShareBlock& b : dq) s.items[n++] = ShareItem{(uint16_t)b.seg, (uint16_t)b.tile};
  for (const ShareBlock& b : dkv) s.items[n++] = ShareItem{(uint16_t)b.seg, (uint16_t)b.tile};
  s.p.dq_blocks = (int)dq.size() * d->num_q_heads;
  s.p.dkv_blocks = (int)dkv.size() * d->num_kv_heads;
  s.p.dq_first = dq[0].steps * 3 >= dkv[0].steps * 4 ? 1 : 0;
  hipError_t e = zero_uncovered(d, a, stream);
  if (e != hipSuccess) return e;
  ProfileEvents pe = profile_events();
  profile_events() = ProfileEvents{};
  if (pe.start && (e = hipEventRecord(pe.start, stream)) != hipSuccess) return e;
  e = d->head_dim == 128 ? launch<128, 4>(s, stream) : d->head_dim == 96 ? launch<96, 4>(s, stream) : waves == 8 ? launch<64, 8>(s, stream) : launch<64, 4>(s, stream);
  if (e == hipSuccess && pe.stop) e = hipEventRecord(pe.stop, stream);
  return e;
}

}  // namespace chunk_attn

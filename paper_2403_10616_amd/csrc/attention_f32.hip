// Causal attention in fp32 on the matrix cores, forward and backward, head sizes 32, 64 and 128.
//
// v_mfma_f32_16x16x4_f32 throughout: operand lane l supplies row (column) l % 16 and contraction index l / 16, and lane
// l of a result holds column l % 16, rows 4 (l / 16) + e, e = 0..3.  As in the bf16 kernels (attention_mfma.h) whatever
// has to be contracted next is made the ROW index of the score tile, so that probabilities go from accumulator
// registers straight into the next product: element e of a 16-row score tile IS the B operand of a product over the four
// rows 4 (l / 16) + e.
//   forward, dQ:   S^T = K.Q^T  (rows = keys, columns = queries)  ->  O^T += V^T.P^T,   dQ^T += K^T.dS^T
//   dK, dV:        S   = Q.K^T  (rows = queries, columns = keys)  ->  dV^T += dO^T.P,   dK^T += Q^T.dS
//
// One workgroup = 8 waves of 16 queries (keys), 128 in all, or 4 waves where the launch is small (few_waves); tiles of 32 keys (queries) go through registers into LDS, two
// stages, one barrier per tile, the next tile's loads in flight during this one's products.  Rows are kept DH + 4 floats
// apart, which serves both kinds of read: 16-byte reads along a row (contraction over the head: lane l takes columns
// 16 c + 4 (l / 16) .. + 3 of row l % 16, good for four products), and 4-byte reads across four rows (contraction over the
// tile's rows: columns l % 16 of row 4 (l / 16) + e), which then fall on 64 different banks.
// The 16-row shape keeps a head of 128 in 32 registers per operand and lane, and gives small batches twice the waves of
// a 32-row one.
// Bound: the fp32 matrix cores (a product of 2048 flop every 32 cycles and SIMD); a tile asks 64 (forward) to 160 (dK/dV)
// of them per wave against 16-40 KB of LDS reads, a quarter of what LDS delivers in that time.
// Measured on 8 sequences x 8 heads x 500 positions, head size 64: forward 41 us, dQ 54, dK / dV 66 with four waves; 49, 64, 81
// with eight (256 workgroups on 256 compute units, the causal triangle's longest block setting the length of each launch);
// one thread per row on the vector ALU: 375, 911, 1517.
// No atomics: every output element has exactly one writer and a fixed summation order.
#include <algorithm>
#include <type_traits>

#include "attention_plain.h"
#include "causal_order.h"
#include "kernels.h"
#include "mma_tile.h"

namespace dipaco {

namespace {

// NW waves of 16 queries (keys) make a workgroup: 8, or 4 where the launch would otherwise be about one workgroup per
// compute unit and as long as the causal triangle's longest block.  Forward / backward in us with 4 | 8 waves, 8 heads of 500
// positions: 256 blocks of 128 rows, head size 32: 26 / 69 | 31 / 82, 64: 41 / 114 | 49 / 139, 128: 68 / 206 | 85 / 247; 512
// blocks 36 / 95 | 39 / 104, 57 / 171 | 63 / 180, 104 / 320 | 107 / 315; 1024 blocks 60 / 163 | 60 / 166, 100 / 294 | 101 / 294,
// 195 / 591 | 176 / 652.
constexpr int F_MANY = 8, F_FEW = 4;
inline bool few_waves(int B, int S, int H) { return (long)B * H * ((S + 127) / 128) <= 512; }
constexpr int F_TILE = 32;             // keys (queries) per tile

template <int DH> constexpr int row_stride() { return DH + 4; }
template <int DH> constexpr int tile_floats() { return F_TILE * row_stride<DH>(); }
template <int DH> constexpr float head_scale() { return DH == 32 ? 0.17677669529663689f : DH == 64 ? 0.125f : 0.088388347648318447f; }

__device__ __forceinline__ f32x4 mfma4(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float sum_groups(float v) {   // over the four lanes that share l % 16
  v += __shfl_xor(v, 16, WAVE);
  v += __shfl_xor(v, 32, WAVE);
  return v;
}
__device__ __forceinline__ float max_groups(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, WAVE));
  v = fmaxf(v, __shfl_xor(v, 32, WAVE));
  return v;
}

// Two operands' tiles of F_TILE rows: thread t moves float4 number t + 64 NW i of tile i / (NLD / 2).
template <int DH, int NW> struct TilePair {
  static constexpr int VEC_ROW = DH / 4;                                   // 16-byte vectors per row
  static constexpr int NLD = 2 * F_TILE * VEC_ROW / (64 * NW);             // per thread, both tiles: 1 .. 8
  static constexpr int PER_TILE = F_TILE * VEC_ROW;                        // vectors per tile: 256, 512, 1024
  f32x4 v[NLD];
  // rows at or beyond rows_total re-read the last valid row (callers give them zero weight)
  __device__ __forceinline__ void load(const float* t0, const float* t1, long ld0, long ld1, int row0, int rows_total) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int n = threadIdx.x + 64 * NW * i;
      const bool first = n < PER_TILE;
      const int m = first ? n : n - PER_TILE;
      const int row = min(row0 + m / VEC_ROW, rows_total - 1);
      v[i] = *reinterpret_cast<const f32x4*>((first ? t0 + row * ld0 : t1 + row * ld1) + 4 * (m % VEC_ROW));
    }
  }
  __device__ __forceinline__ void store(float* stage) const {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int n = threadIdx.x + 64 * NW * i;
      const bool first = n < PER_TILE;
      const int m = first ? n : n - PER_TILE;
      *reinterpret_cast<f32x4*>(stage + (first ? 0 : tile_floats<DH>()) + (m / VEC_ROW) * row_stride<DH>() + 4 * (m % VEC_ROW)) = v[i];
    }
  }
};

// a lane's share of one of its wave's 16 rows: columns 16 c + 4 (l / 16) .. + 3
template <int DH> struct RowFrag { float4 c[DH / 16]; };
template <int DH> __device__ __forceinline__ RowFrag<DH> load_row(const float* row, int g, bool valid) {
  RowFrag<DH> f;
#pragma unroll
  for (int c = 0; c < DH / 16; ++c)
    f.c[c] = valid ? *reinterpret_cast<const float4*>(row + 16 * c + 4 * g) : make_float4(0.f, 0.f, 0.f, 0.f);
  return f;
}
// acc (16 x 16) += rows 16 t .. + 15 of `tile`, contracted over the head with this wave's rows b
template <int DH>
__device__ __forceinline__ void rows_product(f32x4& acc, const float* tile, int t, const RowFrag<DH>& b, int m, int g) {
  const float* r = tile + (16 * t + m) * row_stride<DH>() + 4 * g;
#pragma unroll
  for (int c = 0; c < DH / 16; ++c) {
    const float4 a = *reinterpret_cast<const float4*>(r + 16 * c);
    acc = mfma4(a.x, b.c[c].x, acc);
    acc = mfma4(a.y, b.c[c].y, acc);
    acc = mfma4(a.z, b.c[c].z, acc);
    acc = mfma4(a.w, b.c[c].w, acc);
  }
}
// acc^T[d] (16 head columns x this wave's 16 rows) += (rows 16 t .. + 15 of `tile`)^T . p
template <int DH>
__device__ __forceinline__ void cols_product(f32x4 (&acc)[DH / 16], const float* tile, int t, const f32x4& p, int m, int g) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float* r = tile + (16 * t + 4 * g + e) * row_stride<DH>() + m;
#pragma unroll
    for (int d = 0; d < DH / 16; ++d) acc[d] = mfma4(r[16 * d], p[e], acc[d]);
  }
}
template <int DH> __device__ __forceinline__ void zero_acc(f32x4 (&acc)[DH / 16]) {
#pragma unroll
  for (int d = 0; d < DH / 16; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
}
template <int DH> __device__ __forceinline__ void store_row(float* row, const f32x4 (&acc)[DH / 16], int g, float scale) {
#pragma unroll
  for (int d = 0; d < DH / 16; ++d)
    *reinterpret_cast<float4*>(row + 16 * d + 4 * g) =
        make_float4(acc[d][0] * scale, acc[d][1] * scale, acc[d][2] * scale, acc[d][3] * scale);
}
// Column sums of the workgroup's 16 NW output rows: over the 16 lanes of a group on the DPP lanes, then the waves in order.
// red: LDS [NW][DH].  Every wave calls it; rows with valid = false count as zero.
template <int DH, int NW>
__device__ __forceinline__ void block_column_sums(const f32x4 (&acc)[DH / 16], float scale, bool valid, float* red,
                                                  float* __restrict__ out, int wave, int m, int g) {
  __syncthreads();   // red lies in LDS that was in use before
#pragma unroll
  for (int d = 0; d < DH / 16; ++d)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = valid ? acc[d][e] * scale : 0.f;
      v += dpp_fetch<0xb1, 0xf>(v, 0.f);
      v += dpp_fetch<0x4e, 0xf>(v, 0.f);
      v += dpp_fetch<0x141, 0xf>(v, 0.f);
      v += dpp_fetch<0x140, 0xf>(v, 0.f);
      if (m == 0) red[wave * DH + 16 * d + 4 * g + e] = v;
    }
  __syncthreads();
  for (int c = threadIdx.x; c < DH; c += 64 * NW) {
    float s = red[c];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w * DH + c];
    out[c] = s;
  }
}

template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW, 2) attn_fwd_f32(const float* __restrict__ qkv, float* __restrict__ o,
                                                             float* __restrict__ lse, int S, int H, bool paired) {
  extern __shared__ __attribute__((aligned(16))) float f_smem[];   // [stage][K | V]
  constexpr int STAGE = 2 * tile_floats<DH>();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const CausalPlace at = causal_place(paired);
  const int bh = at.bh, b = bh / H, hd = bh % H, A = H * DH;
  const long ld = 3L * A;
  const float* base = qkv + (long)b * S * ld + hd * DH;
  const int q0 = ((int)gridDim.y - 1 - at.order) * (16 * NW);
  const int qw0 = q0 + 16 * wave, q = qw0 + m;
  const RowFrag<DH> qf = load_row<DH>(base + (long)q * ld, g, q < S);
  const int ntiles = (min(S, q0 + (16 * NW)) + F_TILE - 1) / F_TILE;
  f32x4 ot[DH / 16];
  zero_acc<DH>(ot);
  float mx = -INFINITY, l = 0.f;
  TilePair<DH, NW> next;
  next.load(base + A, base + 2 * A, ld, ld, 0, S);
  next.store(f_smem);
  for (int kt = 0; kt < ntiles; ++kt) {
    const float* k_ = f_smem + (kt & 1) * STAGE;
    const float* v_ = k_ + tile_floats<DH>();
    const int kv0 = kt * F_TILE;
    const bool more = kt + 1 < ntiles;
    if (more) next.load(base + A, base + 2 * A, ld, ld, kv0 + F_TILE, S);
    __syncthreads();   // tile kt is in LDS, and everybody is done with the stage of tile kt - 1
    if (kv0 <= qw0 + 15) {   // wave-uniform: some query of this wave sees this tile
      f32x4 st[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        st[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        rows_product<DH>(st[t], k_, t, qf, m, g);
      }
      float tile_max = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          st[t][e] = kv0 + 16 * t + 4 * g + e > q ? -INFINITY : st[t][e] * head_scale<DH>();
          tile_max = fmaxf(tile_max, st[t][e]);
        }
      const float mn = fmaxf(mx, max_groups(tile_max));   // finite: key 0 is visible to every query
      const float corr = expf(mx - mn);
      mx = mn;
      float part = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          st[t][e] = expf(st[t][e] - mn);
          part += st[t][e];
        }
      l = l * corr + part;   // this lane's quarter of the row's keys
#pragma unroll
      for (int d = 0; d < DH / 16; ++d)
#pragma unroll
        for (int e = 0; e < 4; ++e) ot[d][e] *= corr;
#pragma unroll
      for (int t = 0; t < 2; ++t) cols_product<DH>(ot, v_, t, st[t], m, g);
    }
    if (more) next.store(f_smem + ((kt + 1) & 1) * STAGE);
  }
  l = sum_groups(l);
  if (__any(q < S && plain::not_finite(ot)) && q < S)
    plain::attend<DH>(ot, base, ld, A, q, g, [&](float s) { return expf(s * head_scale<DH>() - mx); });
  if (q < S) {
    store_row<DH>(o + ((long)b * S + q) * A + hd * DH, ot, g, 1.0f / l);
    if (g == 0) lse[(long)bh * S + q] = mx + logf(l);
  }
}

template <int DH> __device__ __forceinline__ float row_dot(const RowFrag<DH>& a, const RowFrag<DH>& b) {
  float d = 0.f;
#pragma unroll
  for (int c = 0; c < DH / 16; ++c) d += (a.c[c].x * b.c[c].x + a.c[c].y * b.c[c].y) + (a.c[c].z * b.c[c].z + a.c[c].w * b.c[c].w);
  return sum_groups(d);
}

// dQ_i = scale * sum_{j<=i} p_ij (dO_i.v_j - D_i) k_j, with D_i = dO_i.o_i (stored for a dK/dV kernel behind it unless dsum is null)
template <int DH, int NW>
__device__ __forceinline__ void dq_block(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                         const float* __restrict__ lse, float* __restrict__ dqkv, float* __restrict__ dsum,
                                         float* __restrict__ colsum, int S, int H, int bh, int qb, int n_blocks) {
  extern __shared__ __attribute__((aligned(16))) float f_smem[];   // [stage][K | V]
  constexpr int STAGE = 2 * tile_floats<DH>();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const int b = bh / H, hd = bh % H, A = H * DH;
  const long ld = 3L * A;
  const float* base = qkv + (long)b * S * ld + hd * DH;
  const int q0 = qb * (16 * NW);
  const int qw0 = q0 + 16 * wave, q = qw0 + m;
  const RowFrag<DH> qf = load_row<DH>(base + (long)q * ld, g, q < S);
  const long orow = ((long)b * S + q) * A + hd * DH;
  const RowFrag<DH> gf = load_row<DH>(d_o + orow, g, q < S);
  const float D = row_dot<DH>(gf, load_row<DH>(o + orow, g, q < S));
  const float L = q < S ? lse[(long)bh * S + q] : INFINITY;   // +inf beyond the sequence: probability 0
  if (dsum && g == 0 && q < S) dsum[(long)bh * S + q] = D;
  const int ntiles = (min(S, q0 + (16 * NW)) + F_TILE - 1) / F_TILE;
  f32x4 dqt[DH / 16];
  zero_acc<DH>(dqt);
  TilePair<DH, NW> next;
  next.load(base + A, base + 2 * A, ld, ld, 0, S);
  next.store(f_smem);
  for (int kt = 0; kt < ntiles; ++kt) {
    const float* k_ = f_smem + (kt & 1) * STAGE;
    const float* v_ = k_ + tile_floats<DH>();
    const int kv0 = kt * F_TILE;
    const bool more = kt + 1 < ntiles;
    if (more) next.load(base + A, base + 2 * A, ld, ld, kv0 + F_TILE, S);
    __syncthreads();
    if (kv0 <= qw0 + 15) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 st = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
        rows_product<DH>(st, k_, t, qf, m, g);
        rows_product<DH>(dp, v_, t, gf, m, g);
#pragma unroll
        for (int e = 0; e < 4; ++e)   // without the 1 / sqrt(d_head) factor, which is applied when dQ is stored
          st[e] = kv0 + 16 * t + 4 * g + e > q ? 0.f : expf(st[e] * head_scale<DH>() - L) * (dp[e] - D);
        cols_product<DH>(dqt, k_, t, st, m, g);
      }
    }
    if (more) next.store(f_smem + ((kt + 1) & 1) * STAGE);
  }
  if (__any(q < S && plain::not_finite(dqt)) && q < S)
    plain::query_grad<DH>(dqt, base, d_o + orow, D, ld, A, q, g, [&](float s) { return expf(s * head_scale<DH>() - L); });
  if (q < S) store_row<DH>(dqkv + ((long)b * S + q) * ld + hd * DH, dqt, g, head_scale<DH>());
  // one row of partial column sums per (document, query block), this head's DH columns of dQ
  if (colsum)
    block_column_sums<DH, NW>(dqt, head_scale<DH>(), q < S, f_smem, colsum + ((long)b * n_blocks + qb) * ld + hd * DH, wave, m, g);
}

// dV_j = sum_{i>=j} p_ij dO_i;  dK_j = scale * sum_{i>=j} p_ij (dO_i.v_j - D_i) q_i
// OWN_D: one block holds the sequence, and D is taken here, from o, by the arithmetic of dq_block; else from dsum
template <int DH, int NW, bool OWN_D>
__device__ __forceinline__ void dkv_block(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                          const float* __restrict__ lse, const float* __restrict__ dsum, float* __restrict__ dqkv,
                                          float* __restrict__ colsum, int S, int H, int bh, int kb, int n_blocks) {
  extern __shared__ __attribute__((aligned(16))) float f_smem[];   // [stage][Q | dO | lse | D]
  constexpr int STAGE = 2 * tile_floats<DH>() + 2 * F_TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const int b = bh / H, hd = bh % H, A = H * DH;
  const long ld = 3L * A;
  const float* base = qkv + (long)b * S * ld + hd * DH;
  const float* gbase = d_o + (long)b * S * A + hd * DH;
  const int k0 = kb * (16 * NW);            // early key blocks are the long ones
  const int kw0 = k0 + 16 * wave, key = kw0 + m;
  const RowFrag<DH> kf = load_row<DH>(base + (long)key * ld + A, g, key < S);
  const RowFrag<DH> vf = load_row<DH>(base + (long)key * ld + 2 * A, g, key < S);
  f32x4 dkt[DH / 16], dvt[DH / 16];
  zero_acc<DH>(dkt);
  zero_acc<DH>(dvt);
  const int first = k0 / F_TILE, ntiles = (S + F_TILE - 1) / F_TILE;
  __shared__ float own_d[OWN_D ? 16 * NW : 1];
  if constexpr (OWN_D) {
    const long orow = ((long)b * S + key) * A + hd * DH;
    const float D = row_dot<DH>(load_row<DH>(d_o + orow, g, key < S), load_row<DH>(o + orow, g, key < S));
    if (g == 0) own_d[key] = D;
    __syncthreads();
  }
  TilePair<DH, NW> next;
  float next_stat = 0.f;
  // statistics of a tile's queries: threads 0..31 move lse (+inf beyond the sequence: probability 0), 32..63 D
  auto load = [&](int qt) {
    next.load(base, gbase, ld, A, qt * F_TILE, S);
    if (threadIdx.x < 2 * F_TILE) {
      const int q = qt * F_TILE + (threadIdx.x & (F_TILE - 1));
      const bool is_lse = threadIdx.x < F_TILE;
      if (OWN_D && !is_lse) next_stat = q < S ? own_d[q] : 0.f;
      else next_stat = q < S ? (is_lse ? lse : dsum)[(long)bh * S + q] : (is_lse ? INFINITY : 0.f);
    }
  };
  auto store = [&](int qt) {
    float* stage = f_smem + ((qt - first) & 1) * STAGE;
    next.store(stage);
    if (threadIdx.x < 2 * F_TILE) stage[2 * tile_floats<DH>() + threadIdx.x] = next_stat;
  };
  load(first);
  store(first);
  for (int qt = first; qt < ntiles; ++qt) {
    const float* q_ = f_smem + ((qt - first) & 1) * STAGE;
    const float* g_ = q_ + tile_floats<DH>();
    const float* Ls = q_ + 2 * tile_floats<DH>();
    const int q0 = qt * F_TILE;
    const bool more = qt + 1 < ntiles;
    if (more) load(qt + 1);
    __syncthreads();
    if (q0 + F_TILE - 1 >= kw0) {   // wave-uniform: some query of this tile sees a key of this wave
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 st = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
        rows_product<DH>(st, q_, t, kf, m, g);
        rows_product<DH>(dp, g_, t, vf, m, g);
        const float4 Lq = *reinterpret_cast<const float4*>(Ls + 16 * t + 4 * g);
        const float4 Dq = *reinterpret_cast<const float4*>(Ls + F_TILE + 16 * t + 4 * g);
        const float L[4] = {Lq.x, Lq.y, Lq.z, Lq.w}, D[4] = {Dq.x, Dq.y, Dq.z, Dq.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = q0 + 16 * t + 4 * g + e < key ? 0.f : expf(st[e] * head_scale<DH>() - L[e]);
          st[e] = p;
          dp[e] = p * (dp[e] - D[e]);
        }
        cols_product<DH>(dvt, g_, t, st, m, g);
        cols_product<DH>(dkt, q_, t, dp, m, g);
      }
    }
    if (more) store(qt + 1);
  }
  if (__any(key < S && (plain::not_finite(dkt) || plain::not_finite(dvt))) && key < S)
    plain::key_grads<DH>(dkt, dvt, base, gbase, ld, A, key, S, g,
                         [&](float s, int i) { return expf(s * head_scale<DH>() - lse[(long)bh * S + i]); },
                         [&](int i) { return OWN_D ? own_d[i] : dsum[(long)bh * S + i]; });
  if (key < S) {
    float* out = dqkv + ((long)b * S + key) * ld + hd * DH;
    store_row<DH>(out + A, dkt, g, head_scale<DH>());
    store_row<DH>(out + 2 * A, dvt, g, 1.0f);
  }
  if (colsum) {
    float* cs = colsum + ((long)b * n_blocks + kb) * ld + hd * DH;
    block_column_sums<DH, NW>(dkt, head_scale<DH>(), key < S, f_smem, cs + A, wave, m, g);
    block_column_sums<DH, NW>(dvt, 1.0f, key < S, f_smem, cs + 2 * A, wave, m, g);
  }
}

template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW, 2) attn_bwd_dq_f32(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                float* __restrict__ dqkv, float* __restrict__ dsum,
                                                                float* __restrict__ colsum, int S, int H, bool paired) {
  const CausalPlace at = causal_place(paired);
  dq_block<DH, NW>(qkv, o, d_o, lse, dqkv, dsum, colsum, S, H, at.bh, (int)gridDim.y - 1 - at.order, gridDim.y);
}
template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW, 2) attn_bwd_dkv_f32(const float* __restrict__ qkv, const float* __restrict__ d_o,
                                                                 const float* __restrict__ lse, const float* __restrict__ dsum,
                                                                 float* __restrict__ dqkv, float* __restrict__ colsum, int S,
                                                                 int H, bool paired) {
  const CausalPlace at = causal_place(paired);
  dkv_block<DH, NW, false>(qkv, nullptr, d_o, lse, dsum, dqkv, colsum, S, H, at.bh, at.order, gridDim.y);
}
// Both in one launch on four waves a block, behind one that takes D_i (by the arithmetic of dq_block: the same bits): each alone ends with its longest
// blocks.  us, two launches -> one: 64 heads x 500 x 64 102 -> 91, x 32 60.8 -> 50.1, x 128 178 -> 162, 24 x 180 x 64 37.8 -> 24.1, 4 x 1000 x 64 170 ->
// 100, 32 x 2000 x 64 549 -> 531; 256 x 250 x 128 (1024 blocks) 193 -> 198, and on eight waves 1 - 5 % behind (512 x 130 x 64 111 -> 116).  Over 90
// sizes of 96 to 1024 blocks 1 - 42 % ahead but for whole rounds of short or very long sequences: 512 blocks of 2 and of 32 at head size 128 (73 -> 75, 610 ->
// 636), 684 and 768 of 3 at 64 (52 -> 54, 53 -> 55).
constexpr long ONE_LAUNCH_WIDE = 512;   // most blocks with head size 128
template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW) attn_stats_f32(const float* __restrict__ o, const float* __restrict__ d_o, float* __restrict__ dsum, int S, int H) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const int bh = blockIdx.x, b = bh / H, hd = bh % H, q = blockIdx.y * (16 * NW) + 16 * wave + m;
  const long orow = (((long)b * S + q) * H + hd) * DH;
  const float D = row_dot<DH>(load_row<DH>(d_o + orow, g, q < S), load_row<DH>(o + orow, g, q < S));
  if (g == 0 && q < S) dsum[(long)bh * S + q] = D;
}
// grid (heads, 2 x blocks)
template <int DH, int NW>
__global__ void __launch_bounds__(64 * NW, 2) attn_bwd_both_f32(const float* __restrict__ qkv, const float* __restrict__ o, const float* __restrict__ d_o,
                                                                  const float* __restrict__ lse, const float* __restrict__ dsum, float* __restrict__ dqkv,
                                                                  float* __restrict__ colsum, int S, int H, bool paired) {
  const CausalPlace at = causal_place(paired);
  const int blocks = gridDim.y >> 1, order = at.order >> 1;   // by length, longest first
  if (at.order & 1) dq_block<DH, NW>(qkv, o, d_o, lse, dqkv, nullptr, colsum, S, H, at.bh, blocks - 1 - order, blocks);
  else dkv_block<DH, NW, false>(qkv, nullptr, d_o, lse, dsum, dqkv, colsum, S, H, at.bh, order, blocks);
}
// Sequences of one block (up to 64 positions on four waves): dQ and dK / dV in one launch, one workgroup each (blockIdx.y), as
// such launches take as long as any launch: 4 x 2 heads x 64 x 32 6.6 + 7.0 us and a gap, 8.2 in one.
template <int DH>
__global__ void __launch_bounds__(64 * F_FEW, 2) attn_bwd_short_f32(const float* __restrict__ qkv, const float* __restrict__ o,
                                                                      const float* __restrict__ d_o, const float* __restrict__ lse,
                                                                      float* __restrict__ dqkv, float* __restrict__ dsum,
                                                                      float* __restrict__ colsum, int S, int H) {
  if (blockIdx.y == 0) dkv_block<DH, F_FEW, true>(qkv, o, d_o, lse, nullptr, dqkv, colsum, S, H, blockIdx.x, 0, 1);
  else dq_block<DH, F_FEW>(qkv, o, d_o, lse, dqkv, dsum, colsum, S, H, blockIdx.x, 0, 1);
}

template <int DH> constexpr int fwd_lds() { return 2 * 2 * tile_floats<DH>() * (int)sizeof(float); }
template <int DH> constexpr int dkv_lds() { return 2 * (2 * tile_floats<DH>() + 2 * F_TILE) * (int)sizeof(float); }

template <int DH, int NW>
dipaco_status fwd_rows(const float* qkv, float* o, float* lse, int B, int S, int H, hipStream_t s) {
  static std::atomic<unsigned long long> lds{0};
  if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_fwd_f32<DH, NW>), fwd_lds<DH>(), lds)) return st;
  const size_t A = (size_t)H * DH;
  const int step = attention_launch_batch(B, H);
  for (int b = 0; b < B; b += step) {
    const size_t row = (size_t)b * S;
    const dim3 grid(std::min(step, B - b) * H, (S + 16 * NW - 1) / (16 * NW));
    static std::atomic<int> resident{0};
    bool paired;
    if (dipaco_status st = causal_paired(reinterpret_cast<const void*>(attn_fwd_f32<DH, NW>), 64 * NW, fwd_lds<DH>(), grid.x, (long)grid.x * grid.y, resident, paired)) return st;
    attn_fwd_f32<DH, NW><<<grid, 64 * NW, fwd_lds<DH>(), s>>>(qkv + row * 3 * A, o + row * A, lse + row * H, S, H, paired);
    DIPACO_LAUNCH_CHECK();
  }
  return DIPACO_OK;
}
template <int DH>
dipaco_status fwd(const float* qkv, float* o, float* lse, int B, int S, int H, hipStream_t s) {
  return few_waves(B, S, H) ? fwd_rows<DH, F_FEW>(qkv, o, lse, B, S, H, s) : fwd_rows<DH, F_MANY>(qkv, o, lse, B, S, H, s);
}
template <int DH, int NW>
dipaco_status bwd(const float* qkv, const float* o, const float* d_o, const float* lse, float* dqkv, float* dsum,
                  float* colsum, int B, int S, int H, hipStream_t s) {
  static_assert(NW * DH <= 2 * 2 * tile_floats<DH>(), "the column sums' scratch fits in the stages");
  const size_t A = (size_t)H * DH;
  const int step = attention_launch_batch(B, H), blocks = (S + 16 * NW - 1) / (16 * NW);
  for (int b = 0; b < B; b += step) {
    const size_t row = (size_t)b * S;
    const dim3 grid(std::min(step, B - b) * H, blocks);
    float* const cs = colsum ? colsum + (size_t)b * blocks * 3 * A : nullptr;
    if constexpr (NW == F_FEW) {
      if (blocks == 1) {
        static std::atomic<unsigned long long> both{0};
        constexpr int LDS = std::max(fwd_lds<DH>(), dkv_lds<DH>());
        if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_short_f32<DH>), LDS, both)) return st;
        attn_bwd_short_f32<DH><<<dim3(grid.x, 2), 64 * NW, LDS, s>>>(qkv + row * 3 * A, o + row * A, d_o + row * A, lse + row * H,
                                                                     dqkv + row * 3 * A, dsum + row * H, cs, S, H);
        DIPACO_LAUNCH_CHECK();
        continue;
      }
    }
    const long n = (long)grid.x * grid.y;
    if constexpr (NW == F_FEW) {
      if (DH < 128 || n <= ONE_LAUNCH_WIDE) {
        static std::atomic<unsigned long long> both{0};
        static std::atomic<int> resident{0};
        bool paired;
        constexpr int LDS = std::max(fwd_lds<DH>(), dkv_lds<DH>());
        const void* const kern = reinterpret_cast<const void*>(attn_bwd_both_f32<DH, NW>);
        if (dipaco_status st = ensure_dynamic_lds(kern, LDS, both)) return st;
        if (dipaco_status st = causal_paired(kern, 64 * NW, LDS, grid.x, 2 * n, resident, paired)) return st;
        attn_stats_f32<DH, NW><<<grid, 64 * NW, 0, s>>>(o + row * A, d_o + row * A, dsum + row * H, S, H);
        DIPACO_LAUNCH_CHECK();
        attn_bwd_both_f32<DH, NW><<<dim3(grid.x, 2 * grid.y), 64 * NW, LDS, s>>>(qkv + row * 3 * A, o + row * A, d_o + row * A, lse + row * H, dsum + row * H,
                                                                                dqkv + row * 3 * A, cs, S, H, paired);
        DIPACO_LAUNCH_CHECK();
        continue;
      }
    }
    if constexpr (NW != F_FEW || DH == 128) {
      static std::atomic<unsigned long long> dq{0}, dkv{0};
      static std::atomic<int> dq_resident{0}, dkv_resident{0};
      bool dq_paired, dkv_paired;
      const void* const dq_kern = reinterpret_cast<const void*>(attn_bwd_dq_f32<DH, NW>);
      const void* const dkv_kern = reinterpret_cast<const void*>(attn_bwd_dkv_f32<DH, NW>);
      if (dipaco_status st = ensure_dynamic_lds(dq_kern, fwd_lds<DH>(), dq)) return st;
      if (dipaco_status st = ensure_dynamic_lds(dkv_kern, dkv_lds<DH>(), dkv)) return st;
      if (dipaco_status st = causal_paired(dq_kern, 64 * NW, fwd_lds<DH>(), grid.x, n, dq_resident, dq_paired)) return st;
      if (dipaco_status st = causal_paired(dkv_kern, 64 * NW, dkv_lds<DH>(), grid.x, n, dkv_resident, dkv_paired)) return st;
      attn_bwd_dq_f32<DH, NW><<<grid, 64 * NW, fwd_lds<DH>(), s>>>(qkv + row * 3 * A, o + row * A, d_o + row * A, lse + row * H,
                                                                   dqkv + row * 3 * A, dsum + row * H, cs, S, H, dq_paired);
      DIPACO_LAUNCH_CHECK();
      attn_bwd_dkv_f32<DH, NW><<<grid, 64 * NW, dkv_lds<DH>(), s>>>(qkv + row * 3 * A, d_o + row * A, lse + row * H, dsum + row * H,
                                                                    dqkv + row * 3 * A, cs, S, H, dkv_paired);
      DIPACO_LAUNCH_CHECK();
    }
  }
  return DIPACO_OK;
}

}  // namespace

dipaco_status launch_attention_fwd_f32(const float* qkv, float* o, float* lse, int B, int S, int H, int dh, hipStream_t s) {
  if (dh == 32) return fwd<32>(qkv, o, lse, B, S, H, s);
  if (dh == 64) return fwd<64>(qkv, o, lse, B, S, H, s);
  if (dh == 128) return fwd<128>(qkv, o, lse, B, S, H, s);
  return fail(DIPACO_ESHAPE, "attention: d_head must be 32, 64 or 128");
}

// for any B and S up to these: four waves write a row per 64 positions, where B H ceil(S / 128) <= 512
size_t attention_bwd_colsum_rows_f32(int B, int S, int H) {
  return std::max<size_t>((size_t)B * ((S + 127) / 128), std::min<size_t>((size_t)B * ((S + 63) / 64), 2 * (512 / H)));
}

dipaco_status launch_attention_bwd_f32(const float* qkv, const float* o, const float* d_o, const float* lse, float* dqkv,
                                       float* dsum, float* colsum_out, float* colsum_partial, int B, int S, int H, int dh,
                                       hipStream_t s, SumBatch* batch, bool coarse) {
  float* partial = colsum_out ? colsum_partial : nullptr;
  const bool few = few_waves(B, S, H) && !(coarse && colsum_out);
  auto run = [&](auto NWc) -> dipaco_status {
    constexpr int NW = decltype(NWc)::value;
    if (dh == 32) return bwd<32, NW>(qkv, o, d_o, lse, dqkv, dsum, partial, B, S, H, s);
    if (dh == 64) return bwd<64, NW>(qkv, o, d_o, lse, dqkv, dsum, partial, B, S, H, s);
    if (dh == 128) return bwd<128, NW>(qkv, o, d_o, lse, dqkv, dsum, partial, B, S, H, s);
    return fail(DIPACO_ESHAPE, "attention: d_head must be 32, 64 or 128");
  };
  const dipaco_status st = few ? run(std::integral_constant<int, F_FEW>{}) : run(std::integral_constant<int, F_MANY>{});
  if (st != DIPACO_OK || !colsum_out) return st;
  const int per = 16 * (few ? F_FEW : F_MANY);
  return launch_sum_rows(colsum_partial, colsum_out, B * ((S + per - 1) / per), 3 * H * dh, s, batch);
}

}  // namespace dipaco

// k-means prefix routing: idx[n] = argmin_k ||z_n - c_k||^2, per-centroid histogram, and the gap between the
// two best scores.  The argmin is taken over s(n,k) = ||c_k||^2 - 2 z_n.c_k (||z_n||^2 is common to all k), so
// the work is one fp32 contraction z.C^T on the matrix cores with the reduction over centroids done in the epilogue:
// scores never reach memory.
//
// route_kernel: every number taken apart into three bf16 parts (split_tile.h).  A workgroup of four waves owns 128 points and walks
// the centroids in tiles of 128; ||c_k||^2 is accumulated by the threads that stage the centroid tile, from the very values they load.
// Two workgroups share a compute unit: one splits, stores and folds scores under the other's MFMAs, which go first (wave priority).
// Bound by the MFMAs and the power they draw (six part products: 2^20 x 768 x 256 is 2.5 TFLOP of them), as gemm_split.hip.  On the
// fp32 matrix instruction 256 x 256 tiles took 3230 us there, now 2470 (2430 without the norms and third scores that near-ties need);
// 300000 x 768 x 1000 3970 -> 2880, 1000000 x 64 x 256 488 -> 356 (344).
// Error of the margins against 64 bits 3.6e-7 (1.9e-6 before) at D = 896, 2.2e-7 (6.2e-7) at 64.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "mma_tile.h"
#include "split_tile.h"

namespace dipaco {

namespace {

constexpr int RB = 128;    // points of a workgroup; centroids of a tile
constexpr int RBK = 32;    // K tile
constexpr int R_PLANE = RB * SPLIT_ROW;
constexpr int R_LDS = 6 * R_PLANE;   // planes of the centroids, planes of the points
constexpr int R_MAX_K = 4096;

// Best and second-best (score, index) of a row, ordered lexicographically: exact ties go to the lower index.
// TOP2 = false: the second index is not tracked (only its score, for the margin).
struct Best {
  float s1; int i1; float s2; int i2;
};
constexpr int NO_INDEX = 0x7fffffff;

// (s, i) before (t, j) in the lexicographic order
__device__ __forceinline__ bool lex_less(float s, int i, float t, int j) { return s < t || (s == t && i < j); }

// Candidate (s, k) whose index k is larger than every index the entry has seen: a tie keeps the earlier entry, so
// plain < decides.  Written as selects: no branch, a NaN score never enters.
template <bool TOP2> __device__ __forceinline__ void best_push_ascending(Best& b, float s, int k) {
  const bool lt1 = s < b.s1, lt2 = s < b.s2;
  if (TOP2) b.i2 = lt1 ? b.i1 : (lt2 ? k : b.i2);
  b.s2 = lt1 ? b.s1 : (lt2 ? s : b.s2);
  b.i1 = lt1 ? k : b.i1;
  b.s1 = lt1 ? s : b.s1;
}
// The two best of the union of two entries over disjoint index sets.  A selection, not arithmetic: the result does
// not depend on the order in which entries are merged.
template <bool TOP2> __device__ __forceinline__ Best best_merge(const Best& a, const Best& b) {
  const bool lt = lex_less(b.s1, b.i1, a.s1, a.i1);
  Best o;
  o.s1 = lt ? b.s1 : a.s1;
  o.i1 = lt ? b.i1 : a.i1;
  const float xs = lt ? a.s1 : b.s1, ys = lt ? b.s2 : a.s2;   // the first that lost, the second of the one that won
  if (TOP2) {
    const int xi = lt ? a.i1 : b.i1, yi = lt ? b.i2 : a.i2;
    const bool ly = lex_less(ys, yi, xs, xi);
    o.s2 = ly ? ys : xs;
    o.i2 = ly ? yi : xi;
  } else {
    o.s2 = ys < xs ? ys : xs;
    o.i2 = NO_INDEX;
  }
  return o;
}

// The third best score beside an entry, before (s, k) is pushed; and of the union of two entries.  A NaN score may put the second best
// in its place, which makes a near-tie of a point that is none
__device__ __forceinline__ void third_push(float& s3, const Best& b, float s) { s3 = __builtin_amdgcn_fmed3f(s, b.s2, s3); }
__device__ __forceinline__ float third_merge(const Best& a, float a3, const Best& b, float b3) {
  return fminf(fminf(a3, b3), fminf(fmaxf(a.s1, b.s2), fmaxf(a.s2, b.s1)));
}

// Near-ties of route_kernel.  An assignment must not turn with the unit that multiplies, so what the part products and the fp32 matrix
// instruction may order differently is decided by the latter's arithmetic.  A chain of D multiply-adds errs by up to 2^-24 of each partial
// sum, which |z| |c| bounds: 0.42 2^-24 sqrt(D) |z| |c| in the root mean square if every one were that large (evenly growing sums: 0.58 of
// it), 2^1/2 times that for the difference of two; CHAIN_ERROR is four times as much.  Numbers below 2^-110 lack bits of their third part
// (split_tile.h): 2^-134 each, held to 2^-24 of the gap.  Two candidates closer together than that (at |z| = 8, |c| = 1, D = 768 a point in
// 7000) are taken again by decide_near_tie; where a third one is as close, or a norm is so large that part products may
// overflow (infinities among them), the workgroup takes the wave's points again against all centroids (again_in_fp32).
constexpr float CHAIN_ERROR = 2.5f / 16777216.0f;
constexpr float LARGE_NORM2 = 8.507059e37f;   // 2^126
__device__ __forceinline__ float near_tie_width(float z2, float c2, int D, float dot_mul, float s1, float s2) {
  const float root = __builtin_amdgcn_sqrtf((float)D);
  const float z1 = __builtin_amdgcn_sqrtf(z2) + root * 0x1p-60f, c1 = __builtin_amdgcn_sqrtf(c2) + root * 0x1p-60f;   // squares may vanish below
  const float rounding = z2 > 0.f ? 1.2e-7f * (fabsf(s1) + fabsf(s2)) : 0.f;   // of the scores, where their dot products differ
  return dot_mul * root * (CHAIN_ERROR * z1 * c1 + 7.7e-34f * (z1 + c1)) + rounding;
}
// |c|^2 is the sum of these over a row, eight sums of every eighth piece added as a tree; written out, since a compiler that contracts
// the plain expression may choose another of its products to round
__device__ __forceinline__ float piece_squares(float x, float y, float z, float w) {
  return __builtin_fmaf(w, w, __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x)));
}
// The two candidates' scores by a chain of multiply-adds in the order of v_mfma_f32_32x32x2_f32 over chunks of four K (0, 4, 1, 5, 2, 6, 3,
// 7 of every eight).  Lanes 0 .. 31 of a wave take their points' best candidates, lanes 32 .. 63 the second ones.
__device__ __forceinline__ void decide_near_tie(Best& b, bool near, const float* __restrict__ z_row, const float* __restrict__ c,
                                                const float* __restrict__ lin_bias, int D, float dot_mul, int lane) {
  constexpr int DEEP = 16;   // pieces of four K in flight: bound by their latency (D = 896: 11 us; 22 with eight, reloaded together)
  float s = 0.f;
  if (near) {   // a lane or two as a rule: the others' rows are not read
    const int k = lane < 32 ? b.i1 : b.i2;
    const float* const c_row = c + (long)k * D;
    float dot = 0.f, n[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float4 x[DEEP];
    uint4 raw[DEEP];
    auto load = [&](int q, int k) {
      const int at = min(k, D - 4);
      x[q] = *reinterpret_cast<const float4*>(z_row + at);
      raw[q] = *reinterpret_cast<const uint4*>(c_row + at);
    };
#pragma unroll
    for (int q = 0; q < DEEP; ++q) load(q, 4 * q);
#pragma unroll 1
    for (int k0 = 0; k0 < D; k0 += 4 * DEEP) {
#pragma unroll
      for (int q = 0; q < DEEP; q += 2) {
        float4 u[2], v[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {   // K beyond the row counts as zero (points that come here are finite)
          u[p] = x[q + p];
          v[p] = __builtin_bit_cast(float4, keep_or_zero(raw[q + p], k0 + 4 * (q + p) < D));
          load(q + p, k0 + 4 * (DEEP + q + p));
          n[(q + p) % 8] += piece_squares(v[p].x, v[p].y, v[p].z, v[p].w);
        }
        dot = __builtin_fmaf(u[0].x, v[0].x, dot); dot = __builtin_fmaf(u[1].x, v[1].x, dot);
        dot = __builtin_fmaf(u[0].y, v[0].y, dot); dot = __builtin_fmaf(u[1].y, v[1].y, dot);
        dot = __builtin_fmaf(u[0].z, v[0].z, dot); dot = __builtin_fmaf(u[1].z, v[1].z, dot);
        dot = __builtin_fmaf(u[0].w, v[0].w, dot); dot = __builtin_fmaf(u[1].w, v[1].w, dot);
      }
    }
    const float cn = ((n[0] + n[1]) + (n[2] + n[3])) + ((n[4] + n[5]) + (n[6] + n[7]));
    s = __builtin_fmaf(-dot_mul, dot, lin_bias ? -lin_bias[k] : cn);
  }
  const float other = __shfl_xor(s, 32, WAVE);   // both halves of the wave hold the same points
  if (!near) return;
  const float s1 = lane < 32 ? s : other, s2 = lane < 32 ? other : s;
  const int k1 = b.i1, k2 = b.i2;
  const bool swap = lex_less(s2, k2, s1, k1);
  b.s1 = swap ? s2 : s1; b.i1 = swap ? k2 : k1;
  b.s2 = swap ? s1 : s2; b.i2 = swap ? k1 : k2;
}

// 32 points (lane l: point l % 32, z_row) against the centroids of tiles `first`, first + `step` .. of 32 on the fp32 matrix instruction, K in
// the order above
__device__ __forceinline__ Best again_in_fp32(const float* __restrict__ z_row, const float* __restrict__ c, const float* __restrict__ lin_bias,
                                              int D, int K, int first, int step, float dot_mul, int lane) {
  const int r = lane & 31, h = lane >> 5;
  Best b;
  b.s1 = INFINITY; b.i1 = NO_INDEX; b.s2 = INFINITY; b.i2 = NO_INDEX;
#pragma unroll 1
  for (int n0 = 32 * first; n0 < K; n0 += 32 * step) {
    const float* const c_row = c + (long)min(n0 + r, K - 1) * D;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    float n[4] = {0.f, 0.f, 0.f, 0.f};
    float4 x[4], y[4];
    auto load = [&](int k0) {   // chunk 2 q + h of 32 K; K beyond the row counts as zero
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + 8 * q + 4 * h, at = min(k, D - 4);
        x[q] = __builtin_bit_cast(float4, keep_or_zero(*reinterpret_cast<const uint4*>(z_row + at), k < D));
        y[q] = __builtin_bit_cast(float4, keep_or_zero(*reinterpret_cast<const uint4*>(c_row + at), k < D));
      }
    };
    load(0);
#pragma unroll 1
    for (int k0 = 0; k0 < D; k0 += RBK) {
      float4 u[4], v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { u[q] = x[q]; v[q] = y[q]; }
      if (k0 + RBK < D) load(k0 + RBK);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v[q].x, u[q].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v[q].y, u[q].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v[q].z, u[q].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v[q].w, u[q].w, acc, 0, 0, 0);
        n[q] += piece_squares(v[q].x, v[q].y, v[q].z, v[q].w);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) n[q] += __shfl_xor(n[q], 32, WAVE);
    const float cn = n0 + r < K ? (lin_bias ? -lin_bias[n0 + r] : (n[0] + n[1]) + (n[2] + n[3])) : INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = acc_row(e, lane);
      best_push_ascending<true>(b, __builtin_fmaf(-dot_mul, acc[e], __shfl(cn, row, WAVE)), n0 + row);
    }
  }
  Best o;
  o.s1 = __shfl_xor(b.s1, 32, WAVE); o.i1 = __shfl_xor(b.i1, 32, WAVE); o.s2 = __shfl_xor(b.s2, 32, WAVE); o.i2 = __shfl_xor(b.i2, 32, WAVE);
  return best_merge<true>(b, o);
}

// z: row n at z + n * ldz.  TOP2: idx is [N, 2] (second entry -1 when K = 1) and hist counts both memberships.
// The product is computed transposed (centroids are the rows of the accumulator), so a lane holds scores of one point of
// each of its four blocks for ascending centroids and folds them into that point's running entry without a merge.
template <bool TOP2>
__global__ void __launch_bounds__(256, 2) route_kernel(const float* __restrict__ z, long ldz, const float* __restrict__ c,
                                                       const float* __restrict__ lin_bias, long N, int D, int K,
                                                       int* __restrict__ idx, unsigned long long* __restrict__ hist,
                                                       float* __restrict__ margin) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ __attribute__((aligned(16))) float cnorm[RB];
  __shared__ unsigned int lhist[R_MAX_K];
  __shared__ float third[4][256];   // a thread's own third best scores: registers are full

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int wc = wave >> 1, wp = wave & 1;   // the wave's 64 centroids of a tile, its 64 points
  const long m0 = (long)blockIdx.x * RB;
  const int rows_left = (int)min((long)RB, N - m0);
  const float* const zb = z + m0 * ldz;
  const float dot_mul = lin_bias ? 1.0f : 2.0f;
  for (int k = tid; k < K; k += 256) lhist[k] = 0;
  const int nkt = (D + RBK - 1) / RBK;

  // staging: wave w loads and splits rows 32 w .. 32 w + 31 of both tiles.  Rows beyond the last point or centroid read that one
  // (their scores are dropped, or +inf)
  using Unit = SplitUnit<true>;
  Unit sc, sz;
  uint32_t off_c[4], off_z[4];
  auto load = [&](int n0, int kt) {
    const int klim = D - kt * RBK;
    if (kt == 0 || klim < RBK) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = 32 * wave + Unit::row(lane, j), k = min(Unit::k(lane, j), klim - 4);
        off_c[j] = (uint32_t)(((long)min(row, K - n0 - 1) * D + k) * 4);
        off_z[j] = (uint32_t)(((long)min(row, rows_left - 1) * ldz + k) * 4);
      }
    }
    const char* const cb = reinterpret_cast<const char*>(c + (long)n0 * D + kt * RBK);
    const char* const pb = reinterpret_cast<const char*>(zb + kt * RBK);
#pragma unroll
    for (int j = 0; j < 4; ++j) sc.load(cb, off_c[j], j);
#pragma unroll
    for (int j = 0; j < 4; ++j) sz.load(pb, off_z[j], j);
  };
  int store_at[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) store_at[q] = 32 * SPLIT_ROW * wave + Unit::store_offset(lane, q);
  const SplitFragments frag(lane);
  const char* const pc = smem + wc * 64 * SPLIT_ROW;
  const char* const pz = smem + 3 * R_PLANE + wp * 64 * SPLIT_ROW;

  Best run[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) { run[j].s1 = INFINITY; run[j].i1 = NO_INDEX; run[j].s2 = INFINITY; run[j].i2 = NO_INDEX; }
#pragma unroll
  for (int j = 0; j < 4; ++j) third[j][tid] = INFINITY;
  float zn[4] = {0.f, 0.f, 0.f, 0.f};   // |z|^2 of the pieces the lane stages, of their first parts, times the tiles of centroids
  float c2 = 0.f;   // the largest |c|^2 the lane has seen

  load(0, 0);
  for (int n0 = 0; n0 < K; n0 += RB) {
    f32x4 acc[4][4];
    float nrm[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
    for (int kt = 0; kt < nkt; ++kt) {
      const int klim = D - kt * RBK;
      if (klim < RBK) {   // K beyond the range counts as zero
        sc.cut(lane, klim);
        sz.cut(lane, klim);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        nrm[q] += piece_squares(sc.v[q][0], sc.v[q][1], sc.v[q][2], sc.v[q][3]);
        sc.template store<R_PLANE>(smem + store_at[q], q);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint2 first = sz.template store<R_PLANE>(smem + 3 * R_PLANE + store_at[q], q);
        zn[q] = add_squares(first.x, add_squares(first.y, zn[q]));   // for every tile of centroids: a branch for the first one costs more
      }
      if (kt + 1 < nkt) load(n0, kt + 1);
      else if (n0 + RB < K) load(n0 + RB, 0);
      __syncthreads();
      __builtin_amdgcn_s_setprio(1);
      split_multiply<4, 4, R_PLANE, R_PLANE>(acc, pc, pz, frag);
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
    }
    // ||c||^2: lane l staged piece l % 8 of the wave's centroid rows l / 8 + 8 q.  The barriers of the next tile's first stage stand
    // between these reads of cnorm and its next writes
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v = nrm[q];
      v += __shfl_xor(v, 1, WAVE);
      v += __shfl_xor(v, 2, WAVE);
      v += __shfl_xor(v, 4, WAVE);
      c2 = fmaxf(c2, v);   // a NaN passes by: such a centroid is nobody's
      if ((lane & 7) == 0) {
        const int col = 32 * wave + (lane >> 3) + 8 * q;
        // linear router: the score to minimise is -(w_k.z + b_k), so -b_k takes the place of ||c_k||^2
        // a centroid beyond K scores +inf: it never enters a best entry
        cnorm[col] = n0 + col < K ? (lin_bias ? -lin_bias[n0 + col] : v) : INFINITY;
      }
    }
    __syncthreads();
    const int k0 = 64 * wc + 4 * kg;   // the lane's rows of block i: k0 + 16 i + e
    float s3[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s3[j] = third[j][tid];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 cn4 = *reinterpret_cast<const float4*>(cnorm + k0 + 16 * i);
      const float cn[4] = {cn4.x, cn4.y, cn4.z, cn4.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float s = __builtin_fmaf(-dot_mul, acc[i][j][e], cn[e]);
          third_push(s3[j], run[j], s);
          best_push_ascending<true>(run[j], s, n0 + k0 + 16 * i + e);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) third[j][tid] = s3[j];
  }

  // the four lane groups of a point, then the two waves that share its points, through LDS (the planes are free: every wave has passed
  // the barriers that end the last stage)
  float* const red_s1 = reinterpret_cast<float*>(smem);
  float* const red_s2 = red_s1 + 2 * RB;
  float* const red_s3 = red_s2 + 2 * RB;
  int* const red_i1 = reinterpret_cast<int*>(red_s3 + 2 * RB);
  int* const red_i2 = red_i1 + 2 * RB;
  float* const red_z2 = reinterpret_cast<float*>(red_i2 + 2 * RB);   // [4][256]
  float* const red_c2 = red_z2 + 4 * 256;
  int* const red_again = reinterpret_cast<int*>(red_c2 + 4);
  float* const again_s1 = reinterpret_cast<float*>(red_again + 4);
  float* const again_s2 = again_s1 + RB;
  int* const again_i1 = reinterpret_cast<int*>(again_s2 + RB);
  int* const again_i2 = again_i1 + RB;
  static_assert((22 * RB + 8) * sizeof(float) <= R_LDS, "the merge arrays fit in the planes");
#pragma unroll
  for (int q = 0; q < 4; ++q) red_z2[256 * q + tid] = zn[q];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float s3 = third[j][tid];
#pragma unroll
    for (int m = 16; m < WAVE; m <<= 1) {
      Best o;
      o.s1 = __shfl_xor(run[j].s1, m, WAVE); o.i1 = __shfl_xor(run[j].i1, m, WAVE); o.s2 = __shfl_xor(run[j].s2, m, WAVE);
      o.i2 = __shfl_xor(run[j].i2, m, WAVE);
      s3 = third_merge(run[j], s3, o, __shfl_xor(s3, m, WAVE));
      run[j] = best_merge<true>(run[j], o);
    }
    if (kg == 0) {
      const int at = wc * RB + 64 * wp + 16 * j + r;
      red_s1[at] = run[j].s1; red_i1[at] = run[j].i1; red_s2[at] = run[j].s2; red_i2[at] = run[j].i2; red_s3[at] = s3;
    }
  }
  c2 = wave_max(c2);
  if (lane == 0) red_c2[wave] = c2;
  __syncthreads();
  const int point = 32 * wave + (lane & 31);   // both halves of the wave hold its 32 points
  Best b, o;
  b.s1 = red_s1[point]; b.i1 = red_i1[point]; b.s2 = red_s2[point]; b.i2 = red_i2[point];
  o.s1 = red_s1[RB + point]; o.i1 = red_i1[RB + point]; o.s2 = red_s2[RB + point]; o.i2 = red_i2[RB + point];
  const float s3 = third_merge(b, red_s3[point], o, red_s3[RB + point]);
  b = best_merge<true>(b, o);
  c2 = fmaxf(fmaxf(red_c2[0], red_c2[1]), fmaxf(red_c2[2], red_c2[3]));
  float z2 = 0.f;   // point p of the wave: the eight lanes 8 (p % 8) + t staged its pieces as their row p / 8
#pragma unroll
  for (int t = 0; t < 8; ++t) z2 += red_z2[256 * ((lane & 31) >> 3) + 64 * wave + 8 * (lane & 7) + t];
  z2 *= __builtin_amdgcn_rcpf((float)((K + RB - 1) / RB));
  const bool on = point < rows_left;
  const float width = near_tie_width(z2, c2, D, dot_mul, b.s1, b.s2);
  // what is not finite compares false: rows of NaN have no scores, those of infinities are told by their norm
  const bool again = on && (fmaxf(z2, c2) >= LARGE_NORM2 || s3 - (TOP2 ? b.s2 : b.s1) < width);
  const bool near = on && !again && b.i2 != NO_INDEX && b.s2 - b.s1 < width;
  const float* const z_row = zb + (long)min(point, rows_left - 1) * ldz;
  if (__any(near)) decide_near_tie(b, near, z_row, c, lin_bias, D, dot_mul, lane);
  const bool wave_again = __any(again);
  if (lane == 0) red_again[wave] = wave_again ? 1 : 0;
  __syncthreads();
  for (int w = 0; w < 4; ++w) {
    if (!red_again[w]) continue;   // uniform
    // the points of wave w, every wave a quarter of the centroids (two nearest of 200000 x 896 x 200 849 us with wave w alone, 686 so)
    const Best part = again_in_fp32(zb + (long)min(32 * w + (lane & 31), rows_left - 1) * ldz, c, lin_bias, D, K, wave, 4, dot_mul, lane);
    if (lane < 32) {
      const int at = 32 * wave + lane;
      again_s1[at] = part.s1; again_i1[at] = part.i1; again_s2[at] = part.s2; again_i2[at] = part.i2;
    }
    __syncthreads();
    if (again && wave == w) {
      b.s1 = b.s2 = INFINITY; b.i1 = b.i2 = NO_INDEX;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int at = 32 * q + (lane & 31);
        Best o;
        o.s1 = again_s1[at]; o.i1 = again_i1[at]; o.s2 = again_s2[at]; o.i2 = again_i2[at];
        b = best_merge<true>(b, o);
      }
    }
    __syncthreads();   // the entries are read: the next points' may be written
  }
  if (lane < 32 && point < rows_left) {
    // A row none of whose scores compares below +inf (NaN or infinite features: a diverged path) never entered an
    // entry.  It is given the first centroid (the first two with TOP2) and a NaN margin, which is what the plain
    // definition's argmin over a row of NaN distances yields; it must not reach the histogram with an unset index.
    if (b.i1 == NO_INDEX) {
      b.i1 = 0;
      b.i2 = K > 1 ? 1 : NO_INDEX;
      b.s1 = b.s2 = __builtin_nanf("");
    }
    if (TOP2) {
      const bool has2 = b.i2 != NO_INDEX;
      idx[2 * (m0 + point)] = b.i1;
      idx[2 * (m0 + point) + 1] = has2 ? b.i2 : -1;
      if (has2) atomicAdd(&lhist[b.i2], 1u);
    } else {
      idx[m0 + point] = b.i1;
    }
    if (margin) margin[m0 + point] = b.s2 - b.s1;
    atomicAdd(&lhist[b.i1], 1u);
  }
  __syncthreads();
  for (int k = tid; k < K; k += 256) {
    const unsigned int v = lhist[k];
    if (v) atomicAdd(&hist[k], (unsigned long long)v);
  }
}

// ---- few points, or few centroids ----------------------------------------------------------------------------
// A workgroup of route_kernel owns 128 points and multiplies them with 128 centroids at a time: a batch of N points runs
// on N / 128 compute units and takes the time of one workgroup, a serial walk over 128 D, however small it is, and fewer
// than 128 centroids are padded.  Here a wave owns 16 PT points and 32 centroids of a sweep (v_mfma_f32_16x16x4_f32): wc
// waves of a workgroup take different centroids, 8 / wc different points.  A wave stages its own operand rows, K tiles of
// 32 in a ring of ST stages, straight into LDS: a lane-to-row assignment in which eight adjacent lanes read one 128-byte
// line (fragments fetched directly would touch 16 lines per 16 lanes: measured 44 us against 25 at 100 x 896 x 256).
// Nothing is shared between waves before the end, so there is no barrier in the loop.  The product is computed transposed
// (centroids are the rows of the accumulator), so a lane holds scores of one point for ascending centroids and folds
// them into its running entry without a merge.
constexpr int RS_WAVES = 8;
constexpr int RS_LDS_HIST = 256;
template <int PT> struct RouteSmall {
  static constexpr int ST = PT == 1 ? 3 : 2;                  // 144 KB / 128 KB of LDS
  static constexpr int STAGE = (32 + 16 * PT) * TILE_ROW_BYTES;
  static constexpr int LOADS = STAGE / 1024;                  // wave-level loads per stage
  static constexpr int LDS = RS_WAVES * ST * STAGE;
};

// Bounds: point and centroid rows are clamped to the last valid one (their scores are dropped, or +inf); K indices
// beyond D read the last four elements and are zeroed on both sides when they are used.
template <bool TOP2, int PT>
__global__ void __launch_bounds__(RS_WAVES * WAVE) route_small_kernel(const float* __restrict__ z, long ldz,
                                                                      const float* __restrict__ c,
                                                                      const float* __restrict__ lin_bias, long N, int D,
                                                                      int K, int wc, int* __restrict__ idx,
                                                                      unsigned long long* __restrict__ hist,
                                                                      float* __restrict__ margin) {
  using P = RouteSmall<PT>;
  constexpr int PTS = 16 * PT, ST = P::ST, STAGE = P::STAGE, LOADS = P::LOADS;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ float red_s1[RS_WAVES][PTS], red_s2[RS_WAVES][PTS];
  __shared__ int red_i1[RS_WAVES][PTS], red_i2[RS_WAVES][PTS];
  __shared__ unsigned int lhist[RS_LDS_HIST];
  const bool use_lhist = K <= RS_LDS_HIST;   // more centroids: a workgroup's few points go to the global counts directly
  if (use_lhist && threadIdx.x < RS_LDS_HIST) lhist[threadIdx.x] = 0;   // its first use is behind the barrier below
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int wk = wave & (wc - 1), wp = wave / wc;              // wc is a power of two
  const long m0 = ((long)blockIdx.x * (RS_WAVES / wc) + wp) * PTS;
  const int rows_left = (int)max(0L, min((long)PTS, N - m0));   // wave-uniform
  const float dot_mul = lin_bias ? 1.0f : 2.0f;

  Best run[PT];
#pragma unroll
  for (int p = 0; p < PT; ++p) { run[p].s1 = INFINITY; run[p].i1 = NO_INDEX; run[p].s2 = INFINITY; run[p].i2 = NO_INDEX; }

  // load i of a stage covers tile rows 8 i .. 8 i + 7 (rows 0..31 centroids, then the points), lane l chunk l & 7 of row
  // l >> 3 at chunk position (l & 7): the swizzle is applied by choosing which chunk that is
  char* const ring = smem + wave * ST * STAGE;
  const uint32_t ring_addr = (uint32_t)(uintptr_t)ring;
  const int nst = (D + RBK - 1) / RBK;
  const int lrow = lane >> 3;
  for (int c0 = 32 * wk; rows_left > 0 && c0 < K; c0 += 32 * wc) {   // wave-uniform
    const float* src[LOADS];
    int chunk[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int row = 8 * i + lrow;
      src[i] = row < 32 ? c + (long)min(c0 + row, K - 1) * D : z + (m0 + min(row - 32, rows_left - 1)) * ldz;
      chunk[i] = 4 * ((lane & 7) ^ swz(row));
    }
    auto issue = [&](int kt, int stage) {
#pragma unroll
      for (int i = 0; i < LOADS; ++i)
        load16_to_lds(src[i] + min(kt * RBK + chunk[i], D - 4), ring_addr + stage * STAGE + i * 1024);
    };
    f32x4 acc[2][PT];
    float nrm[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][p][e] = 0.f;

#pragma unroll
    for (int s = 0; s < ST; ++s)
      if (s < nst) issue(s, s);
    int stage = 0;
    for (int kt = 0; kt < nst; ++kt) {
      // own loads of tile kt have landed: all but those of the tiles behind it
      const int behind = min(ST - 1, nst - 1 - kt);
      if (ST > 2 && behind == 2) wait_vmcnt<2 * LOADS>();
      else if (behind == 1) wait_vmcnt<LOADS>();
      else wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      char* const tile = ring + stage * STAGE;
      float4 fc[2][2], fz[2][PT];   // [16-deep half][row tile]
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int j = 0; j < 2; ++j) fc[h][j] = *reinterpret_cast<const float4*>(tile_chunk(tile, 16 * j + r, 4 * h + kg));
#pragma unroll
        for (int p = 0; p < PT; ++p) fz[h][p] = *reinterpret_cast<const float4*>(tile_chunk(tile, 32 + 16 * p + r, 4 * h + kg));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the fragments are in registers: the stage may be refilled
      __builtin_amdgcn_sched_barrier(0);
      if (kt + ST < nst) issue(kt + ST, stage);
      stage = stage + 1 == ST ? 0 : stage + 1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (kt * RBK + 16 * h + 4 * kg >= D) {   // only in the last tile
#pragma unroll
          for (int j = 0; j < 2; ++j) fc[h][j] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int p = 0; p < PT; ++p) fz[h][p] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float4 v = fc[h][j];
          nrm[j] += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)   // the same K on both operands; 2 PT independent accumulators in turn
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int p = 0; p < PT; ++p)
              acc[j][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&fc[h][j])[q],
                                                               reinterpret_cast<const float*>(&fz[h][p])[q], acc[j][p], 0, 0, 0);
      }
    }

    // ||c||^2 of centroid row r of a tile: summed over the four lane groups, then handed to the lanes that hold the row
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      nrm[j] += __shfl_xor(nrm[j], 16, WAVE);
      nrm[j] += __shfl_xor(nrm[j], 32, WAVE);
      const int mine = c0 + 16 * j + r;
      const float cn = mine < K ? (lin_bias ? -lin_bias[mine] : nrm[j]) : INFINITY;   // beyond K: never enters an entry
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = 4 * kg + e;
        const float cne = __shfl(cn, row, WAVE);
#pragma unroll
        for (int p = 0; p < PT; ++p)
          best_push_ascending<TOP2>(run[p], __builtin_fmaf(-dot_mul, acc[j][p][e], cne), c0 + 16 * j + row);
      }
    }
  }

  // the four lane groups of a point, then the wc waves that share its points (disjoint centroids: a selection in the (score, index) order)
#pragma unroll
  for (int p = 0; p < PT; ++p) {
#pragma unroll
    for (int m = 16; m < WAVE; m <<= 1) {
      Best o;
      o.s1 = __shfl_xor(run[p].s1, m, WAVE); o.i1 = __shfl_xor(run[p].i1, m, WAVE); o.s2 = __shfl_xor(run[p].s2, m, WAVE);
      o.i2 = TOP2 ? __shfl_xor(run[p].i2, m, WAVE) : NO_INDEX;
      run[p] = best_merge<TOP2>(run[p], o);
    }
    if (lane < 16) {
      red_s1[wave][16 * p + r] = run[p].s1; red_s2[wave][16 * p + r] = run[p].s2;
      red_i1[wave][16 * p + r] = run[p].i1; red_i2[wave][16 * p + r] = run[p].i2;
    }
  }
  __syncthreads();
  const bool on = wk == 0 && lane < rows_left;
  Best b;
  b.i1 = -1; b.i2 = -1;
  if (on) {
    b.s1 = red_s1[wave][lane]; b.i1 = red_i1[wave][lane]; b.s2 = red_s2[wave][lane]; b.i2 = red_i2[wave][lane];
    for (int w = wave + 1; w < wave + wc; ++w) {
      Best o;
      o.s1 = red_s1[w][lane]; o.i1 = red_i1[w][lane]; o.s2 = red_s2[w][lane]; o.i2 = red_i2[w][lane];
      b = best_merge<TOP2>(b, o);
    }
    if (b.i1 == NO_INDEX) {   // no score below +inf (NaN or infinite features): as in route_kernel
      b.i1 = 0;
      b.i2 = K > 1 ? 1 : NO_INDEX;
      b.s1 = b.s2 = __builtin_nanf("");
    }
    if (TOP2) {
      if (b.i2 == NO_INDEX) b.i2 = -1;
      idx[2 * (m0 + lane)] = b.i1;
      idx[2 * (m0 + lane) + 1] = b.i2;
    } else {
      idx[m0 + lane] = b.i1;
    }
    if (margin) margin[m0 + lane] = b.s2 - b.s1;
  }
  if (on) {
    if (use_lhist) {
      atomicAdd(&lhist[b.i1], 1u);
      if (TOP2 && b.i2 >= 0) atomicAdd(&lhist[b.i2], 1u);
    } else {
      atomicAdd(&hist[b.i1], 1ull);
      if (TOP2 && b.i2 >= 0) atomicAdd(&hist[b.i2], 1ull);
    }
  }
  if (use_lhist) {
    __syncthreads();
    if (tid < K && lhist[tid]) atomicAdd(&hist[tid], (unsigned long long)lhist[tid]);
  }
}

// ---- a batch of documents -----------------------------------------------------------------------------------------
// Fewer points than a round of the kernel above: there 100 x 896 x 256 are seven workgroups of 16 points, whose fp32 MFMAs are 12 us of
// a compute unit while most idle.  Here a wave takes PTS points and 64 centroids, a lane each: a chain of plain multiply-adds per score,
// the point's number handed to all lanes through a scalar register.  wc waves of a workgroup take different centroids, 4 / wc
// different points.  Four stages of 32 K in flight, straight into LDS; the numbers of the next tile are read under the
// multiply-adds of this one.  No barrier before the end.  Bound by what one compute unit reads through its L1 (every workgroup reads all
// centroids, 64 bytes a clock: 6 us of 917 KB) and, level with it, by the vector instructions of a tile; 11 us of a call are the two
// launches and the latencies of their ends.  Microseconds a call, kernel above -> this: 100 x 896 x 256 27.0 -> 17.9, 250 x 896 x 256 27.0 -> 19.0,
// 500 x 896 x 256 (two points a wave) 27.2 -> 23.1, 256 x 896 x 1000 89 -> 57, 100 x 896 x 64 25.9 -> 17.2, 100 x 64 x 256 level (11.1); with points and
// centroids from memory, every workgroup's trip to them on the way, 100 x 896 x 256 27.8 -> 20.7, one point 27.4 -> 22.5.
// Left out: v_mfma_f32_4x4x1_16b_f32 with four points a matrix row (a dependent one takes 20 clocks: 27 us for any N up to 2048).
// The chain of a score takes K as v_mfma_f32_16x16x4_f32 does above (0, 4, 8, 12, 1, 5, .. of every sixteen) and ||c||^2 is
// added up in the same four sums: the same scores, bit for bit.
constexpr int RF_WAVES = 4, RF_ST = 4;
constexpr int RF_STAGE = (64 + 8) * TILE_ROW_BYTES, RF_LOADS = RF_STAGE / 1024;
constexpr int RF_LDS = RF_WAVES * RF_ST * RF_STAGE;

template <bool TOP2, int PTS>
__global__ void __launch_bounds__(RF_WAVES * WAVE) route_few_kernel(const float* __restrict__ z, long ldz, const float* __restrict__ c,
                                                                    const float* __restrict__ lin_bias, long N, int D, int K, int wc,
                                                                    int* __restrict__ idx, float* __restrict__ margin) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ Best red[RF_WAVES][PTS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave & (wc - 1), wp = wave / wc;   // wc is a power of two
  const long m0 = ((long)blockIdx.x * (RF_WAVES / wc) + wp) * PTS;
  const int rows_left = (int)max(0L, min((long)PTS, N - m0));   // wave-uniform
  const float dot_mul = lin_bias ? 1.0f : 2.0f;

  Best run[PTS];
#pragma unroll
  for (int p = 0; p < PTS; ++p) { run[p].s1 = INFINITY; run[p].i1 = NO_INDEX; run[p].s2 = INFINITY; run[p].i2 = NO_INDEX; }

  char* const ring = smem + wave * RF_ST * RF_STAGE;
  const uint32_t ring_addr = (uint32_t)(uintptr_t)ring;
  const int nst = (D + RBK - 1) / RBK, lrow = lane >> 3;
  for (int c0 = 64 * wk; rows_left > 0 && c0 < K; c0 += 64 * wc) {   // wave-uniform
    // load i of a stage covers rows 8 i .. 8 i + 7: 64 centroids, then the points; rows beyond the last re-read it, K beyond D the last
    // four.  The bases move on with the tiles, which are requested in order
    const float* base_c = c + (long)c0 * D;
    const float* base_z = z + m0 * ldz;
    uint32_t off[RF_LOADS];
    auto offsets = [&](int last) {   // `last`: the first of the last four K, from the tile's first one
#pragma unroll
      for (int i = 0; i < RF_LOADS; ++i) {
        const long row = i < 8 ? (long)min(8 * i + lrow, K - 1 - c0) * D : min(lrow, rows_left - 1) * ldz;
        off[i] = (uint32_t)((row + min(4 * ((lane & 7) ^ swz(8 * i + lrow)), last)) * 4);
      }
    };
    offsets(RBK);
    auto issue = [&](int kt, int stage) {
      if (D - kt * RBK < RBK) offsets(D - kt * RBK - 4);   // the last tile
#pragma unroll
      for (int i = 0; i < RF_LOADS; ++i)
        load16_to_lds_at(i < 8 ? base_c : base_z, off[i], __builtin_amdgcn_readfirstlane(ring_addr + stage * RF_STAGE + i * 1024));
      base_c += RBK; base_z += RBK;
    };
    auto landed = [&](int kt) {   // own loads of tile kt: all but those of the tiles behind it
      const int behind = min(RF_ST - 1, nst - 1 - kt);
      if (behind == 3) wait_vmcnt<3 * RF_LOADS>();
      else if (behind == 2) wait_vmcnt<2 * RF_LOADS>();
      else if (behind == 1) wait_vmcnt<RF_LOADS>();
      else wait_vmcnt<0>();
      asm volatile("" ::: "memory");
    };
    float4 fc[2][8];       // the lane's centroid, 32 K
    int fz[2][PTS];        // lane l: K l % 32 of a point
    auto read = [&](auto SET, int stage) {
      constexpr int set = decltype(SET)::value;
      char* const tile = ring + stage * RF_STAGE;
#pragma unroll
      for (int p = 0; p < PTS; ++p) fz[set][p] = reinterpret_cast<const int*>(tile_chunk(tile, 64 + p, (lane >> 2) & 7))[lane & 3];
#pragma unroll
      for (int q = 0; q < 8; ++q) fc[set][q] = *reinterpret_cast<const float4*>(tile_chunk(tile, lane, q));
    };
    float dot[PTS], nrm[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < PTS; ++p) dot[p] = 0.f;
    auto multiply = [&](auto SET, auto WHOLE, int left) {   // `left`: K of the tile, a multiple of 4
      constexpr int set = decltype(SET)::value;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        auto on = [&](int kg) { return decltype(WHOLE)::value || 16 * h + 4 * kg < left; };
#pragma unroll
        for (int p = 0; p < PTS; ++p) {   // sixteen scalars together: read and used in turn each pair is a stall
          float zs[16];
#pragma unroll
          for (int k = 0; k < 16; ++k) zs[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(fz[set][p], 16 * h + k));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int kg = 0; kg < 4; ++kg)
              if (on(kg)) dot[p] = __builtin_fmaf(zs[4 * kg + q], reinterpret_cast<const float*>(&fc[set][4 * h + kg])[q], dot[p]);
        }
#pragma unroll
        for (int kg = 0; kg < 4; ++kg)
          if (on(kg)) {
            const float4 v = fc[set][4 * h + kg];
            nrm[kg] += __builtin_fmaf(v.w, v.w, __builtin_fmaf(v.z, v.z, __builtin_fmaf(v.x, v.x, v.y * v.y)));
          }
      }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    auto registers_filled = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); __builtin_amdgcn_sched_barrier(0); };
#pragma unroll
    for (int s = 0; s < RF_ST; ++s)
      if (s < nst) issue(s, s);
    landed(0);
    read(C0{}, 0);
    registers_filled();
    auto step = [&](auto SET, int kt) {   // tile kt is in registers; its stage takes tile kt + RF_ST
      constexpr int set = decltype(SET)::value;
      if (kt + RF_ST < nst) issue(kt + RF_ST, kt % RF_ST);
      if (kt + 1 < nst) {
        landed(kt + 1);
        read(std::integral_constant<int, set ^ 1>{}, (kt + 1) % RF_ST);
      }
      if (D - kt * RBK >= RBK) multiply(SET, std::true_type{}, RBK);   // uniform
      else multiply(SET, std::false_type{}, D - kt * RBK);
      registers_filled();
    };
    for (int kt = 0; kt < nst; kt += 2) {
      step(C0{}, kt);
      if (kt + 1 < nst) step(C1{}, kt + 1);
    }
    const int mine = c0 + lane;   // beyond K: never enters an entry
    const float cn = mine < K ? (lin_bias ? -lin_bias[mine] : (nrm[0] + nrm[1]) + (nrm[2] + nrm[3])) : INFINITY;
#pragma unroll
    for (int p = 0; p < PTS; ++p) best_push_ascending<TOP2>(run[p], __builtin_fmaf(-dot_mul, dot[p], cn), mine);
  }

  auto from = [&](const Best& b, int m) {
    Best o;
    o.s1 = __shfl_xor(b.s1, m, WAVE); o.i1 = __shfl_xor(b.i1, m, WAVE); o.s2 = __shfl_xor(b.s2, m, WAVE);
    o.i2 = TOP2 ? __shfl_xor(b.i2, m, WAVE) : NO_INDEX;
    return o;
  };
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
    for (int p = 0; p < PTS; ++p) run[p] = best_merge<TOP2>(run[p], from(run[p], m));
  if (lane == 0) {
#pragma unroll
    for (int p = 0; p < PTS; ++p) red[wave][p] = run[p];
  }
  __syncthreads();
  if (wk == 0 && lane < rows_left) {
    Best b = red[wave][lane];
    for (int w = wave + 1; w < wave + wc; ++w) b = best_merge<TOP2>(b, red[w][lane]);
    if (b.i1 == NO_INDEX) {   // no score below +inf (NaN or infinite features): as in route_kernel
      b.i1 = 0;
      b.i2 = K > 1 ? 1 : NO_INDEX;
      b.s1 = b.s2 = __builtin_nanf("");
    }
    if (TOP2) {
      idx[2 * (m0 + lane)] = b.i1;
      idx[2 * (m0 + lane) + 1] = b.i2 == NO_INDEX ? -1 : b.i2;
    } else {
      idx[m0 + lane] = b.i1;
    }
    if (margin) margin[m0 + lane] = b.s2 - b.s1;
  }
}
// Its histogram, in place of the zeros that the other kernels add to: hist[k] = how many of the n indices are k.  The few points of a workgroup
// share no centroid in general, and additions to memory take 9 ns each behind the others of their 128-byte line: 900 x 256 x 4 19.1 us with them, 11.2 so (11.4 in
// route_small_kernel), 900 x 640 x 30 18.4 -> 14.2, 1000 x 896 x 64 22.6 -> 18.1; where all points are of one centroid 500 x 896 x 256 26.8 -> 22.1 us
// (26.6), their two nearest 900 x 64 x 4 27.2 -> 11.3 (10.9); 100 x 896 x 256 18.6 -> 17.9.
constexpr int RF_MOST = 2 * 256 * RF_WAVES, RF_COUNT_THREADS = 512, MOST_CENTROIDS = 4096;   // indices of a launch; centroids of a call
__global__ void __launch_bounds__(RF_COUNT_THREADS) route_count_kernel(const int* __restrict__ idx, int n, int K, unsigned long long* __restrict__ hist) {
  __shared__ int counts[MOST_CENTROIDS];
  const int tid = threadIdx.x;
  int mine[RF_MOST / RF_COUNT_THREADS];
#pragma unroll
  for (int i = 0; i < RF_MOST / RF_COUNT_THREADS; ++i) {
    const int at = tid + RF_COUNT_THREADS * i;
    mine[i] = at < n ? idx[at] : -1;
  }
  for (int k = tid; k < K; k += RF_COUNT_THREADS) counts[k] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RF_MOST / RF_COUNT_THREADS; ++i)
    if ((unsigned)mine[i] < (unsigned)K) atomicAdd(&counts[mine[i]], 1);
  __syncthreads();
  for (int k = tid; k < K; k += RF_COUNT_THREADS) hist[k] = (unsigned long long)counts[k];
}

// ---- K-class logistic regression: per-row softmax cross-entropy --------------------------------------------------
// One wave per row of logits [rows, K] (K a multiple of 4, at most LOGIT_MAX_K): nll[row] = logsumexp - logit[label],
// and in place logits <- (softmax - onehot(label)) * inv_n.  A row whose label is outside [0, K) gives 0 and zeros.
constexpr int LOGIT_MAX_VEC = 16;                 // float4 per lane
constexpr int LOGIT_MAX_K = 64 * 4 * LOGIT_MAX_VEC;
__global__ void __launch_bounds__(256) logistic_rows_kernel(float* __restrict__ logits, const int* __restrict__ labels,
                                                            long rows, int K, float inv_n, float* __restrict__ nll) {
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const int nvec = K >> 2;
  float4* lr = reinterpret_cast<float4*>(logits + row * K);
  float4 v[LOGIT_MAX_VEC];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < LOGIT_MAX_VEC; ++i) {
    const int c = lane + 64 * i;
    if (c < nvec) {
      v[i] = lr[c];
      mx = fmaxf(mx, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  const int label = labels[row];
  const bool valid = label >= 0 && label < K;
  float sum = 0.f, at_label = 0.f;   // at_label: logit[label] - max, held by one lane
#pragma unroll
  for (int i = 0; i < LOGIT_MAX_VEC; ++i) {
    const int c = lane + 64 * i;
    if (c < nvec) {
      float x[4] = {v[i].x - mx, v[i].y - mx, v[i].z - mx, v[i].w - mx};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (valid && 4 * c + q == label) at_label = x[q];
      v[i].x = expf(x[0]); v[i].y = expf(x[1]); v[i].z = expf(x[2]); v[i].w = expf(x[3]);
      sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
  const float scale = valid ? inv_n / sum : 0.f;
#pragma unroll
  for (int i = 0; i < LOGIT_MAX_VEC; ++i) {
    const int c = lane + 64 * i;
    if (c < nvec) {
      float e[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
      float o[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = e[q] * scale - ((valid && 4 * c + q == label) ? inv_n : 0.f);
      lr[c] = make_float4(o[0], o[1], o[2], o[3]);
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) at_label += __shfl_xor(at_label, o, 64);
  if (lane == 0) nll[row] = valid ? logf(sum) - at_label : 0.f;
}

// The same for K <= 1024, where a row is at most four 16-byte vectors per lane: a wave takes up to eight rows at once, so that
// eight loads are in flight per lane instead of one (a million one-kilobyte rows are latency-bound otherwise), and the
// reductions run on the DPP lanes.  Rows behind the last are that one again, without a label, so that nothing branches between
// rows and their chains interleave; what a row has once (the quotient, the logarithm) is taken for all of them together, a lane each.
// Up to 128 (64, 32) classes a vector holds two (four, eight) rows, LANES lanes each: the instructions are a vector's, whatever it holds.
// Groups of ROWS vectors are dealt to at most 1024 workgroups, each of which leaves one row of partial sums: the column sums of what it
// stores (the bias gradient) and, in column K, its rows' losses; logistic_finish_kernel adds these rows.  Bound by its vector instructions and
// HBM together: 50000 x 256 28.7 us with the rows one behind the other, 22.1 so (the next group's rows requested ahead: 23.2); gradient of
// 300000 x 64 x 256 404 -> 372, 3000 x 64 x 256 27.1 -> 24.7, 1000000 x 64 x 128 833 -> 719, 676 with two rows a vector, 200000 x 64 x 64
// 182 -> 162, 130 with four, 1000000 x 64 x 8 579 -> 524, 351 with four, 327 with eight; 3000 x 64 x 64 and x 128 level.  Above 256
// classes a lane has VEC vectors of a row, and the row's loss, its mean and the column sums need no kernels and no pass of their own: 50000 x 768 x 512
// 614 -> 582, 50000 x 64 x 512 162 -> 127, 3000 x 64 x 512 51 -> 30, 50000 x 64 x 1024 256 -> 225; more than four would not leave the registers.
// A lane's rows grow with N (256 of 2^20): a group's are added in 32 bits, groups in 64, at no cost that shows (1048576 x 64 x 512 2561 us both ways).
// In one 32-bit chain like rows drift: weights of zero, 2^20 rows, K = 64 / 512 / 1024 off by 6.0e-7 / 2.6e-6 / 3.2e-6 of the summands'
// magnitude, so by 1.4e-7 - 1.6e-7, the rounding of a row's own values.
constexpr int LOGIT_SMALL_ROWS = 8, LOGIT_SMALL_BLOCKS = 1024, LOGIT_SMALL_K = 1024;
constexpr int logistic_stride(int K) { return K + 4; }   // floats between rows of partial sums
__device__ __forceinline__ float lane_value(float v, int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); }
// over a row's LANES lanes, in each of them
template <int LANES> __device__ __forceinline__ float row_max(float v) {
  if constexpr (LANES == 64) return wave_max(v);
  v = fmaxf(v, dpp_fetch<0xb1, 0xf>(v, -INFINITY));
  v = fmaxf(v, dpp_fetch<0x4e, 0xf>(v, -INFINITY));
  v = fmaxf(v, dpp_fetch<0x141, 0xf>(v, -INFINITY));
  if constexpr (LANES > 8) v = fmaxf(v, dpp_fetch<0x140, 0xf>(v, -INFINITY));
  return LANES == 32 ? fmaxf(v, __shfl_xor(v, 16, 64)) : v;
}
template <int LANES> __device__ __forceinline__ float row_sum(float v) {
  if constexpr (LANES == 64) return wave_sum(v);
  v += dpp_fetch<0xb1, 0xf>(v, 0.f);
  v += dpp_fetch<0x4e, 0xf>(v, 0.f);
  v += dpp_fetch<0x141, 0xf>(v, 0.f);
  if constexpr (LANES > 8) v += dpp_fetch<0x140, 0xf>(v, 0.f);
  return LANES == 32 ? v + __shfl_xor(v, 16, 64) : v;
}
template <int LANES, int VEC> __global__ void __launch_bounds__(256) logistic_rows_small_kernel(float* __restrict__ logits, const int* __restrict__ labels,
                                                                                                long rows, int K, float inv_n,
                                                                                                float* __restrict__ partial, int blocks) {
  constexpr int ROWS = LOGIT_SMALL_ROWS / VEC, PER = 64 / LANES, GROUP = ROWS * PER;   // K <= 4 LANES VEC
  static_assert(VEC == 1 || LANES == 64);
  constexpr int STRIDE = logistic_stride(4 * LANES * VEC);
  __shared__ __attribute__((aligned(16))) float red[4 * PER * STRIDE];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int piece = lane / LANES, x = lane % LANES;   // the lane's row of a vector, its place in it
  bool on[VEC];
  double sums[VEC][4];
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    on[k] = x + LANES * k < (K >> 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) sums[k][q] = 0.0;
  }
  double loss = 0.0;   // of lane i: of the i-th row of each group
  const long step = (long)blocks * 4 * GROUP;
  for (long row0 = ((long)blockIdx.x * 4 + wave) * GROUP; row0 < rows; row0 += step) {   // whole waves: the reductions see all 64 lanes
    float4 v[ROWS][VEC];
    int own_label = -1;
    if (lane < GROUP && row0 + lane < rows) own_label = labels[row0 + lane];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        v[r][k] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (on[k]) v[r][k] = reinterpret_cast<const float4*>(logits + std::min(row0 + r * PER + piece, rows - 1) * K)[x + LANES * k];
      }
    const bool own_valid = own_label >= 0 && own_label < K;
    if (!own_valid) own_label = -1;
    auto label_of = [&](int r) { return PER == 1 ? __builtin_amdgcn_readlane(own_label, r) : __shfl(own_label, r * PER + piece, 64); };
    // the lane that holds the first of the row of which lane i is the owner, and the label's
    const int own_first = lane % PER * LANES, own_holder = own_first + (own_valid ? own_label >> 2 : 0);
    float own_sum = 1.f, own_at = 0.f;   // own_at: logit[label] - max
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int label = label_of(r);
      float mx = -INFINITY, sum = 0.f, pick = 0.f;
#pragma unroll
      for (int k = 0; k < VEC; ++k) mx = fmaxf(mx, fmaxf(fmaxf(v[r][k].x, v[r][k].y), fmaxf(v[r][k].z, v[r][k].w)));
      mx = row_max<LANES>(mx);
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        float4& w = v[r][k];
        w = make_float4(w.x - mx, w.y - mx, w.z - mx, w.w - mx);
        const float p = label & 2 ? (label & 1 ? w.w : w.z) : (label & 1 ? w.y : w.x);
        if (k == 0 || label >> 8 == k) pick = p;
        w = make_float4(expf(w.x), expf(w.y), expf(w.z), expf(w.w));   // exp(-inf) = 0 off the row
        sum += (w.x + w.y) + (w.z + w.w);
      }
      const float at = PER == 1 ? lane_value(pick, label < 0 ? 0 : (label >> 2) % 64) : __shfl(pick, own_holder, 64);
      sum = row_sum<LANES>(sum);
      if constexpr (PER > 1) sum = __shfl(sum, own_first, 64);
      if (lane / PER == r) { own_sum = sum; own_at = at; }
    }
    const float own_scale = own_valid ? inv_n / own_sum : 0.f;
    loss += (double)(own_valid ? logf(own_sum) - own_at : 0.f);
    float group[VEC][4] = {};
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const int label = label_of(r);
      const float scale = PER == 1 ? lane_value(own_scale, r) : __shfl(own_scale, r * PER + piece, 64);
      const long row = row0 + r * PER + piece;
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        const float e[4] = {v[r][k].x, v[r][k].y, v[r][k].z, v[r][k].w};
        float o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[q] = e[q] * scale - (4 * (x + LANES * k) + q == label ? inv_n : 0.f);
          group[k][q] += o[q];
        }
        if (on[k] && row < rows) reinterpret_cast<float4*>(logits + row * K)[x + LANES * k] = make_float4(o[0], o[1], o[2], o[3]);
      }
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) sums[k][q] += (double)group[k][q];
  }
#pragma unroll
  for (int o = 1; o < GROUP; o <<= 1) loss += __shfl_xor(loss, o, 64);
  float* mine = red + (wave * PER + piece) * STRIDE;
#pragma unroll
  for (int k = 0; k < VEC; ++k)
    if (on[k]) *reinterpret_cast<float4*>(mine + 4 * (x + LANES * k)) = make_float4((float)sums[k][0], (float)sums[k][1], (float)sums[k][2], (float)sums[k][3]);
  if (x == 0) mine[K] = piece ? 0.f : (float)loss;
  __syncthreads();
  for (int c = threadIdx.x; c <= K; c += 256) {
    float t = red[c];
#pragma unroll
    for (int k = 1; k < 4 * PER; ++k) t += red[k * STRIDE + c];
    partial[(size_t)blockIdx.x * logistic_stride(K) + c] = t;
  }
}
// columns 0 .. K - 1 of the partial rows' sum to db, column K over n to loss.  Losses are of one sign and a chain of them drifts: both kernels
// add them in 64 bits.  In 32 the mean was off by 9.0e-8 (root mean square, 1000 .. 20000 rows), where a tree over the rows had 6.5e-8; so it
// is 2.8e-8, the rounding of the result, for 0.3 % (10^6 x 64 x 128 882 -> 884 us in all).
constexpr int LF_COLS = 32, LF_PHASES = 32;
__global__ void __launch_bounds__(LF_COLS * LF_PHASES) logistic_finish_kernel(const float* __restrict__ partial, int n_partials, int K, float n,
                                                                              float* __restrict__ db, float* __restrict__ loss) {
  __shared__ double red[LF_PHASES][LF_COLS + 1];
  const int x = threadIdx.x % LF_COLS, y = threadIdx.x / LF_COLS, c = blockIdx.x * LF_COLS + x;
  double s = 0.0;
  if (c <= K) {
#pragma unroll 8
    for (int p = y; p < n_partials; p += LF_PHASES) s += partial[(size_t)p * logistic_stride(K) + c];
  }
  red[y][x] = s;
  __syncthreads();
  if (y != 0 || c > K) return;
  double t = red[0][x];
#pragma unroll
  for (int q = 1; q < LF_PHASES; ++q) t += red[q][x];
  if (c < K) db[c] = (float)t;
  else loss[0] = (float)(t / (double)n);
}

}  // namespace

size_t logistic_partial_floats(int64_t rows, int K) {
  return std::max((size_t)LOGIT_SMALL_BLOCKS * logistic_stride(K), colsum_partial_floats((int)rows, K));
}

dipaco_status launch_logistic_rows(float* logits, const int* labels, int64_t rows, int K, float* nll, int* n_valid, float* partial, float* loss,
                                   float* db, hipStream_t s) {
  if (K < 4 || K % 4 || K > LOGIT_MAX_K) return fail(DIPACO_ESHAPE, "logistic rows: K must be a multiple of 4 in [4, 4096]");
  const float inv_n = (float)(1.0 / (double)rows);
  const int64_t blocks = (rows + 3) / 4;
  if (K > 256 && !launch_fits(blocks, 256)) return fail(DIPACO_ESHAPE, "logistic rows: too many rows");
  if (K <= LOGIT_SMALL_K) {
    auto run = [&](auto lanes, auto vec) {
      const int64_t per = 4 * LOGIT_SMALL_ROWS / vec * (64 / lanes);
      const int n = (int)std::min<int64_t>((rows + per - 1) / per, LOGIT_SMALL_BLOCKS);
      logistic_rows_small_kernel<lanes, vec><<<n, 256, 0, s>>>(logits, labels, (long)rows, K, inv_n, partial, n);
      return n;
    };
    using std::integral_constant;
    constexpr integral_constant<int, 1> one{};
    const int n = K <= 32 ? run(integral_constant<int, 8>{}, one) : K <= 64 ? run(integral_constant<int, 16>{}, one)
                  : K <= 128 ? run(integral_constant<int, 32>{}, one) : K <= 256 ? run(integral_constant<int, 64>{}, one)
                  : K <= 512 ? run(integral_constant<int, 64>{}, integral_constant<int, 2>{})
                             : run(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    DIPACO_LAUNCH_CHECK();
    logistic_finish_kernel<<<(K + 1 + LF_COLS - 1) / LF_COLS, LF_COLS * LF_PHASES, 0, s>>>(partial, n, K, (float)rows, db, loss);
    DIPACO_LAUNCH_CHECK();
    return DIPACO_OK;
  }
  logistic_rows_kernel<<<(unsigned)blocks, 256, 0, s>>>(logits, labels, (long)rows, K, inv_n, nll);
  DIPACO_LAUNCH_CHECK();
  dipaco_status st = launch_fill_i32(n_valid, (int)rows, 1, s);
  if (st != DIPACO_OK) return st;
  st = launch_mean_loss(nll, n_valid, loss, (int)rows, s);
  if (st != DIPACO_OK) return st;
  return launch_colsum(logits, db, partial, (int)rows, K, s);
}

// Waves of a small-kernel workgroup along the centroids: as many as there are groups of 32, so that none is idle.
static int route_small_wc(int K) { return K > 128 ? 8 : K > 64 ? 4 : K > 32 ? 2 : 1; }

// 1 / 2: route_small_kernel with 16 / 32 points per wave, 0: route_kernel.  All take time in whole rounds over the compute units,
// proportional to D.  Measured at D = 896: 512 workgroups of route_kernel (65536 points) with 256 centroids 169 us, up to 256 of them 125; a
// round of the small kernel with 32 points per wave (2048 wave tasks) 43 us, with 16 points 28 us.  The 16-point form is taken where one round
// of it holds everything (1000 x 256: 27 us, 45 with 32 points, 120 in route_kernel), below that route_few_kernel.  Else route_kernel where 230 us for a round of 65536
// points x 256 centroids would be the cheaper: at 16384 x 256 91 | 125 us, 65536 x 256 328 | 169, 300000 x 768 x 256 1300 | 720, x 16 202 | 371.
// The line lies where it did when route_kernel took those 230 us: nearer to it the two err differently (the small kernel's chain takes K
// in another order than decide_near_tie), and a program's assignments would turn at near-ties.
static int route_pick(int64_t N, int64_t ldz, int D, int K) {
  const int64_t wc = route_small_wc(K), sweeps = (K + 32 * wc - 1) / (32 * wc), tasks = 256 * RS_WAVES;
  if ((N + 15) / 16 * wc <= tasks) return 1;
  if (!launch_fits((N + 31) / 32 * wc / RS_WAVES + 1, RS_WAVES * WAVE)) return 0;
  if (std::max<int64_t>(ldz, D) * 4 * RB >= 1LL << 32) return 2;   // route_kernel's byte offsets within a tile are 32-bit
  const int64_t small = 43 * (((N + 31) / 32 * wc + tasks - 1) / tasks) * sweeps;
  const int64_t big = 230 * ((N + 65535) / 65536) * ((K + 255) / 256);
  return small < big ? 2 : 0;
}

// Points of a wave of route_few_kernel, 0: not taken.  While one round of 256 workgroups, one to a compute unit, holds the batch: a second
// round costs as much again (500 x 896 x 256 36.6 us with one point a wave, 23.6 with two, 27.2 in the kernel above).  Two points a wave only where a
// workgroup's waves share them: 1000 x 256 x 100 14.6 us, 12.9 above, 2000 x 896 x 64 33.0 | 26.6.  32-bit byte offsets within a tile.
static int route_few_points(int64_t N, int64_t ldz, int D, int wc) {
  if (std::max<int64_t>(64 * (int64_t)D, 2 * ldz) * 4 >= 1LL << 32) return 0;
  if (N * wc <= 256 * RF_WAVES) return 1;
  return wc == RF_WAVES && N <= 512 ? 2 : 0;
}

dipaco_status launch_route(const float* z, int64_t ldz, const float* c, const float* lin_bias, int64_t N, int D, int K,
                           int n_best, int* idx, long long* hist, float* margin, hipStream_t s) {
  auto* h = reinterpret_cast<unsigned long long*>(hist);
  const int pick = N ? route_pick(N, ldz, D, K) : 0;
  if (N && pick == 1) {
    const int fc = K > 128 ? 4 : K > 64 ? 2 : 1;
    auto few = [&](auto PTC) -> dipaco_status {
      constexpr int PTS = decltype(PTC)::value;
      static std::atomic<unsigned long long> set_one{0}, set_two{0};
      if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_few_kernel<false, PTS>), RF_LDS, set_one)) return e;
      if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_few_kernel<true, PTS>), RF_LDS, set_two)) return e;
      const int64_t pts = PTS * (RF_WAVES / fc), nb = (N + pts - 1) / pts;
      if (n_best == 2) route_few_kernel<true, PTS><<<(unsigned)nb, RF_WAVES * WAVE, RF_LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, fc, idx, margin);
      else route_few_kernel<false, PTS><<<(unsigned)nb, RF_WAVES * WAVE, RF_LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, fc, idx, margin);
      DIPACO_LAUNCH_CHECK();
      route_count_kernel<<<1, RF_COUNT_THREADS, 0, s>>>(idx, (int)(N * n_best), K, h);
      DIPACO_LAUNCH_CHECK();
      return DIPACO_OK;
    };
    const int take = route_few_points(N, ldz, D, fc);
    if (take == 1) return few(std::integral_constant<int, 1>{});
    if (take == 2) return few(std::integral_constant<int, 2>{});
  }
  dipaco_status st = launch_fill_i64(hist, 0, (size_t)K, s);
  if (st != DIPACO_OK) return st;
  if (N == 0) return DIPACO_OK;
  const int wc = route_small_wc(K);
  auto small = [&](auto PTC) -> dipaco_status {
    constexpr int PT = decltype(PTC)::value, LDS = RouteSmall<PT>::LDS;
    static std::atomic<unsigned long long> set_one{0}, set_two{0};
    if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_small_kernel<false, PT>), LDS, set_one)) return e;
    if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_small_kernel<true, PT>), LDS, set_two)) return e;
    const int64_t pts = 16 * PT * (RS_WAVES / wc), nb = (N + pts - 1) / pts;
    if (n_best == 2) route_small_kernel<true, PT><<<(unsigned)nb, RS_WAVES * WAVE, LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, wc, idx, h, margin);
    else route_small_kernel<false, PT><<<(unsigned)nb, RS_WAVES * WAVE, LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, wc, idx, h, margin);
    DIPACO_LAUNCH_CHECK();
    return DIPACO_OK;
  };
  if (pick == 1) return small(std::integral_constant<int, 1>{});
  if (pick == 2) return small(std::integral_constant<int, 2>{});
  static std::atomic<unsigned long long> lds_one{0}, lds_two{0};
  if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_kernel<false>), R_LDS, lds_one)) return e;
  if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(route_kernel<true>), R_LDS, lds_two)) return e;
  const int64_t blocks = (N + RB - 1) / RB;
  if (!launch_fits(blocks, 256)) return fail(DIPACO_ESHAPE, "route: N too large");
  if (n_best == 2) route_kernel<true><<<(unsigned)blocks, 256, R_LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, idx, h, margin);
  else route_kernel<false><<<(unsigned)blocks, 256, R_LDS, s>>>(z, (long)ldz, c, lin_bias, (long)N, D, K, idx, h, margin);
  DIPACO_LAUNCH_CHECK();
  return DIPACO_OK;
}

}  // namespace dipaco

// Attention rows over their visible pairs alone, for a wave whose results are not finite.
//
// The matrix-core kernels multiply whole tiles: a pair that the causal mask hides, and a row past the end of the sequence, take part
// with probability 0.  0 x Inf and 0 x NaN are NaN, so one non-finite value would reach the rows of its tile that must not see it.  A
// row it reaches cannot end finite; so a wave that ends with any value of its valid rows not finite computes these rows once more
// here, pair by pair, and rows that see only finite values come out finite again.  No other wave pays more than a multiply-add per
// accumulator element.  Not for speed: LP lanes share a row, each forms the whole scores and keeps its columns 4 (LP i + sub) .. + 3.
#pragma once
#include "common.h"

namespace dipaco {

namespace plain {

template <int N> __device__ __forceinline__ bool not_finite(const f32x4 (&acc)[N]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) z = __builtin_fmaf(acc[i][e], 0.f, z);
  return z != z;
}
template <int N> __device__ __forceinline__ bool not_finite(const f32x16 (&acc)[N]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) z = __builtin_fmaf(acc[i][e], 0.f, z);
  return z != z;
}
template <int N> __device__ __forceinline__ void clear(f32x16 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
}
template <int N> __device__ __forceinline__ void clear(f32x4 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ void load4(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load4(const bf16* p, float (&v)[4]) {
  const bf16x4 t = *reinterpret_cast<const bf16x4*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = to_f32(t[e]);
}
// acc += w * row, this lane's columns: four lanes a row hold f32x4 tiles of 16 columns, two lanes f32x16 tiles of 32
template <int N> __device__ __forceinline__ void add_row(f32x4 (&acc)[N], float w, const float* row, int sub) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float v[4];
    load4(row + 16 * i + 4 * sub, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[i][e] += w * v[e];
  }
}

template <int N> __device__ __forceinline__ void add_row(f32x16 (&acc)[N], float w, const bf16* row, int sub) {
#pragma unroll
  for (int i = 0; i < 4 * N; ++i) {
    float v[4];
    load4(row + 8 * i + 4 * sub, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[i >> 2][4 * (i & 3) + e] += w * v[e];
  }
}

template <int DH, typename T> __device__ __forceinline__ float dot(const T* a, const T* b) {
  constexpr int VEC = Vec16<T>::N;
  float s = 0.f;
#pragma unroll 1
  for (int c = 0; c < DH; c += VEC) {
    float x[VEC], y[VEC];
    load_vec16(a + c, x);
    load_vec16(b + c, y);
#pragma unroll
    for (int e = 0; e < VEC; ++e) s += x[e] * y[e];
  }
  return s;
}

// O of query q: sum over j <= q of prob(q.k_j) v_j.  base: row 0 of this head's q in qkv (k at + A, v at + 2 A, rows ld apart)
template <int DH, typename T, typename ACC, typename PROB>
__device__ __forceinline__ void attend(ACC& o, const T* base, long ld, int A, int q, int sub, PROB prob) {
  clear(o);
#pragma unroll 1
  for (int j = 0; j <= q; ++j) {
    const T* k = base + (long)j * ld + A;
    add_row(o, prob(dot<DH>(base + (long)q * ld, k)), k + A, sub);
  }
}
// dQ of query q without the score scale: sum over j <= q of prob(q.k_j) (dO.v_j - D) k_j
template <int DH, typename T, typename ACC, typename PROB>
__device__ __forceinline__ void query_grad(ACC& dq, const T* base, const T* d_o, float D, long ld, int A, int q, int sub, PROB prob) {
  clear(dq);
#pragma unroll 1
  for (int j = 0; j <= q; ++j) {
    const T* k = base + (long)j * ld + A;
    add_row(dq, prob(dot<DH>(base + (long)q * ld, k)) * (dot<DH>(d_o, k + A) - D), k, sub);
  }
}
// dK (without the score scale) and dV of a key: sums over i >= key of p_i (dO_i.v - D_i) q_i and p_i dO_i, p_i = prob(q_i.k, i).
// gbase: row 0 of this head's dO (rows A apart)
template <int DH, typename T, typename ACC, typename PROB, typename STAT>
__device__ __forceinline__ void key_grads(ACC& dk, ACC& dv, const T* base, const T* gbase, long ld, int A, int key, int S, int sub,
                                          PROB prob, STAT D) {
  clear(dk);
  clear(dv);
  const T* k = base + (long)key * ld + A;
#pragma unroll 1
  for (int i = key; i < S; ++i) {
    const T* q = base + (long)i * ld;
    const T* g = gbase + (long)i * A;
    const float p = prob(dot<DH>(q, k), i);
    add_row(dv, p, g, sub);
    add_row(dk, p * (dot<DH>(g, k + A) - D(i)), q, sub);
  }
}

}  // namespace plain

}  // namespace dipaco

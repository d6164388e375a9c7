// Epilogue of the products whose workgroup is G groups of waves along K times WM x WN waves over the tile (gemm_fit.hip,
// gemm_split.hip): the groups' partial sums meet in LDS and are added in group order, then bias / activation / residual are
// applied on, and C is written with, eight columns per item.
#pragma once
#include <type_traits>

#include "gemm_common.h"

namespace dipaco {

constexpr int FIT_PAD = 4;   // floats between rows of the staging region
// LDS bytes of the staging region: 16 n16 rows of every wave at a time
constexpr int fit_epilogue_bytes(int n16, int TN, int WM, int WN, int G) { return G * WM * 16 * n16 * (16 * TN * WN + FIT_PAD) * 4; }

// The operands of the epilogue of a tile that is one item a thread (32 x 64 and smaller), requested in front of the product: behind it
// they are one more trip to memory, 0.5 - 0.7 of a launch of 4 - 6 us.
template <typename T> struct FitAhead { Raw8<T> bias, in; };
template <typename T, int TN, int TM, int NW> __device__ __forceinline__ FitAhead<T> fit_request(const GemmDev& g, int tid, int m0, int n0) {
  constexpr int CG = 2 * TN;
  static_assert(16 * TM * CG <= 64 * NW, "one item a thread");
  FitAhead<T> f;
  const int row = m0 + tid / CG, col = n0 + 8 * (tid % CG);
  if (g.splits > 1 || col >= g.N) return f;
  if (g.bias) f.bias = raw8_load(static_cast<const T*>(g.bias) + col);
  const T* const ahead = static_cast<const T*>(g.act == 2 || g.act == 4 ? g.aux_in : g.resid);
  if (ahead && tid / CG < 16 * TM && row < g.M) f.in = raw8_load(ahead + (size_t)row * g.ldc + col);
  return f;
}

// acc: the wave's TM x TN tiles of 16 x 16 (lane l: column l % 16, rows 4 (l / 16) + e), taken in two passes of IC and TM - IC
// tile rows.  red: LDS, free once every wave has reached this call.
// early: what fit_request has asked for, or null.
template <typename T, typename TC, int TM, int TN, int WM, int WN, int G, int IC>
__device__ __forceinline__ void fit_epilogue(const GemmDev& g, const f32x4 (&acc)[TM][TN], float* red, int tid, int grp, int wm, int wn,
                                             int m0, int n0, int tile_m, int split, const FitAhead<T>* early = nullptr) {
  static_assert(TM <= 2 * IC, "two passes");
  constexpr int NW = WM * WN * G, BN = 16 * TN * WN, LDW = BN + FIT_PAD, CG = BN / 8;
  const int lane = tid & 63, wave = tid >> 6, r = lane & 15, kg = lane >> 4;
  static_assert((64 * NW) % CG == 0, "a thread keeps its column group over the items");
  const int cg = tid % CG, col = n0 + 8 * cg;
  const bool col_ok = col < g.N, partial = g.splits > 1;
  const T* const bias = static_cast<const T*>(g.bias);
  const T* const resid = static_cast<const T*>(g.resid);
  const T* const aux_in = static_cast<const T*>(g.aux_in);
  const bool want_aux = g.act == 2 || g.act == 4;
  const T* const ahead = want_aux ? aux_in : resid;
  const long ldc = g.ldc;
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (bias && col_ok) raw8_unpack(early ? early->bias : raw8_load(bias + col), bv);
  auto pass = [&](auto I0, auto N16) {   // 16-row blocks I0 .. I0 + N16 - 1 of every wave
    constexpr int i0 = decltype(I0)::value, n16 = decltype(N16)::value;
    constexpr int ROWS = WM * 16 * n16, ITERS = (ROWS * CG + 64 * NW - 1) / (64 * NW);
    auto row_of = [&](int rr) { return m0 + (rr / (16 * n16)) * 16 * TM + 16 * i0 + rr % (16 * n16); };
    Raw8<T> rin[ITERS];
    if (early) {
      rin[0] = early->in;
    } else if (ahead) {
#pragma unroll
      for (int it = 0; it < ITERS; ++it) {
        const int rr = (tid + 64 * NW * it) / CG, row = row_of(rr);
        if (rr < ROWS && row < g.M && col_ok) rin[it] = raw8_load(ahead + (size_t)row * ldc + col);
      }
    }
    __syncthreads();   // the ring (or the pass before) has been read
#pragma unroll
    for (int i = 0; i < n16; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          red[((grp * WM + wm) * 16 * n16 + 16 * i + 4 * kg + e) * LDW + (wn * TN + j) * 16 + r] = acc[i0 + i][j][e];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const int rr = (tid + 64 * NW * it) / CG, row = row_of(rr);
      if (rr >= ROWS || row >= g.M || !col_ok) continue;
      float v[8];
      OutVec<float>::load(red + rr * LDW + 8 * cg, v);
#pragma unroll
      for (int q = 1; q < G; ++q) {
        float w[8];
        OutVec<float>::load(red + (q * ROWS + rr) * LDW + 8 * cg, w);
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] += w[c];
      }
      if (partial) {
        OutVec<float>::store(g.partial + ((size_t)split * g.M + row) * g.N + col, v);
        continue;
      }
      const size_t o = (size_t)row * ldc + col;
      if constexpr (std::is_same<T, TC>::value) {
        if (bias) {
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] += bv[c];
        }
        if (g.act == 1) {
          OutVec<T>::store(static_cast<T*>(g.aux_out) + o, v);   // GELU is applied to the stored value
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] = gelu_t<T>(to_f32(from_f32<T>(v[c])));
        } else if (g.act == 3) {
          float dv[8];
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] = gelu_with_grad_t<T>(v[c], dv[c]);
          OutVec<T>::store(static_cast<T*>(g.aux_out) + o, dv);
        } else if (g.act == 5) {
          float dv;
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] = gelu_with_grad_t<T>(v[c], dv);
        } else if (want_aux) {
          float u[8];
          raw8_unpack(rin[it], u);
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] *= g.act == 2 ? gelu_grad_t<T>(u[c]) : u[c];
        }
        if (resid) {
          float rv[8];
          raw8_unpack(want_aux ? raw8_load(resid + o) : rin[it], rv);
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] += rv[c];
        }
      }
      OutVec<TC>::store(static_cast<TC*>(g.C) + o, v);
#pragma unroll
      for (int c = 0; c < 8; ++c) cs[c] += v[c];
    }
  };
  pass(std::integral_constant<int, 0>{}, std::integral_constant<int, IC>{});
  if constexpr (TM > IC) pass(std::integral_constant<int, IC>{}, std::integral_constant<int, TM - IC>{});
  if (g.colsum_partial) {   // one row of column sums per tile: lanes with the same columns, then the waves in order
#pragma unroll
    for (int m = CG; m < WAVE; m <<= 1)
#pragma unroll
      for (int c = 0; c < 8; ++c) cs[c] += __shfl_xor(cs[c], m, WAVE);
    __syncthreads();
    if (lane < CG) OutVec<float>::store(red + wave * BN + 8 * lane, cs);
    __syncthreads();
    if (tid < CG && col_ok) {
      float s[8];
      OutVec<float>::load(red + 8 * tid, s);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        float x[8];
        OutVec<float>::load(red + w * BN + 8 * tid, x);
#pragma unroll
        for (int c = 0; c < 8; ++c) s[c] += x[c];
      }
      OutVec<float>::store(g.colsum_partial + (size_t)tile_m * g.N + col, s);
    }
  }
}

}  // namespace dipaco

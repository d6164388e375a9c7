// fp32 products on the bf16 matrix cores (three bf16 parts of every number, six part products: split_tile.h), all three operand
// layouts of the path step, any M, N, K that launch_gemm accepts: the fp32 products of many tiles.
//
// A workgroup is four waves of 64 x 64 outputs on a 128 x 128 tile, or, for one round of smaller tiles, eight on a 64 x 128 tile: four groups
// of two along K, whose sums meet in the epilogue (4000 x 512 x 2048 in 250 workgroups 71 - 80 us on the fp32 instruction, 65 here; the
// groups split and multiply in step, and LDS serves 221 KB a stage).  A wave loads its share of the next 32 of K into registers while it
// multiplies; then the shares are taken apart, each number once per workgroup, into one stage of LDS.  Two workgroups share a compute
// unit: one splits and stores under the other's MFMAs, which go first (wave priority: 4096^3 678 -> 640 us).
// Bound by the MFMAs and the power they draw: 4096^3 takes 504 us without loads and splitting, 640 with, 950 on the fp32 instruction
// (16384 x 4096 x 1024 990 -> 690, 4000 x 8192 x 512 265 -> 185); error against 64 bits 2.2e-7 | 8.1e-7 there (K = 4096), 9e-8 | 2.9e-7 at 512.
// Left out, measured: eight waves on 256 x 128 with two stages and the splitting dealt over the MFMAs (630 us, and a workgroup's ends uncovered:
// 4000 x 2048 x 512 59 us against 55), tiles split by the waves that read them (VALU: 770), 64 x 64 and 64 x 128 tiles on
// four waves (level with the fp32 instruction: 4000 x 512 x 2048 65 - 72 us against 75).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "gemm_fit_epilogue.h"
#include "kernels.h"
#include "split_tile.h"

namespace dipaco {

namespace {

constexpr int SP_T = 4;   // 16-row blocks of a wave's 64 rows and columns

// G groups of WM x WN waves; a group takes its own 32 of a stage's 32 G of K
template <int WM, int WN, int G> struct SplitGemm {
  static constexpr int BM = 64 * WM, BN = 64 * WN, BK = 32 * G, THREADS = 64 * WM * WN * G;
  static constexpr int UA = 2 / WN, UB = 2 / WM;   // 32-row units of each operand that a wave stages
  static constexpr int PLANE_A = BM * SPLIT_ROW, PLANE_B = BN * SPLIT_ROW;
  static constexpr int GROUP = 3 * (PLANE_A + PLANE_B);   // planes of A, planes of B
  static constexpr int EPI_ROWS = G == 1 ? 2 : 4;         // blocks of an epilogue pass
  static constexpr int LDS = G * GROUP;
  static_assert(fit_epilogue_bytes(EPI_ROWS, SP_T, WM, WN, G) <= LDS && LDS * (512 / THREADS) <= 160 * 1024, "two waves a SIMD");
};

// The workgroup's sums that the parts cannot give, on v_mfma_f32_16x16x4_f32.  Where the operands' largest number (NaN aside) is small enough
// for every product and sum to be finite, a sum that is not comes of a NaN operand and stays.  tiny: numbers below SPLIT_LEAST, each of
// which errs by up to 2^-134 in its parts; sums of up to `floor` could show that in their 24 bits.
// 2048^3 146 us: 175 with all sums NaN or small numbers that no sum depends on, 350 - 530 with an infinity in every tile (a serial chain
// for each sum: 17 - 33 ms).
// red: LDS of as many floats as waves
template <bool A_KC, bool B_KC, int WM, int WN, int G>
__device__ __forceinline__ void split_again(const GemmDev& g, f32x4 (&acc)[SP_T][SP_T], float* red, int tid, int grp, int wm, int wn, int m0, int n0,
                                            int k_begin, int k_end, bool tiny) {
  using P = SplitGemm<WM, WN, G>;
  constexpr int NW = WM * WN * G;
  const int lane = tid & 63, r = lane & 15, kg = lane >> 4, depth = k_end - k_begin;
  const float* const A = static_cast<const float*>(g.A);
  const float* const B = static_cast<const float*>(g.B);
  float top = 0.f;
  auto scan = [&](auto KCc, const float* p, long ld, int row0, int rows) {   // rows and depth are multiples of 4 along the contiguous index
    constexpr bool KC = decltype(KCc)::value;
    const int inner = (KC ? depth : rows) / 4, outer = KC ? rows : depth;
    const float* const base = p + (KC ? row0 * ld + k_begin : k_begin * ld + row0);
    constexpr int STEP = 64 * NW / 32, AHEAD = 8;
    for (int i0 = 0; i0 < inner; i0 += 32)
      for (int o0 = 0; o0 < outer; o0 += AHEAD * STEP) {
        float4 x[AHEAD];   // what lies beyond the operand reads its last numbers
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
          x[u] = *reinterpret_cast<const float4*>(base + min(o0 + STEP * u + tid / 32, outer - 1) * ld + 4 * min(i0 + tid % 32, inner - 1));
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) top = fmaxf(fmaxf(fmaxf(top, fabsf(x[u].x)), fmaxf(fabsf(x[u].y), fabsf(x[u].z))), fabsf(x[u].w));
      }
  };
  scan(std::bool_constant<A_KC>{}, A, g.lda, m0, min(P::BM, g.M - m0));
  scan(std::bool_constant<B_KC>{}, B, g.ldb, n0, min(P::BN, g.N - n0));
  top = wave_max(top);
  if (lane == 0) red[tid >> 6] = top;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) top = fmaxf(top, red[w]);
  if (!tiny && top < 281474976710656.f) return;   // 2^48: products below 2^96, sums of 2^31 of them below 2^127
  const float floor = tiny ? top * (float)depth * 0x1p-109f : 0.f;
  auto holds = [&](float v) { return fabsf(v) >= floor && fabsf(v) < INFINITY; };
  bool all_hold = true;
#pragma unroll
  for (int i = 0; i < SP_T; ++i)
#pragma unroll
    for (int j = 0; j < SP_T; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) all_hold &= holds(acc[i][j][e]);
  if (__all(all_hold)) return;   // the wave's own sums: no barrier follows here
  auto load = [&](auto KCc, const float* p, long ld, int row, int k, float (&v)[4]) {   // K k .. k + 3 of a row; beyond k_end: zero
    if constexpr (decltype(KCc)::value) {
      const float4 x = *reinterpret_cast<const float4*>(p + row * ld + min(k, k_end - 4));
      const bool in = k < k_end;
      v[0] = in ? x.x : 0.f; v[1] = in ? x.y : 0.f; v[2] = in ? x.z : 0.f; v[3] = in ? x.w : 0.f;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float x = p[min(k + q, k_end - 1) * ld + row];
        v[q] = k + q < k_end ? x : 0.f;
      }
    }
  };
#pragma unroll
  for (int i = 0; i < SP_T; i += 2) {   // two blocks of 16 rows at a time
    f32x4 t[2][2][SP_T];   // every second 16 of K each, as in the fitted tile: a chain half as long errs less
    int row[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      row[u] = min(m0 + 64 * wm + 16 * (i + u) + r, g.M - 1);
#pragma unroll
      for (int j = 0; j < SP_T; ++j) t[0][u][j] = t[1][u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int k0 = k_begin + 32 * grp; k0 < k_end; k0 += P::BK)   // the group's 32 of every stage
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float a[2][4], b[SP_T][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) load(std::bool_constant<A_KC>{}, A, g.lda, row[u], k0 + 16 * h + 4 * kg, a[u]);
#pragma unroll
        for (int j = 0; j < SP_T; ++j) load(std::bool_constant<B_KC>{}, B, g.ldb, min(n0 + 64 * wn + 16 * j + r, g.N - 1), k0 + 16 * h + 4 * kg, b[j]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < SP_T; ++j) t[h][u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][q], b[j][q], t[h][u][j], 0, 0, 0);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < SP_T; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!holds(acc[i + u][j][e])) acc[i + u][j][e] = t[0][u][j][e] + t[1][u][j][e];
  }
}

template <bool A_KC, bool B_KC, int WM, int WN, int G>
__global__ void __launch_bounds__(64 * WM * WN * G, 2) gemm_split_kernel(const GemmDev g) {
  using P = SplitGemm<WM, WN, G>;
  constexpr int UA = P::UA, UB = P::UB, BK = P::BK;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave_all / (WM * WN), wave = wave_all % (WM * WN), wm = wave / WN, wn = wave % WN;

  int split, tile_m, tile_n;
  if (g.splits > 1) {   // each XCD gets a contiguous, slice-major range
    const int tiles = g.tiles_m * g.tiles_n, v = xcd_contiguous(blockIdx.x, tiles * g.splits);
    split = v / tiles;
    tile_m = (v - split * tiles) % g.tiles_m;
    tile_n = (v - split * tiles) / g.tiles_m;
  } else {
    gemm_tile_of_block(g, blockIdx.x, split, tile_m, tile_n);
  }
  const int m0 = tile_m * P::BM, n0 = tile_n * P::BN;
  const int k_begin = split * g.k_per_split, k_end = min(g.K, k_begin + g.k_per_split);
  const int nkt = (k_end - k_begin + BK - 1) / BK;
  const int k_grp = k_end - k_begin - 32 * grp;   // K left to the group at stage 0

  // ---- staging: a wave loads and splits UA and UB units of 32 rows of the group's operand tiles ----
  using UnitA = SplitUnit<A_KC>;
  using UnitB = SplitUnit<B_KC>;
  const long kb = k_begin + 32 * grp;
  const char* base_a = static_cast<const char*>(g.A) + (A_KC ? (long)m0 * g.lda + kb : kb * g.lda + m0) * 4;
  const char* base_b = static_cast<const char*>(g.B) + (B_KC ? (long)n0 * g.ldb + kb : kb * g.ldb + n0) * 4;
  const long adv_a = (A_KC ? (long)BK : BK * g.lda) * 4, adv_b = (B_KC ? (long)BK : BK * g.ldb) * 4;
  UnitA sa[UA];
  UnitB sb[UB];
  uint32_t off_a[UA][4], off_b[UB][4];
  // byte offsets relative to the operands' bases at the group's first K of a stage; klim: K left there
  auto offsets = [&](int klim) {
    auto offset = [&](auto KCc, int unit, int j, long ld, int left) {
      using Unit = SplitUnit<decltype(KCc)::value>;
      const int row = 32 * unit + Unit::row(lane, j), k = Unit::k(lane, j);
      if (decltype(KCc)::value) return (uint32_t)(((long)min(row, left - 1) * ld + min(k, klim - 4)) * 4);
      return (uint32_t)(((long)min(k, klim - 1) * ld + min(row, left - 4)) * 4);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int u = 0; u < UA; ++u) off_a[u][j] = offset(std::bool_constant<A_KC>{}, UA * wave + u, j, g.lda, g.M - m0);
#pragma unroll
      for (int u = 0; u < UB; ++u) off_b[u][j] = offset(std::bool_constant<B_KC>{}, UB * wave + u, j, g.ldb, g.N - n0);
    }
  };
  auto load = [&](int kt) {   // stage kt, if the group has one; stages are requested in order
    const int klim = k_grp - kt * BK;
    if (klim <= 0) return;
    if (klim < 32) offsets(klim);   // the last one, where the range ends inside it
#pragma unroll
    for (int u = 0; u < UA; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) sa[u].load(base_a, off_a[u][j], j);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) sb[u].load(base_b, off_b[u][j], j);
    base_a += adv_a;
    base_b += adv_b;
  };
  char* const stage = smem + grp * P::GROUP;
  int store_a[4], store_b[4];   // of the wave's first units; the next ones lie 32 rows on
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    store_a[q] = 32 * SPLIT_ROW * UA * wave + UnitA::store_offset(lane, q);
    store_b[q] = 3 * P::PLANE_A + 32 * SPLIT_ROW * UB * wave + UnitB::store_offset(lane, q);
  }
  float least = INFINITY;   // |x| of a stage's numbers
  bool tiny = false;        // some lie below SPLIT_LEAST and are not zero
  auto store = [&](int kt) {
    const int klim = k_grp - kt * BK;
    if (klim < 32) {   // K beyond the range counts as zero
#pragma unroll
      for (int u = 0; u < UA; ++u) sa[u].cut(lane, klim);
#pragma unroll
      for (int u = 0; u < UB; ++u) sb[u].cut(lane, klim);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int u = 0; u < UA; ++u) sa[u].least(least, q);
#pragma unroll
      for (int u = 0; u < UB; ++u) sb[u].least(least, q);
    }
    if (__any(least < SPLIT_LEAST)) {
      least = INFINITY;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int u = 0; u < UA; ++u) tiny |= sa[u].tiny(q);
#pragma unroll
        for (int u = 0; u < UB; ++u) tiny |= sb[u].tiny(q);
      }
    }
#pragma unroll
    for (int u = 0; u < UA; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) sa[u].template store<P::PLANE_A>(stage + store_a[q] + 32 * SPLIT_ROW * u, q);
#pragma unroll
    for (int u = 0; u < UB; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) sb[u].template store<P::PLANE_B>(stage + store_b[q] + 32 * SPLIT_ROW * u, q);
  };

  f32x4 acc[SP_T][SP_T];
#pragma unroll
  for (int i = 0; i < SP_T; ++i)
#pragma unroll
    for (int j = 0; j < SP_T; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  const SplitFragments frag(lane);
  const char* const pa = stage + wm * 64 * SPLIT_ROW;
  const char* const pb = stage + 3 * P::PLANE_A + wn * 64 * SPLIT_ROW;

  offsets(1 << 30);
  load(0);
  for (int kt = 0; kt < nkt; ++kt) {
    store(kt);
    load(kt + 1);
    __syncthreads();
    __builtin_amdgcn_s_setprio(1);
    split_multiply<SP_T, SP_T, P::PLANE_A, P::PLANE_B>(acc, pa, pb, frag);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  }

  // What the parts do not carry (split_tile.h) is looked for once the sums are there: infinities and overflow where a sum is not
  // finite, and numbers below SPLIT_LEAST.  Such sums are taken again on the fp32 instruction.
  float* const red = reinterpret_cast<float*>(smem);
  {
    float finite = 0.f;   // NaN where a sum is not
#pragma unroll
    for (int i = 0; i < SP_T; ++i)
#pragma unroll
      for (int j = 0; j < SP_T; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) finite = __builtin_fmaf(acc[i][j][e], 0.f, finite);
    const bool any_tiny = __any(tiny), any = __any(finite != 0.f);   // votes of all lanes: outside the branch
    if (lane == 0) red[wave_all] = any_tiny ? 2.f : any ? 1.f : 0.f;
    __syncthreads();
    float seen = 0.f;
#pragma unroll
    for (int w = 0; w < WM * WN * G; ++w) seen = fmaxf(seen, red[w]);
    if (seen != 0.f)   // uniform
      split_again<A_KC, B_KC, WM, WN, G>(g, acc, red + WM * WN * G, tid, grp, wm, wn, m0, n0, k_begin, k_end, seen == 2.f);
  }
  fit_epilogue<float, float, SP_T, SP_T, WM, WN, G, P::EPI_ROWS>(g, acc, red, tid, grp, wm, wn, m0, n0, tile_m, split);
}

template <bool A_KC, bool B_KC, int WM, int WN, int G> dipaco_status run_split(const GemmArgs& a, hipStream_t s) {
  using P = SplitGemm<WM, WN, G>;
  auto kern = gemm_split_kernel<A_KC, B_KC, WM, WN, G>;
  static std::atomic<unsigned long long> lds_set{0};   // per instantiation
  if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), P::LDS, lds_set)) return e;
  GemmDev g;
  g.A = a.A; g.B = a.B; g.C = a.C; g.M = a.M; g.N = a.N; g.K = a.K;
  g.lda = a.lda; g.ldb = a.ldb; g.ldc = a.ldc;
  g.bias = a.bias; g.resid = a.resid; g.aux_out = a.aux_out; g.aux_in = a.aux_in; g.act = a.act;
  g.partial = a.partial;
  g.tiles_m = (a.M + P::BM - 1) / P::BM;
  g.tiles_n = (a.N + P::BN - 1) / P::BN;
  const int steps = (a.K + P::BK - 1) / P::BK, want = std::max(1, std::min(a.splits, steps));
  g.k_per_split = (steps + want - 1) / want * P::BK;
  g.splits = (a.K + g.k_per_split - 1) / g.k_per_split;
  const long blocks = (long)g.tiles_m * g.tiles_n * g.splits;
  if (!launch_fits(blocks, P::THREADS)) return fail(DIPACO_ESHAPE, "gemm: too many tiles");
  g.colsum_partial = a.colsum ? a.colsum_partial : nullptr;
  kern<<<(unsigned)blocks, P::THREADS, P::LDS, s>>>(g);
  DIPACO_LAUNCH_CHECK();
  if (g.splits > 1) return launch_splitk_reduce(a.partial, static_cast<float*>(a.C), a.M, a.N, a.ldc, g.splits, s);
  if (a.colsum) return launch_sum_rows(a.colsum_partial, a.colsum, g.tiles_m, a.N, s, a.sum_batch);
  return DIPACO_OK;
}

}  // namespace

template <bool A_KC, bool B_KC> dipaco_status run_split_shape(const GemmArgs& a, int rows, hipStream_t s) {
  if (rows == 64) return run_split<A_KC, B_KC, 1, 2, 4>(a, s);
  return run_split<A_KC, B_KC, 2, 2, 1>(a, s);
}
dipaco_status launch_gemm_split(const GemmArgs& a, int rows, hipStream_t s) {
  if (a.out_f32) return run_split_shape<false, false>(a, rows, s);
  if (!a.trans_b) return run_split_shape<true, false>(a, rows, s);
  return run_split_shape<true, true>(a, rows, s);
}

}  // namespace dipaco

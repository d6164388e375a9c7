// fp32 products on the bf16 matrix cores (three bf16 parts of every number, six part products: split_tile.h), all three operand
// layouts of the path step, any M, N, K that launch_gemm accepts: the fp32 products of many tiles.
//
// A workgroup is four waves of 64 x 64 outputs on a 128 x 128 tile.  A wave loads its share of the next 32 of K into registers while it
// multiplies; then the shares are taken apart, each number once per workgroup, into one stage of LDS.  Two workgroups share a compute
// unit: one splits and stores under the other's MFMAs, which go first (wave priority: 4096^3 678 -> 640 us).
// Bound by the MFMAs and the power they draw: 4096^3 takes 504 us without loads and splitting, 640 with, 950 on the fp32 instruction
// (16384 x 4096 x 1024 990 -> 690, 4000 x 8192 x 512 265 -> 185); error against 64 bits 2.2e-7 | 8.1e-7 there (K = 4096), 9e-8 | 2.9e-7 at 512.
// Left out, measured: eight waves on 256 x 128 with two stages and the splitting dealt over the MFMAs (630 us, and a workgroup's ends uncovered:
// 4000 x 2048 x 512 59 us against 55), tiles split by the waves that read them (VALU: 770), 64 x 64 and 64 x 128 tiles (level with the
// fp32 instruction: 4000 x 512 x 2048 65 - 72 us against 75).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "gemm_fit_epilogue.h"
#include "kernels.h"
#include "split_tile.h"

namespace dipaco {

namespace {

constexpr int SP_TILE = 128, SP_T = 4;   // tile side; 16-row blocks of a wave's 64 rows and columns
constexpr int SP_PLANE = SP_TILE * SPLIT_ROW;
constexpr int SP_EPI_ROWS = 2;           // blocks of an epilogue pass
constexpr int SP_LDS = 6 * SP_PLANE;     // planes of A, planes of B
static_assert(fit_epilogue_bytes(SP_EPI_ROWS, SP_T, 2, 2, 1) <= SP_LDS && 2 * SP_LDS <= 160 * 1024, "two workgroups on a compute unit");

template <bool A_KC, bool B_KC> __global__ void __launch_bounds__(256, 2) gemm_split_kernel(const GemmDev g) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  int split, tile_m, tile_n;
  if (g.splits > 1) {   // each XCD gets a contiguous, slice-major range
    const int tiles = g.tiles_m * g.tiles_n, v = xcd_contiguous(blockIdx.x, tiles * g.splits);
    split = v / tiles;
    tile_m = (v - split * tiles) % g.tiles_m;
    tile_n = (v - split * tiles) / g.tiles_m;
  } else {
    gemm_tile_of_block(g, blockIdx.x, split, tile_m, tile_n);
  }
  const int m0 = tile_m * SP_TILE, n0 = tile_n * SP_TILE;
  const int k_begin = split * g.k_per_split, k_end = min(g.K, k_begin + g.k_per_split);
  const int nkt = (k_end - k_begin + 31) / 32;

  // ---- staging: wave w loads and splits rows 32 w .. 32 w + 31 of both operand tiles ----
  using UnitA = SplitUnit<A_KC>;
  using UnitB = SplitUnit<B_KC>;
  const char* base_a = static_cast<const char*>(g.A) + (A_KC ? (long)m0 * g.lda + k_begin : (long)k_begin * g.lda + m0) * 4;
  const char* base_b = static_cast<const char*>(g.B) + (B_KC ? (long)n0 * g.ldb + k_begin : (long)k_begin * g.ldb + n0) * 4;
  const long adv_a = (A_KC ? 32L : 32 * g.lda) * 4, adv_b = (B_KC ? 32L : 32 * g.ldb) * 4;
  UnitA sa;
  UnitB sb;
  uint32_t off_a[4], off_b[4];
  // byte offsets relative to the operands' bases at the stage's first K; klim: K left there
  auto offsets = [&](int klim) {
    auto offset = [&](auto KCc, int j, long ld, int left) {
      using Unit = SplitUnit<decltype(KCc)::value>;
      const int row = 32 * wave + Unit::row(lane, j), k = Unit::k(lane, j);
      if (decltype(KCc)::value) return (uint32_t)(((long)min(row, left - 1) * ld + min(k, klim - 4)) * 4);
      return (uint32_t)(((long)min(k, klim - 1) * ld + min(row, left - 4)) * 4);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      off_a[j] = offset(std::bool_constant<A_KC>{}, j, g.lda, g.M - m0);
      off_b[j] = offset(std::bool_constant<B_KC>{}, j, g.ldb, g.N - n0);
    }
  };
  auto load = [&](int kt) {   // stage kt, if it exists; stages are requested in order
    const int klim = k_end - k_begin - kt * 32;
    if (klim <= 0) return;
    if (klim < 32) offsets(klim);   // the last one, where the range ends inside it
#pragma unroll
    for (int j = 0; j < 4; ++j) sa.load(base_a, off_a[j], j);
#pragma unroll
    for (int j = 0; j < 4; ++j) sb.load(base_b, off_b[j], j);
    base_a += adv_a;
    base_b += adv_b;
  };
  int store_a[4], store_b[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    store_a[q] = 32 * SPLIT_ROW * wave + UnitA::store_offset(lane, q);
    store_b[q] = 3 * SP_PLANE + 32 * SPLIT_ROW * wave + UnitB::store_offset(lane, q);
  }
  auto store = [&](int kt) {
    const int klim = k_end - k_begin - kt * 32;
    if (klim < 32) {   // K beyond the range counts as zero
      sa.cut(lane, klim);
      sb.cut(lane, klim);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) sa.template store<SP_PLANE>(smem + store_a[q], q);
#pragma unroll
    for (int q = 0; q < 4; ++q) sb.template store<SP_PLANE>(smem + store_b[q], q);
  };

  f32x4 acc[SP_T][SP_T];
#pragma unroll
  for (int i = 0; i < SP_T; ++i)
#pragma unroll
    for (int j = 0; j < SP_T; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  const SplitFragments frag(lane);
  const char* const pa = smem + wm * 64 * SPLIT_ROW;
  const char* const pb = smem + 3 * SP_PLANE + wn * 64 * SPLIT_ROW;

  offsets(1 << 30);
  load(0);
  for (int kt = 0; kt < nkt; ++kt) {
    store(kt);
    load(kt + 1);
    __syncthreads();
    __builtin_amdgcn_s_setprio(1);
    split_multiply<SP_T, SP_T, SP_PLANE, SP_PLANE>(acc, pa, pb, frag);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  }

  // An infinity among the operands leaves NaN here where fp32 has an infinity: sums that are not finite are taken again
  auto fix = [&](float (&v)[8], int row, int col) {
    const float *a = static_cast<const float*>(g.A), *b = static_cast<const float*>(g.B);
#pragma unroll 1
    for (int c = 0; c < 8; ++c) {
      if (__builtin_isfinite(v[c])) continue;
      float s = 0.f;
      for (long k = k_begin; k < k_end; ++k)
        s = __builtin_fmaf(A_KC ? a[row * g.lda + k] : a[k * g.lda + row], B_KC ? b[(col + c) * g.ldb + k] : b[k * g.ldb + col + c], s);
      v[c] = s;
    }
  };
  fit_epilogue<float, float, SP_T, SP_T, 2, 2, 1, SP_EPI_ROWS>(g, acc, reinterpret_cast<float*>(smem), tid, 0, wm, wn, m0, n0, tile_m,
                                                                split, fix);
}

template <bool A_KC, bool B_KC> dipaco_status run_split(const GemmArgs& a, hipStream_t s) {
  auto kern = gemm_split_kernel<A_KC, B_KC>;
  static std::atomic<unsigned long long> lds_set{0};   // per instantiation
  if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), SP_LDS, lds_set)) return e;
  GemmDev g;
  g.A = a.A; g.B = a.B; g.C = a.C; g.M = a.M; g.N = a.N; g.K = a.K;
  g.lda = a.lda; g.ldb = a.ldb; g.ldc = a.ldc;
  g.bias = a.bias; g.resid = a.resid; g.aux_out = a.aux_out; g.aux_in = a.aux_in; g.act = a.act;
  g.partial = a.partial;
  g.tiles_m = (a.M + SP_TILE - 1) / SP_TILE;
  g.tiles_n = (a.N + SP_TILE - 1) / SP_TILE;
  const int steps = (a.K + 31) / 32, want = std::max(1, std::min(a.splits, steps));
  g.k_per_split = (steps + want - 1) / want * 32;
  g.splits = (a.K + g.k_per_split - 1) / g.k_per_split;
  const long blocks = (long)g.tiles_m * g.tiles_n * g.splits;
  if (!launch_fits(blocks, 256)) return fail(DIPACO_ESHAPE, "gemm: too many tiles");
  g.colsum_partial = a.colsum ? a.colsum_partial : nullptr;
  kern<<<(unsigned)blocks, 256, SP_LDS, s>>>(g);
  DIPACO_LAUNCH_CHECK();
  if (g.splits > 1) return launch_splitk_reduce(a.partial, static_cast<float*>(a.C), a.M, a.N, a.ldc, g.splits, s);
  if (a.colsum) return launch_sum_rows(a.colsum_partial, a.colsum, g.tiles_m, a.N, s, a.sum_batch);
  return DIPACO_OK;
}

}  // namespace

dipaco_status launch_gemm_split(const GemmArgs& a, hipStream_t s) {
  if (a.out_f32) return run_split<false, false>(a, s);
  if (!a.trans_b) return run_split<true, false>(a, s);
  return run_split<true, true>(a, s);
}

}  // namespace dipaco

// The GEMM entry: argument checks, the choice between the matrix-core kernels and their K splits, and the sum of
// split-K partial planes.
//   gemm_dlds.hip   bf16, 256 x 256 tiles (and oblong ones), uneven split-K: products that fill the chip with such tiles
//   gemm_fit.hip    every other product: ragged contractions, everything smaller, and fp32, with tiles fitted to the grid
//   gemm_split.hip  of those, the fp32 products that are ahead in three bf16 parts (gemm_fit.hip chooses)
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

namespace dipaco {

namespace {
// C = sum of the partial planes in slice order; the number of K slices may depend on where the element lies:
// n_slices[(row >= row_edge) + 2 * (col >= col_edge)]
__global__ void __launch_bounds__(128) splitk_reduce_classes_kernel(const float* __restrict__ partial,
                                                                    float* __restrict__ C, int M, int N, long ldc,
                                                                    int row_edge, int col_edge, int s0, int s1, int s2,
                                                                    int s3) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  const size_t total = (size_t)M * N, quads = total / 4;
  const size_t stride = (size_t)gridDim.x * 128;
  // one 16-byte vector per thread in the usual launch; a plane is read once (streaming loads), the first eight
  // slices are requested together and added in slice order
  for (size_t q = (size_t)blockIdx.x * 128 + threadIdx.x; q < quads; q += stride) {
    const size_t i = 4 * q;
    const size_t row = i / N, col = i - row * N;   // N is a multiple of 8: the four elements share a row
    const bool er = (int)row >= row_edge, ec = (int)col >= col_edge;
    const int n = er ? (ec ? s3 : s1) : (ec ? s2 : s0);
    f32x4_t v[8];
#pragma unroll
    for (int z = 0; z < 8; ++z)
      if (z < n) v[z] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(partial + (size_t)z * total + i));
    f32x4_t acc = v[0];
#pragma unroll
    for (int z = 1; z < 8; ++z)
      if (z < n) acc += v[z];
    for (int z = 8; z < n; ++z) acc += __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(partial + (size_t)z * total + i));
    *reinterpret_cast<f32x4_t*>(C + row * ldc + col) = acc;
  }
}
}  // namespace

dipaco_status launch_splitk_reduce_classes(const float* partial, float* C, int M, int N, long ldc, int row_edge,
                                           int col_edge, const int (&n_slices)[4], hipStream_t s) {
  if (N % 8 || ldc % 4 || col_edge % 4) return fail(DIPACO_ESHAPE, "split-K reduce: N, ldc, col_edge must be multiples of 8, 4, 4");
  const size_t quads = (size_t)M * N / 4;
  const unsigned rb = (unsigned)std::min<size_t>((quads + 127) / 128, 0x7fffffffu);
  splitk_reduce_classes_kernel<<<rb, 128, 0, s>>>(partial, C, M, N, ldc, row_edge, col_edge, n_slices[0], n_slices[1],
                                                  n_slices[2], n_slices[3]);
  DIPACO_LAUNCH_CHECK();
  return DIPACO_OK;
}

dipaco_status launch_splitk_reduce(const float* partial, float* C, int M, int N, long ldc, int splits, hipStream_t s) {
  const int n_slices[4] = {splits, splits, splits, splits};
  return launch_splitk_reduce_classes(partial, C, M, N, ldc, M, N, n_slices, s);
}

// test / tuning hook (dipaco_k_set_gemm_tile), not a per-call setting: 0 = the rules below, FORCED_FIT / FORCED_DLDS = that
// kernel wherever it takes the shape
constexpr int FORCED_FIT = 1, FORCED_DLDS = 2;
static std::atomic<int> g_forced_kernel{0};

void set_gemm_tile(int t) {
  const bool fit = (t >= 1 && t <= 4) || t == 14;
  set_gemm_fit_shape(!fit ? 0 : t == 14 ? 5 : t);
  g_forced_kernel = fit ? FORCED_FIT : t ? FORCED_DLDS : 0;
  set_gemm_dlds_shape(!fit && t > 5 ? t - 5 : 0);
}

size_t gemm_colsum_partial_floats(int M, int N) { return (size_t)((M + 31) / 32) * N; }

// microseconds to add `splits` fp32 planes: measured 4 us at least, 5.6-6 TB/s
static double reduce_cost(int M, int N, int splits) {
  return splits > 1 ? 2.5 + (splits + 1) * (double)M * N * (4.0 / 6.5e6) : 0.0;
}
static double plane_cost(int M, int N, int splits) { return splits > 1 ? splits * (double)M * N * (4.0 / 6.0e6) : 0.0; }

// Most slices a weight gradient (K = tokens) is cut into: a slice keeps at least 256 of K, and a small output under a
// very long fp32 contraction (the router's 256 x 768 gradient over 2^20 documents) may still fill the chip.
constexpr int GEMM_SLICE_CAP_F32 = 128;
struct SplitPlan { int splits; bool dlds; double us; };

// The cheaper of the two kernels for C[M, N] = X^T dY over K tokens, by the times of gemm_fit_cost and of the
// direct-to-LDS kernel (8 us + 23 us per 1000 of the longest workgroup's K).  Measured in bf16, product + reduction: 1024 x 4096
// over 4096 tokens 38 us unsplit here against 42 + 15 there, 896 x 896 over 8192 24 + 5 / 27 + 9; over 32768 tokens
// 896 x 2688 171 + 12 / 155 + 10, 1024 x 4096 294 / 212 + 14: beyond 16384 tokens the tiles of a one-round launch drift
// apart and re-read their panels, and the direct-to-LDS plan is taken wherever there is one.
static SplitPlan plan_splits(int M, int N, int K, bool bf16_operands, bool dlds_allowed, int limit = GEMM_SLICE_CAP_F32) {
  const int cap = std::max(1, std::min({bf16_operands ? GEMM_SLICE_CAP : GEMM_SLICE_CAP_F32, K / 256, limit}));
  SplitPlan best{1, false, 1e30};
  double cost = 1e30;
  const GemmFitTiles tiles = gemm_fit_tiles(M, N, bf16_operands, false);
  for (int s = 1; s <= cap; ++s) {
    const double planes = plane_cost(M, N, s) + reduce_cost(M, N, s);
    if (planes > cost) break;   // grows with s
    const double c = gemm_fit_cost(tiles, (K + s - 1) / s, s) + planes;
    if (c < cost) { cost = best.us = c; best.splits = s; }
  }
  if (bf16_operands && dlds_allowed && K % 32 == 0) {
    double length = 0.0;
    int s = gemm_dlds_plan_slices(M, N, K, cap, false, &length);
    const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
    if (!s) { s = 1; length = (double)((tiles + 255) / 256) * K; }
    const bool fills = tiles * s >= 160;
    const double c = 8.0 + 0.023 * length + plane_cost(M, N, s) + reduce_cost(M, N, s);
    if (fills && (c < cost || K > 16384)) best = SplitPlan{s, true, c};
  }
  return best;
}

int gemm_plan_splits(int M, int N, int K, bool bf16_operands, int limit) {
  if (bf16_operands && g_forced_kernel == FORCED_DLDS) {
    const int s = gemm_dlds_plan_slices(M, N, K, std::max(1, std::min({GEMM_SLICE_CAP, K / 256, limit})), false, nullptr);
    if (s) return s;
  }
  return plan_splits(M, N, K, bf16_operands, g_forced_kernel != FORCED_FIT, limit).splits;
}

// The plan's slices go up and down with K, but a workspace that serves K tokens has to serve fewer as well.  So the limit is the
// largest plan, over all tile settings, at the powers of two from 512 (below, nothing is cut) to the one at or above K, and at
// three quarters of each.  A plan between them that would take more is held to it (one in 10000 sizes drawn, by a slice or two).
void gemm_slice_limits(int M, int N, bool bf16_operands, int* limit, int count) {
  int most = 1;
  for (int i = 0; i < count; ++i) {
    for (int quarters = 3; i >= 9 && quarters <= 4; ++quarters) {
      const int K = (int)std::min((1LL << i) / 4 * quarters, 0x7fffffffLL);
      most = std::max(most, plan_splits(M, N, K, bf16_operands, false).splits);
      if (bf16_operands) most = std::max(most, gemm_dlds_plan_slices(M, N, K, std::min(GEMM_SLICE_CAP, K / 256), true, nullptr));
    }
    limit[i] = most;
  }
}

// bf16 products that fill most of the chip's 256 compute units with 256 x 256 tiles go to the direct-to-LDS kernel: measured
// 3000 x 3584 x 896 (168 tiles) 27.8 us against 32.6, 5700 x 2688 x 896 (253) 28.8 / 41; below, tiles fitted to the grid
// win: 3000 x 2688 x 896 (132) 27.3 / 23.8, 8192 x 896 x 3584 (128) 76.8 / 57.4, 3000 x 896 x 3584 (48) 76 / 26.
static bool want_dlds(const GemmArgs& a) {
  if (g_forced_kernel) return g_forced_kernel == FORCED_DLDS;
  if (a.out_f32) return plan_splits(a.M, a.N, a.K, true, true).dlds;
  return (long)((a.M + 255) / 256) * ((a.N + 255) / 256) >= 160;
}

// Rows of a direct-to-LDS product that its whole rounds of 256 workgroups hold, when the rows left over cost clearly less in tiles fitted
// to them than as the last, mostly empty round: 5700 x 3584 x 896 is 322 tiles of 256 x 256, two rounds, 55 us (70 with GELU and its
// derivative); the first 4608 rows (252 tiles) and then 1092 rows in 196 tiles of 160 x 128 take 49 (58); 20000 x 896 x 3584 137 -> 116,
// 5000 x 3584 x 3584 156 -> 110, 12000 x 3584 x 3584 (modelled 77 against 90) 246 -> 242.  The second launch has to be modelled a tenth below
// the round: at 118 against 123 5000 x 5000 x 4992 is level to 5 % slower (233 -> 244 with GELU), at 28.5 against 28.6 32768 x 2688 x 896 147
// -> 151.  Else, and where column sums are wanted (their partial rows are numbered by one launch's tiles), all of them.
static int dlds_rows(const GemmArgs& a) {
  const long tn = (a.N + 255) / 256, tiles = (a.M + 255) / 256 * tn, rounds = (tiles + 255) / 256;
  if (a.out_f32 || a.colsum || g_forced_kernel || rounds < 2) return a.M;
  const long rows = (rounds - 1) * 256 / tn * 256;
  if (rows < 256 || rows >= a.M) return a.M;
  const double round = 8.0 + 0.023 * a.K;
  return gemm_fit_cost(gemm_fit_tiles((int)(a.M - rows), a.N, true, true), a.K, 1) + 4.0 < 0.9 * round ? (int)rows : a.M;
}

template <typename T> static dipaco_status check_gemm(const GemmArgs& a) {
  constexpr int VEC = 16 / sizeof(T);
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return fail(DIPACO_ESHAPE, "gemm: empty operand");
  // 16-byte vectors run along the contiguous index of each operand and along the rows of C
  if ((a.trans_a ? a.M : a.K) % VEC || (a.trans_b ? a.K : a.N) % VEC || a.lda % VEC || a.ldb % VEC)
    return fail(DIPACO_ESHAPE, "gemm: contiguous extents and leading dimensions must be multiples of 16 bytes");
  if (a.ldc % 8 || a.N % 8) return fail(DIPACO_ESHAPE, "gemm: N and ldc must be multiples of 8");
  // the declared range; inside it gemm_fit.hip addresses every operand (rows too far apart for its 32-bit offsets: in 64 bits)
  const long ext_a = (a.trans_a ? 64 : (long)a.M) * a.lda + a.M, ext_b = (a.trans_b ? (long)a.N : 64) * a.ldb + a.N;
  if (ext_a >= (1L << 32) || ext_b >= (1L << 32)) return fail(DIPACO_ESHAPE, "gemm: operand above 2^32 elements");
  if (!aligned16(a.A) || !aligned16(a.B) || !aligned16(a.C) || !aligned16(a.bias) || !aligned16(a.resid) ||
      !aligned16(a.aux_in) || !aligned16(a.aux_out) || !aligned16(a.partial))
    return fail(DIPACO_EALIGN, "gemm: operand not 16-byte aligned");
  if (a.act < 0 || a.act > 5) return fail(DIPACO_EINVAL, "gemm: act must be 0..5");
  if ((a.act == 1 || a.act == 3) && !a.aux_out) return fail(DIPACO_EINVAL, "gemm: act 1 / 3 need aux_out");
  if ((a.act == 2 || a.act == 4) && !a.aux_in) return fail(DIPACO_EINVAL, "gemm: act 2 / 4 need aux_in");
  if (a.out_f32 && (a.bias || a.resid || a.act)) return fail(DIPACO_EINVAL, "gemm: fp32 output takes no epilogue");
  if (a.colsum && (!a.colsum_partial || a.splits > 1 || a.out_f32 || !aligned16(a.colsum_partial)))
    return fail(DIPACO_EINVAL, "gemm: column sums need their scratch, no split-K and an output of the operands' type");
  if (a.raw_planes) {
    if (a.splits < 2 || a.out_f32 || a.trans_a || a.trans_b || a.bias || a.resid || a.act || a.colsum || !a.partial)
      return fail(DIPACO_EINVAL, "gemm: raw planes come from a split forward product without an epilogue");
    return DIPACO_OK;
  }
  if (a.splits > 1 && (!a.out_f32 || a.bias || a.resid || a.act || !a.partial))
    return fail(DIPACO_EINVAL, "gemm: split-K needs fp32 output, a partial buffer and no epilogue");
  if (a.out_f32 && !(a.trans_a && !a.trans_b)) return fail(DIPACO_EUNSUPPORTED, "gemm: fp32 output only for A^T.B");
  if (!a.out_f32 && a.trans_a) return fail(DIPACO_EUNSUPPORTED, "gemm: operand layout not instantiated");
  return DIPACO_OK;
}

template <typename T> dipaco_status launch_gemm(const GemmArgs& a, hipStream_t s) {
  if (dipaco_status st = check_gemm<T>(a)) return st;
  if (a.raw_planes) return launch_gemm_fit<T>(a, s);
  if constexpr (std::is_same<T, bf16>::value) {
    if (want_dlds(a) && gemm_dlds_eligible(a)) {
      const int rows = dlds_rows(a);
      if (rows == a.M) return launch_gemm_dlds(a, s);
      GemmArgs first = a, rest = a;
      first.M = rows;
      rest.M = a.M - rows;
      auto below = [&](auto p, long ld) { return p ? (decltype(p))((uintptr_t)p + (size_t)rows * ld * sizeof(T)) : p; };
      rest.A = below(a.A, a.lda);
      rest.C = below(a.C, a.ldc);
      rest.resid = below(a.resid, a.ldc);
      rest.aux_in = below(a.aux_in, a.ldc);
      rest.aux_out = below(a.aux_out, a.ldc);
      if (dipaco_status st = launch_gemm_dlds(first, s)) return st;
      return launch_gemm_fit<T>(rest, s);
    }
  }
  return launch_gemm_fit<T>(a, s);
}

template <typename T> dipaco_status launch_norm_gemm(const T* x, const T* gain, const T* shift, float* mean, float* rstd, float eps, const GemmArgs& a, hipStream_t s) {
  if constexpr (std::is_same<T, float>::value) {
    if (!g_forced_kernel && gemm_norm_takes(a)) {
      GemmArgs rows = a;
      rows.A = x;
      if (dipaco_status st = check_gemm<T>(a)) return st;
      if (dipaco_status st = check_gemm<T>(rows)) return st;
      return launch_gemm_norm(rows, RowNorm{gain, shift, static_cast<float*>(const_cast<void*>(a.A)), mean, rstd, eps}, s);
    }
  }
  if (dipaco_status st = launch_layernorm_fwd<T>(x, gain, shift, static_cast<T*>(const_cast<void*>(a.A)), mean, rstd, a.M, a.K, eps, s)) return st;
  return launch_gemm<T>(a, s);
}

// K of the longest chain of sums in dW's own launch: a slice in the direct-to-LDS kernel, a group of waves' part of one in a fitted tile
static int dw_chain(const GemmArgs& dw) {
  const int splits = std::max(1, dw.splits), k = (dw.K + splits - 1) / splits;
  const int groups = want_dlds(dw) && gemm_dlds_eligible(dw) ? 1 : gemm_fit_groups(dw.M, dw.N, k, splits);
  return (k + groups - 1) / groups;
}

// dW and dX in one launch of fitted tiles (gemm_fit_pair_wide_kernel, dW uncut) where that is modelled clearly below two launches and dW's chains of
// sums are no longer than there (896 x 896 over 3000 tokens is two slices of two groups: in one launch 1.3e-7 off where it was 1.0e-7).
// Whole forward and backward passes, us, two launches -> one: 150M path, 1 x 1000 tokens 3689 -> 3204, 2 x 700 3996 -> 3452, 6 x 900 8760 ->
// 8454, 3 x 1000 5753 -> 5616, 8 x 1000 11998 -> 11696; 512 wide, 3 x 777 1565 -> 1406; level at 1024 wide, 8 x 512, and 512 wide, 12 x 700.  The price
// knows no epilogue.  The down-projection's dX, with GELU' and column sums, is 93 of the 485 us at 1 x 1000, 71 of 544 at 2 x 700, 22 - 40 of 137 at 3 x
// 1000, level at 8 x 1000, and loses 13 of 1921 at 1024 wide, 2 x 512.  With no margin a 1024-wide path of 4096 tokens, whose products are
// whole rounds, is 0.3 % behind.  Contractions above 16384 stay with the direct-to-LDS kernel (plan_splits).
static GemmWidePair pick_wide_pair(const GemmArgs& dw, const GemmArgs& dx) {
  const GemmWidePair none{0, true, 1e30};
  if (dw.K > 16384 || (dw.K + GEMM_WIDE_GROUPS - 1) / GEMM_WIDE_GROUPS > dw_chain(dw)) return none;
  GemmArgs whole = dw;
  whole.splits = 1;
  const GemmWidePair one = gemm_fit_pair_wide(whole, dx);
  const double w = plan_splits(dw.M, dw.N, dw.K, true, true, std::max(1, dw.splits)).us;
  const double rounds = (double)(((long)((dx.M + 255) / 256) * ((dx.N + 255) / 256) + 255) / 256);
  const double x = want_dlds(dx) && gemm_dlds_eligible(dx) ? 3.0 + rounds * (8.0 + 0.023 * dx.K) : gemm_fit_cost(gemm_fit_tiles(dx.M, dx.N, true, true), dx.K, 1);
  return one.us < 0.93 * (w + 1.0 + x) ? one : none;
}

template <typename T> dipaco_status launch_gemm_pair(const GemmArgs& dw, const GemmArgs& dx, hipStream_t s) {
  if (dipaco_status st = check_gemm<T>(dw)) return st;
  if (dipaco_status st = check_gemm<T>(dx)) return st;
  if (!g_forced_kernel && dw.out_f32 && dx.trans_b && !dx.out_f32 && gemm_fit_pair_takes<T>(dw, dx)) return launch_gemm_fit_pair<T>(dw, dx, s);
  if constexpr (std::is_same<T, bf16>::value) {
    if (!g_forced_kernel && dw.out_f32 && dx.trans_b && !dx.out_f32) {
      GemmArgs whole = dw;
      whole.splits = 1;
      const GemmWidePair pair = pick_wide_pair(dw, dx);
      if (pair.rows) return launch_gemm_fit_pair_wide(whole, dx, pair, s);
    }
  }
  if (dipaco_status st = launch_gemm<T>(dw, s)) return st;
  return launch_gemm<T>(dx, s);
}

void gemm_pair_plan_info(int tokens, int k_in, int n_out, int max_slices, int* out) {
  GemmArgs dw{}, dx{};
  dw.M = k_in; dw.N = n_out; dw.K = tokens; dw.lda = k_in; dw.ldb = dw.ldc = n_out; dw.trans_a = dw.out_f32 = 1;
  dw.splits = gemm_plan_splits(k_in, n_out, tokens, true, max_slices);
  dx.M = tokens; dx.N = k_in; dx.K = n_out; dx.lda = dx.ldb = n_out; dx.ldc = k_in; dx.trans_b = 1; dx.splits = 1;
  const bool small = !g_forced_kernel && gemm_fit_pair_takes<bf16>(dw, dx);
  const GemmWidePair pair = g_forced_kernel || small ? GemmWidePair{0, true, 1e30} : pick_wide_pair(dw, dx);
  out[0] = small ? 32 : pair.rows;
  out[1] = small || (pair.rows && pair.dw_first);
  out[3] = dw_chain(dw);
  out[2] = small ? out[3] : pair.rows ? (tokens + GEMM_WIDE_GROUPS - 1) / GEMM_WIDE_GROUPS : 0;
}

template dipaco_status launch_norm_gemm<float>(const float*, const float*, const float*, float*, float*, float, const GemmArgs&, hipStream_t);
template dipaco_status launch_norm_gemm<bf16>(const bf16*, const bf16*, const bf16*, float*, float*, float, const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm_pair<float>(const GemmArgs&, const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm_pair<bf16>(const GemmArgs&, const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm<float>(const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm<bf16>(const GemmArgs&, hipStream_t);

}  // namespace dipaco

// Matrix-core GEMM for every product that does not fill the chip with 256 x 256 tiles, and for ragged contractions and the fp32
// products that are not ahead in bf16 parts (gemm_split.hip): bf16 (v_mfma_f32_16x16x32_bf16) or fp32 (v_mfma_f32_16x16x4_f32),
// all three operand layouts of the path step, any M, N, K that launch_gemm accepts.
//
// What bounds these products is the number of compute units at work and the latency of a K loop, not the matrix cores.
// So the tile is fitted to the grid: its height BM is chosen among 64 .. 160 rows (BN = 128) so that the tiles make whole
// rounds over the 256 compute units (3000 x 896: 96-row tiles, 224 workgroups; 5700 x 896: 160-row tiles, 252), and a
// product of few tiles takes 32 x 64 ones.  A workgroup is eight waves in G groups along K x WM x WN over the tile:
// group g multiplies the g-th 64 bytes of K of every stage, so that two waves share a SIMD with 64 x 64 outputs each
// (fewer LDS bytes per flop than eight waves of 64 x 32), and a 32 x 64 tile walks K eight steps at a time.  The groups'
// partial sums are added in group order through LDS in front of the epilogue.
//
// Operand tiles go from global memory straight into LDS (16-byte global_load_lds, linear in the lane, swizzles applied on
// the global side) in a ring of ST stages of 64 G bytes of K:
//   * operand contiguous along K: tile row r is 64 G bytes; 16-byte chunk c at c ^ sw(r) (sw below).  A fragment is one
//     ds_read_b128: lane l holds row l % 16, K chunk l / 16 of its group's 64 bytes: 8 bf16, or 4 floats = 4 MFMAs.
//   * operand contiguous along its rows: K-row t is the tile's rows; 16-row blocks are permuted by rc_pos(block, t).  bf16
//     fragments come from two transposing ds_read_b64_tr_b16 (K-rows 8 (l / 16) + 0..3 and + 4..7), fp32 ones from four
//     ds_read_b32 (K-rows 4 (l / 16) + 0..3): the same K per lane and element as above, so any mix multiplies correctly.
// The chunk and block permutations make the lanes that the LDS serves together touch different slots of the 256-byte bank
// space (see mma_tile.h for the lane sets); the one exception is fp32 in 32-row blocks of K-rows (two lanes per bank).
//
// Loop, one barrier per stage: own loads of stage t have landed (vmcnt) and own fragments of t - 1 are in registers ->
// barrier -> the stage t - 1 occupied is refilled, the fragments of t are read, and the MFMAs of t - 1 run over both.
// K beyond the range: loads re-read the last valid K, groups beyond it skip their MFMAs, a group that straddles it zeroes
// the excess in its fragments (both operands).  Rows beyond M or N re-read the last ones and are not stored.
// A lane's byte offsets into a stage's operand tile are 32-bit; rows so far apart that a tile spans 4 GiB or more take the
// 32 x 64 tile with 64-bit addresses (FAR).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"
#include "gemm_fit_epilogue.h"
#include "kernels.h"
#include "mma_tile.h"

namespace dipaco {

namespace {

constexpr int FIT_WAVES = 8;
constexpr int FIT_STEP = 64;   // bytes of K per group and stage

typedef short fit_v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) fit_v4s* fit_lds_ptr;

// position of 16-row block blk in K-row t of a row-contiguous tile whose K-rows are R bytes (its own inverse)
template <typename T, int R> __device__ __forceinline__ int rc_pos(int blk, int t) {
  if constexpr (sizeof(T) == 2) {
    if constexpr (R >= 256) return (((blk >> 1) ^ (t & 3)) << 1) | ((blk ^ (t >> 3)) & 1);
    else if constexpr (R == 128) return blk ^ (t & 2) ^ ((t >> 3) & 1);
    else return blk ^ ((t >> 3) & 1);
  } else {
    if constexpr (R >= 256) return blk ^ ((t >> 2) & 3);
    else return blk ^ ((t >> 2) & 1);
  }
}

template <typename T, typename TC, bool A_KC, bool B_KC, int TM, int TN, int WM, int WN, int G, int ST> struct Fit {
  static_assert(WM * WN * G == FIT_WAVES && (G == 2 || G == 8), "eight waves; swizzles for rows of 128 and 512 bytes");
  static constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
  static constexpr int E = 16 / sizeof(T);                 // elements per 16-byte chunk
  static constexpr int KD = FIT_STEP / sizeof(T);          // K per group and stage
  static constexpr int BK = KD * G;                        // K per stage
  static constexpr int ROWB = FIT_STEP * G;                // bytes of a K-contiguous tile row
  static constexpr int TILE_A = BM * ROWB, TILE_B = BN * ROWB, STAGE = TILE_A + TILE_B;
  static constexpr int RA = BM * (int)sizeof(T), RB = BN * (int)sizeof(T);   // bytes of a K-row
  static constexpr int NLA = TILE_A / 1024, NL = STAGE / 1024;               // wave-level loads of a stage
  static constexpr int LPS = (NL + FIT_WAVES - 1) / FIT_WAVES;
  static constexpr int IC = TM <= 4 ? TM : 3;              // 16-row blocks per wave and epilogue pass
  static constexpr int EPI = fit_epilogue_bytes(IC, TN, WM, WN, G);
  static constexpr int LDS = ST * STAGE > EPI ? ST * STAGE : EPI;
  // Workgroups on a compute unit, two waves a SIMD each: the register budget has to leave room for both (132 registers in the
  // 64 x 128 A.B^T kernel of fp32 left one: 36311 x 3488 x 104 435 us, 338 with both)
  static constexpr int PER_CU = 2 * LDS <= 160 * 1024 ? 2 : 1;
  static_assert(A_KC || (BM & (BM - 1)) == 0, "row-contiguous tiles have power-of-two sides");
  static_assert(LDS <= 160 * 1024 && TILE_A % 1024 == 0 && STAGE % 1024 == 0 && (ST == 3 || ST == 4), "ring");
};

// chunk swizzle of a K-contiguous tile row
template <int G> __device__ __forceinline__ int kc_sw(int row) { return G == 2 ? (row >> 1) & 7 : row & 15; }

// Where lane `lane` of wave-level load jj of an operand tile reads: row (relative to the tile) and K offset (elements,
// relative to the stage) of its 16 bytes
template <typename T, bool KC, int ROWB, int R, int G>
__device__ __forceinline__ void fit_source(int jj, int lane, int& row, int& k) {
  constexpr int E = 16 / sizeof(T);
  if constexpr (KC) {
    constexpr int LPR = ROWB / 16;
    row = jj * (64 / LPR) + lane / LPR;
    k = ((lane % LPR) ^ kc_sw<G>(row)) * E;
  } else {
    const int byte = jj * 1024 + lane * 16;
    k = byte / R;
    const int in_row = byte % R, bb = 16 * (int)sizeof(T);   // bytes of a 16-row block
    row = rc_pos<T, R>(in_row / bb, k) * 16 + (in_row % bb) / (int)sizeof(T);
  }
}

// Bytes from the first to past the last byte that a stage's loads touch in one operand tile, `rows` x `depth` of K at most
// (both clamped to the operand); what a lane's offset has to hold.
inline uint64_t fit_span(bool k_contiguous, int rows, int depth, int extent, int K, long ld, int elem) {
  const uint64_t r = std::min(rows, extent), k = std::min(depth, K);
  return (k_contiguous ? (r - 1) * ld + k : (k - 1) * ld + r) * elem;
}

template <typename T, typename TC, bool A_KC, bool B_KC, int TM, int TN, int WM, int WN, int G, int ST, bool FAR>
__device__ __forceinline__ void fit_product(const GemmDev& g, int block) {
  using F = Fit<T, TC, A_KC, B_KC, TM, TN, WM, WN, G, ST>;
  constexpr int BM = F::BM, BN = F::BN, E = F::E, KD = F::KD, BK = F::BK, ROWB = F::ROWB, LPS = F::LPS;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  const int r = lane & 15, kg = lane >> 4;

  int split, tile_m, tile_n;
  if (g.splits > 1) {   // split-K: each XCD gets a contiguous, slice-major range (neighbours share operand panels in its L2)
    const int tiles = g.tiles_m * g.tiles_n, v = xcd_contiguous(block, tiles * g.splits);
    split = v / tiles;
    tile_m = (v - split * tiles) % g.tiles_m;
    tile_n = (v - split * tiles) / g.tiles_m;
  } else if (g.fast_map) {
    split = 0;
    gemm_tile_of_block_fast(g, block, tile_m, tile_n);
  } else {
    gemm_tile_of_block(g, block, split, tile_m, tile_n);
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  constexpr bool EARLY = WM * WN == 1;
  FitAhead<T> early;
  if constexpr (EARLY) early = fit_request<T, TN, TM, FIT_WAVES>(g, tid, m0, n0);
  const int k_begin = split * g.k_per_split, k_end = min(g.K, k_begin + g.k_per_split);
  const int nkt = (k_end - k_begin + BK - 1) / BK;

  // ---- loads: wave-level load i of this wave is number wave + 8 i of the stage (the last number is repeated to fill up) ----
  const char* base_a = static_cast<const char*>(g.A) + (A_KC ? (long)m0 * g.lda + k_begin : (long)k_begin * g.lda + m0) * (long)sizeof(T);
  const char* base_b = static_cast<const char*>(g.B) + (B_KC ? (long)n0 * g.ldb + k_begin : (long)k_begin * g.ldb + n0) * (long)sizeof(T);
  const long adv_a = A_KC ? ROWB : (long)BK * g.lda * (long)sizeof(T), adv_b = B_KC ? ROWB : (long)BK * g.ldb * (long)sizeof(T);
  const uint32_t smem_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + 1024 * wave);
  // byte offset of load i relative to its operand's base at the stage's first K; klim: K left in the range there
  using Off = std::conditional_t<FAR, uint64_t, uint32_t>;
  auto source = [&](int i, int klim) -> Off {
    const int j = min(wave + FIT_WAVES * i, F::NL - 1);
    int row, k;
    if (j < F::NLA) {
      fit_source<T, A_KC, ROWB, F::RA, G>(j, lane, row, k);
      if (A_KC) return (Off)(((long)min(row, g.M - 1 - m0) * g.lda + min(k, klim - E)) * (long)sizeof(T));
      return (Off)(((long)min(k, klim - 1) * g.lda + min(row, g.M - E - m0)) * (long)sizeof(T));
    }
    fit_source<T, B_KC, ROWB, F::RB, G>(j - F::NLA, lane, row, k);
    if (B_KC) return (Off)(((long)min(row, g.N - 1 - n0) * g.ldb + min(k, klim - E)) * (long)sizeof(T));
    return (Off)(((long)min(k, klim - 1) * g.ldb + min(row, g.N - E - n0)) * (long)sizeof(T));
  };
  Off off[LPS];
  uint32_t ldst[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    off[i] = source(i, 1 << 30);
    ldst[i] = smem_base + 1024 * (min(wave + FIT_WAVES * i, F::NL - 1) - wave);
  }
  // Stages are requested in order: the bases move on with them.  Which operand load i belongs to is known at compile time but
  // for the one i whose eight numbers straddle the operands.
  auto issue = [&](int i, int slot) {   // load i of the next stage, inside the range
    const bool a = FIT_WAVES * i + FIT_WAVES <= F::NLA || (FIT_WAVES * i < F::NLA && wave + FIT_WAVES * i < F::NLA);
    const uint32_t dst = __builtin_amdgcn_readfirstlane(ldst[i] + slot * F::STAGE);
    if constexpr (FAR) load16_to_lds((a ? base_a : base_b) + off[i], dst);
    else load16_to_lds_at(a ? base_a : base_b, off[i], dst);
  };
  auto issued = [&] { base_a += adv_a; base_b += adv_b; };
  auto issue_any = [&](int kt, int slot) {   // all loads of stage kt, the next one, if it exists
    if (kt >= nkt) return;
    const int klim = k_end - k_begin - kt * BK;
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      if (klim < BK) off[i] = source(i, klim);   // the last stage, where the range ends inside it: clamped K
      issue(i, slot);
    }
    issued();
  };

  // ---- fragments ----
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  uint4 fa[2][TM], fb[2][TN];
  const int koff = r * ROWB + (((4 * grp + kg) ^ kc_sw<G>(r)) << 4);   // K-contiguous tile
  // row-contiguous tile: this lane's part of 16-row block i (j) of its group's K step
  int toffa[TM], toffb[TN];
  auto rc_off = [&](int blk, auto Rc) {
    constexpr int R = decltype(Rc)::value;
    const int t = sizeof(T) == 2 ? 32 * grp + 8 * kg + (r >> 2) : 16 * grp + 4 * kg;
    return t * R + rc_pos<T, R>(blk, t) * 16 * (int)sizeof(T) + (sizeof(T) == 2 ? 8 * (r & 3) : 4 * r);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i) toffa[i] = A_KC ? (wm * TM + i) * 16 * ROWB + koff : rc_off(wm * TM + i, std::integral_constant<int, F::RA>{});
#pragma unroll
  for (int j = 0; j < TN; ++j)
    toffb[j] = F::TILE_A + (B_KC ? (wn * TN + j) * 16 * ROWB + koff : rc_off(wn * TN + j, std::integral_constant<int, F::RB>{}));
  auto rc_read = [&](const char* p, auto Rc) {
    constexpr int R = decltype(Rc)::value;
    uint4 o;
    if constexpr (sizeof(T) == 2) {
      const fit_v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((fit_lds_ptr)(uintptr_t)(uint32_t)(uintptr_t)p);
      const fit_v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((fit_lds_ptr)(uintptr_t)(uint32_t)(uintptr_t)(p + 4 * R));
      o.x = (uint16_t)lo[0] | ((uint32_t)(uint16_t)lo[1] << 16);
      o.y = (uint16_t)lo[2] | ((uint32_t)(uint16_t)lo[3] << 16);
      o.z = (uint16_t)hi[0] | ((uint32_t)(uint16_t)hi[1] << 16);
      o.w = (uint16_t)hi[2] | ((uint32_t)(uint16_t)hi[3] << 16);
    } else {
      const uint32_t* w = reinterpret_cast<const uint32_t*>(p);
      o.x = w[0]; o.y = w[R / 4]; o.z = w[2 * (R / 4)]; o.w = w[3 * (R / 4)];
    }
    return o;
  };
  constexpr int NR = TM + TN;
  auto read = [&](auto SET, int q, const char* stage) {   // fragment q of a stage: B first, then A
    constexpr int set = decltype(SET)::value;
    if (q < TN) {
      if constexpr (B_KC) fb[set][q] = *reinterpret_cast<const uint4*>(stage + toffb[q]);
      else fb[set][q] = rc_read(stage + toffb[q], std::integral_constant<int, F::RB>{});
    } else {
      if constexpr (A_KC) fa[set][q - TN] = *reinterpret_cast<const uint4*>(stage + toffa[q - TN]);
      else fa[set][q - TN] = rc_read(stage + toffa[q - TN], std::integral_constant<int, F::RA>{});
    }
  };
  // MFMA m of a step
  constexpr int NM = TM * TN * (sizeof(T) == 2 ? 1 : 4);
  auto mfma = [&](auto SET, int m) {
    constexpr int set = decltype(SET)::value;
    if constexpr (sizeof(T) == 2) {
      const int i = m / TN, j = m % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[set][i]),
                                                          __builtin_bit_cast(bf16x8, fb[set][j]), acc[i][j], 0, 0, 0);
    } else {
      const int q = m / (TM * TN), i = m % (TM * TN) / TN, j = m % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(reinterpret_cast<const float*>(&fa[set][i])[q],
                                                       reinterpret_cast<const float*>(&fb[set][j])[q], acc[i][j], 0, 0, 0);
    }
  };
  // the last stage: `left` = K of this group's step that lies in the range (may be <= 0 or >= KD)
  auto multiply_last = [&](auto SET) {
    constexpr int set = decltype(SET)::value;
    const int left = k_end - k_begin - (nkt - 1) * BK - grp * KD;   // wave-uniform
    if (left <= 0) return;
    if (left < KD) {
      constexpr int PER = 4 / sizeof(T);   // elements per 32-bit word
      const int keep = left - E * kg;      // elements of this lane's fragments that count
      uint32_t m[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) m[d] = keep >= PER * (d + 1) ? 0xffffffffu : (PER == 2 && keep == 2 * d + 1) ? 0xffffu : 0u;
#pragma unroll
      for (int i = 0; i < TM; ++i) { fa[set][i].x &= m[0]; fa[set][i].y &= m[1]; fa[set][i].z &= m[2]; fa[set][i].w &= m[3]; }
#pragma unroll
      for (int j = 0; j < TN; ++j) { fb[set][j].x &= m[0]; fb[set][j].y &= m[1]; fb[set][j].z &= m[2]; fb[set][j].w &= m[3]; }
    }
#pragma unroll
    for (int x = 0; x < NM; ++x) mfma(SET, x);
  };

  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  // own loads of every stage but the n newest have landed
  auto wait_but = [&](int n) {
    if (ST > 3 && n >= 2) wait_vmcnt<2 * LPS>();
    else if (n >= 1) wait_vmcnt<LPS>();
    else wait_vmcnt<0>();
  };
#pragma unroll
  for (int s = 0; s < ST - 1; ++s) issue_any(s, s);
  wait_but(min(ST - 2, nkt - 1));
  __syncthreads();
  issue_any(ST - 1, ST - 1);
#pragma unroll
  for (int q = 0; q < NR; ++q) read(C0{}, q, smem);
  int slot = 1;   // of stage t
  // stage t >= 1.  STEADY: stage t + ST - 1 exists and lies in the range, no conditions.
  auto step = [&](auto SET, auto STEADY, int t) {
    using Prev = std::integral_constant<int, decltype(SET)::value ^ 1>;
    constexpr bool steady = decltype(STEADY)::value;
    if (steady) wait_vmcnt<(ST - 2) * LPS>();
    else wait_but(min(ST - 2, nkt - 1 - t));
    __syncthreads();   // also waits for this wave's fragments of t - 1
    const char* stage = smem + slot * F::STAGE;
    const int refill = slot == 0 ? ST - 1 : slot - 1;
    if (!steady) issue_any(t + ST - 1, refill);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if (m < NR) read(SET, m, stage);
      if (steady) {
#pragma unroll
        for (int i = m * LPS / NM; i < (m + 1) * LPS / NM; ++i) issue(i, refill);
      }
      mfma(Prev{}, m);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (steady) issued();
    slot = slot + 1 == ST ? 0 : slot + 1;
  };
  static_assert(NR <= NM, "a stage's fragments are read under the MFMAs of a step");
  const int nfull = (k_end - k_begin) / BK;
  int t = 1;
  for (; t + ST < nfull; t += 2) {
    step(C1{}, std::true_type{}, t);
    step(C0{}, std::true_type{}, t + 1);
  }
  for (; t < nkt; t += 2) {
    step(C1{}, std::false_type{}, t);
    if (t + 1 < nkt) step(C0{}, std::false_type{}, t + 1);
  }
  if (nkt & 1) multiply_last(C0{});
  else multiply_last(C1{});

  fit_epilogue<T, TC, TM, TN, WM, WN, G, F::IC>(g, acc, reinterpret_cast<float*>(smem), tid, grp, wm, wn, m0, n0, tile_m, split,
                                                EARLY ? &early : nullptr);
}

template <typename T, typename TC, bool A_KC, bool B_KC, int TM, int TN, int WM, int WN, int G, int ST, bool FAR>
__global__ void __launch_bounds__(64 * FIT_WAVES, (2 * Fit<T, TC, A_KC, B_KC, TM, TN, WM, WN, G, ST>::PER_CU)) gemm_fit_kernel(const GemmDev g) {
  fit_product<T, TC, A_KC, B_KC, TM, TN, WM, WN, G, ST, FAR>(g, blockIdx.x);
}

// fp32 over a short K: 32 x 64 tiles, or 32 x 32 as below, whose operands go from memory straight into the lanes that multiply them.  G waves
// take 16 of K each at a time, two such steps in flight; their sums meet in the epilogue.  Such a product is bound by its launch, one trip
// to memory and the instructions in front of and behind it (2 - 3 ns each): the ring above costs a second trip through LDS, a
// barrier and the arithmetic of its addresses.  Four waves for up to DIRECT_K (256 x 192 x 64 6.0 us there, 4.9 here; 256 x 64 x 64 6.5 | 4.7),
// eight for twice that while 32 x 32 tiles make one round.  A step that lies inside the matrix has no clamps and one multiplication an operand
// for its addresses: both products of a layer's backward pass 5.8 -> 5.2 us.
constexpr int DIRECT_K = 128, DIRECT_G = 4;
// LN: A's rows go through a LayerNorm first, which the waves take together (each holds its K of the 32 rows): a launch of 2.8 us less in front of a
// product that takes 5.2 us for 3.6 - 4.2 (256 x 64 -> 192; step of a 64-wide path on 256 tokens 155 -> 150 us).  The first column of tiles writes what the backward pass reads.
template <bool A_KC, bool B_KC, int TN, int G, bool LN = false>
__device__ __forceinline__ void direct_product(const GemmDev& g, int block, const RowNorm* ln = nullptr) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, kg = lane >> 4;
  const int tile_n = block / g.tiles_m, tile_m = block - tile_n * g.tiles_m;
  const int m0 = tile_m * 32, n0 = tile_n * 16 * TN;
  const float* const A = static_cast<const float*>(g.A);
  const float* const B = static_cast<const float*>(g.B);
  // rows and columns beyond the matrix re-read the last ones (their results are not stored); K beyond it counts as zero
  uint32_t ra[2], rb[TN];
#pragma unroll
  for (int i = 0; i < 2; ++i) ra[i] = (uint32_t)min(m0 + 16 * i + r, g.M - 1);
#pragma unroll
  for (int j = 0; j < TN; ++j) rb[j] = (uint32_t)min(n0 + 16 * j + r, g.N - 1);
  const uint32_t lda = (uint32_t)g.lda, ldb = (uint32_t)g.ldb;
  auto load = [&](auto KCc, auto WHOLE, const float* p, uint32_t ld, uint32_t row, int k, float (&v)[4]) {   // K k .. k + 3 of a row
    constexpr bool whole = decltype(WHOLE)::value;   // they lie inside the matrix
    if constexpr (decltype(KCc)::value) {   // K is a multiple of 4
      const float4 x = *reinterpret_cast<const float4*>(p + (row * ld + (uint32_t)(whole ? k : min(k, g.K - 4))));
      const bool in = whole || k < g.K;
      v[0] = in ? x.x : 0.f; v[1] = in ? x.y : 0.f; v[2] = in ? x.z : 0.f; v[3] = in ? x.w : 0.f;
    } else if constexpr (whole) {
      const uint32_t at = (uint32_t)k * ld + row;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = p[at + q * ld];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float x = p[(uint32_t)min(k + q, g.K - 1) * ld + row];
        v[q] = k + q < g.K ? x : 0.f;
      }
    }
  };
  constexpr int AHEAD = 2;
  static_assert(DIRECT_K / DIRECT_G == 16 * AHEAD, "a wave's steps are all in flight");
  float a[AHEAD][2][4], b[AHEAD][TN][4];
  const FitAhead<float> early = fit_request<float, TN, 2, G>(g, tid, m0, n0);
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) {
    const int k0 = 16 * (wave + G * s), k = k0 + 4 * kg;   // k0: uniform
    auto step = [&](auto WHOLE) {
#pragma unroll
      for (int i = 0; i < 2; ++i) load(std::bool_constant<A_KC>{}, WHOLE, A, lda, ra[i], k, a[s][i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) load(std::bool_constant<B_KC>{}, WHOLE, B, ldb, rb[j], k, b[s][j]);
    };
    if (k0 + 16 <= g.K) {
      step(std::true_type{});
    } else if (k0 < g.K) {
      step(std::false_type{});
    } else {   // not multiplied
#pragma unroll
      for (int q = 0; q < 4; ++q) a[s][0][q] = a[s][1][q] = 0.f;
    }
  }
  if constexpr (LN) {
    static_assert(A_KC, "a lane holds four K of a row");
    float4 gain[AHEAD], shift[AHEAD];
    bool in[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
      const int k = 16 * (wave + G * s) + 4 * kg;
      in[s] = k < g.K;
      gain[s] = *reinterpret_cast<const float4*>(ln->gain + min(k, g.K - 4));
      shift[s] = *reinterpret_cast<const float4*>(ln->shift + min(k, g.K - 4));
    }
    float* const part = reinterpret_cast<float*>(smem);   // [2][G][32]
    auto row_mean = [&](float (&v)[2], int which) {   // over the row's lanes, then the waves in order
      float* const p = part + which * 32 * G;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        v[i] += __shfl_xor(v[i], 16, WAVE);
        v[i] += __shfl_xor(v[i], 32, WAVE);
        if (kg == 0) p[32 * wave + 16 * i + r] = v[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        v[i] = p[16 * i + r];
#pragma unroll
        for (int w = 1; w < G; ++w) v[i] += p[32 * w + 16 * i + r];
        v[i] /= g.K;
      }
    };
    float mu[2] = {0.f, 0.f}, rs[2] = {0.f, 0.f};
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)   // K beyond the row is zero
#pragma unroll
      for (int i = 0; i < 2; ++i) mu[i] += (a[s][i][0] + a[s][i][1]) + (a[s][i][2] + a[s][i][3]);
    row_mean(mu, 0);
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
      if (in[s]) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) { const float t = a[s][i][q] - mu[i]; rs[i] += t * t; }
      }
    row_mean(rs, 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) rs[i] = 1.0f / sqrtf(rs[i] + ln->eps);
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
      if (in[s]) {
        const float gs[4] = {gain[s].x, gain[s].y, gain[s].z, gain[s].w}, bs[4] = {shift[s].x, shift[s].y, shift[s].z, shift[s].w};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
          for (int q = 0; q < 4; ++q) a[s][i][q] = (a[s][i][q] - mu[i]) * rs[i] * gs[q] + bs[q];
          const int row = m0 + 16 * i + r;
          if (tile_n == 0 && row < g.M)
            *reinterpret_cast<float4*>(ln->y + (size_t)row * g.K + 16 * (wave + G * s) + 4 * kg) = make_float4(a[s][i][0], a[s][i][1], a[s][i][2], a[s][i][3]);
        }
      }
    if (tile_n == 0 && wave == 0 && kg == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = m0 + 16 * i + r;
        if (row < g.M) { ln->mean[row] = mu[i]; ln->rstd[row] = rs[i]; }
      }
    }
  }
  // each step in sums of its own, as many as the fitted tile's groups: one chain over both errs by a quarter more (K = 128, root mean
  // square, 1.25e-6 against 1.00e-6 on normal numbers) and is no faster
  f32x4 acc[2][TN], step[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = step[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) {
    if (16 * (wave + G * s) >= g.K) break;   // uniform
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f32x4& sum = s == 0 ? acc[i][j] : step[i][j];
          sum = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][i][q], b[s][j][q], sum, 0, 0, 0);
        }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += step[i][j];
  fit_epilogue<float, float, 2, TN, 1, 1, G, 2>(g, acc, reinterpret_cast<float*>(smem), tid, wave, 0, 0, m0, n0, tile_m, 0, &early);
}
template <bool A_KC, bool B_KC, int TN, int G> __global__ void __launch_bounds__(64 * G, 2) gemm_direct_kernel(const GemmDev g) {
  direct_product<A_KC, B_KC, TN, G>(g, blockIdx.x);
}
template <int TN> __global__ void __launch_bounds__(64 * DIRECT_G, 2) gemm_direct_norm_kernel(const GemmDev g, const RowNorm ln) {
  direct_product<true, false, TN, DIRECT_G, true>(g, blockIdx.x, &ln);
}

// The two products of a linear layer's backward pass, X^T dY (blocks 0 .. first - 1) and dY W^T, in one launch of 32 x 64 tiles.
// Bound by launches: a step on 256 tokens is fifty of 5 us each, and neither product reads what the other writes (260 -> 209 us).  For
// products whose tiles are on the compute units at once; larger ones gain nothing from company (their tiles fill the same rounds).
template <typename T, int TN> __global__ void __launch_bounds__(64 * FIT_WAVES, 2) gemm_fit_pair_kernel(const GemmDev dw, const GemmDev dx, int first) {
  const int block = blockIdx.x;
  if (block < first) fit_product<T, float, false, false, 2, TN, 1, 1, 8, 3, false>(dw, block);
  else fit_product<T, T, true, true, 2, TN, 1, 1, 8, 3, false>(dx, block - first);
}

// The same in bf16 for products of a round or a few, a workgroup to a compute unit: dW in 128 x 128 tiles, dX in 32 TX x 128 ones.  Each alone
// ends, or never fills, the chip with units idle: 896 x 3584 over 1400 tokens are 196 tiles on 256 units, the dX beside it 105 - 154.
template <int TX> __global__ void __launch_bounds__(64 * FIT_WAVES, 2) gemm_fit_pair_wide_kernel(const GemmDev dw, const GemmDev dx, int n_first, bool dw_first) {
  const int block = blockIdx.x, behind = block - n_first;
  if ((behind < 0) == dw_first) fit_product<bf16, float, false, false, 4, 4, 2, 2, 2, 4, false>(dw, dw_first ? block : behind);
  else fit_product<bf16, bf16, true, true, TX, 4, 2, 2, 2, 4, false>(dx, dw_first ? behind : block);
}

// The same in fp32 where both contractions are short
template <int G> __global__ void __launch_bounds__(64 * G, 2) gemm_direct_pair_kernel(const GemmDev dw, const GemmDev dx, int first) {
  const int block = blockIdx.x;
  if (block < first) direct_product<false, false, 2, G>(dw, block);
  else direct_product<true, true, 2, G>(dx, block - first);
}

template <typename F> GemmDev fit_dev(const GemmArgs& a) {
  GemmDev g;
  g.A = a.A; g.B = a.B; g.C = a.C; g.M = a.M; g.N = a.N; g.K = a.K;
  g.lda = a.lda; g.ldb = a.ldb; g.ldc = a.ldc;
  g.bias = a.bias; g.resid = a.resid; g.aux_out = a.aux_out; g.aux_in = a.aux_in; g.act = a.act;
  g.partial = a.partial;
  g.tiles_m = (a.M + F::BM - 1) / F::BM;
  g.tiles_n = (a.N + F::BN - 1) / F::BN;
  const int steps = (a.K + F::BK - 1) / F::BK;
  const int want = std::max(1, std::min(a.splits, steps));
  g.k_per_split = (steps + want - 1) / want * F::BK;
  g.splits = (a.K + g.k_per_split - 1) / g.k_per_split;
  g.colsum_partial = a.colsum ? a.colsum_partial : nullptr;
  gemm_fast_map(g);
  return g;
}

template <typename T, typename TC, bool A_KC, bool B_KC, int TM, int TN, int WM, int WN, int G, int ST, bool FAR = false>
dipaco_status run_fit(const GemmArgs& a, hipStream_t s) {
  using F = Fit<T, TC, A_KC, B_KC, TM, TN, WM, WN, G, ST>;
  if constexpr (!FAR) {
    constexpr uint64_t most = 1ull << 32;
    if (fit_span(A_KC, F::BM, F::BK, a.M, a.K, a.lda, sizeof(T)) >= most || fit_span(B_KC, F::BN, F::BK, a.N, a.K, a.ldb, sizeof(T)) >= most)
      return run_fit<T, TC, A_KC, B_KC, 2, 4, 1, 1, 8, 3, true>(a, s);
  }
  auto kern = gemm_fit_kernel<T, TC, A_KC, B_KC, TM, TN, WM, WN, G, ST, FAR>;
  static std::atomic<unsigned long long> lds_set{0};   // per instantiation
  if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), F::LDS, lds_set)) return e;
  const GemmDev g = fit_dev<F>(a);
  const long blocks = (long)g.tiles_m * g.tiles_n * g.splits;
  if (!launch_fits(blocks, 64 * FIT_WAVES)) return fail(DIPACO_ESHAPE, "gemm: too many tiles");
  kern<<<(unsigned)blocks, 64 * FIT_WAVES, F::LDS, s>>>(g);
  DIPACO_LAUNCH_CHECK();
  if (a.raw_planes) return g.splits == a.splits ? DIPACO_OK : fail(DIPACO_EINVAL, "gemm: raw planes take the splits of gemm_raw_splits");
  if (g.splits > 1) return launch_splitk_reduce(a.partial, static_cast<float*>(a.C), a.M, a.N, a.ldc, g.splits, s);
  if (a.colsum) return launch_sum_rows(a.colsum_partial, a.colsum, g.tiles_m, a.N, s, a.sum_batch);
  return DIPACO_OK;
}

// whether a 32 x 64 tile's product over up to `most_k` is taken by direct_product (32-bit element offsets)
bool direct_takes(const GemmArgs& a, bool a_kc, bool b_kc, int most_k) {
  const uint64_t most = 1ull << 32;
  return a.K <= most_k && std::max(1, a.splits) == 1 && !a.raw_planes && (uint64_t)(a_kc ? a.M : a.K) * a.lda < most &&
         (uint64_t)(b_kc ? a.N : a.K) * a.ldb < most;
}
template <int TN> struct DirectTile { static constexpr int BM = 32, BN = 16 * TN, BK = 16; };
template <bool A_KC, bool B_KC, int TN, int G> dipaco_status run_direct(const GemmArgs& a, hipStream_t s) {
  const GemmDev g = fit_dev<DirectTile<TN>>(a);
  const long blocks = (long)g.tiles_m * g.tiles_n;
  if (!launch_fits(blocks, 64 * G)) return fail(DIPACO_ESHAPE, "gemm: too many tiles");
  constexpr int LDS = fit_epilogue_bytes(2, TN, 1, 1, G);
  static_assert(LDS <= 64 * 1024, "no limit to raise");
  gemm_direct_kernel<A_KC, B_KC, TN, G><<<(unsigned)blocks, 64 * G, LDS, s>>>(g);
  DIPACO_LAUNCH_CHECK();
  if (a.colsum) return launch_sum_rows(a.colsum_partial, a.colsum, g.tiles_m, a.N, s, a.sum_batch);
  return DIPACO_OK;
}

// Tile shapes: 1 = 32 x 64, 2 .. 5 = 64, 96, 128, 160 rows x 128.  fp32 has 1, 2 (its matrix-core steps are sixteen times as
// long: 64 x 128 tiles, two workgroups per compute unit, were the fastest of the 128-column ones on every product measured) and, on the
// bf16 matrix cores (gemm_split.hip), 4 and a 64 x 128 tile as number 3; row-contiguous A in bf16 1, 2 and 4.
bool fit_built(int t, bool bf16_operands, bool a_kc) { return t <= 2 || t == 4 || (t == 3 && !bf16_operands) || (bf16_operands && a_kc); }

// Microseconds of `tiles` tiles over K: rounds of 256 workgroups x (fixed + per 1000 of K).  Fitted to launches of 256 .. 8192
// rows, K 64 .. 8192 (rel. error 15 %): 3000 x 896 x 3584 bf16 34.8 / 26.0 / 28.8 / 33.7 us for shapes 2 .. 5, 5700 x 896 x 3584
// 51 / 49 / 53 / 38, 1000 x 896 x 3584 20 (shape 1) / 21 / 24 / 28, 256 x 896 x 3584 10.5 / 19.
// The 64 x 128 shape runs two workgroups on a compute unit, so that over several rounds one loads and stores while the other
// multiplies: bf16, outputs in many rounds, K = 48 / 200 / 520: 111 / 25.7 / 38.7 us, the next best shape 145 / 31.2 / 42.7
// (9780 x 13336, 2540 x 7248, 9000 x 2000).  In a weight gradient, whose workgroups all end together, 257 .. 512
// of them are one round of twice the length, and a third 256 behind them lands two to a unit again: 256 x 768 over 2^20 rows in
// fp32 2930 us in 504 workgroups, 3500 - 3900 in 768, 2980 in 1536.
// fp32 in 128 x 128 tiles, us against 64 x 128 ones, by tiles over K (K = 256 / 512 / 2048 / 8192): 256 tiles 28 / 42 / 124 / 452 against
// 25 / 39 / 126 / 477, 384 35 / 53 / 160 / 620 against 34 / 55 / 188 / 726, 512 39 / 57 / 182 / 700 against 42 / 70 / 245 / 948, 2048
// 132 / 206 / 708 against 150 / 262 / 968; at K = 64 512 tiles are level.  A round of 512 workgroups is two to a compute unit.
// In 64 x 128 tiles of bf16 parts, one to a compute unit: 250 tiles 21.5 / 65 / 225 us (K = 512 / 2048 / 8192) against 22.5 / 71 - 80 /
// 252 - 280 on the fp32 instruction, 750 tiles 58 against 55: here taken for one round.
long shape_tiles(int t, int M, int N, bool bf16_operands) {
  const int bm = t == 3 && !bf16_operands ? 64 : 32 * t, bn = t == 1 ? 64 : 128;
  return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
}
constexpr double BF16_FIXED[6] = {0, 3.0, 3.5, 4.5, 5.0, 6.0}, BF16_PER_K[6] = {0, 1.8, 4.2, 5.2, 6.4, 8.1};
inline __attribute__((always_inline)) double shape_cost(int t, long tiles, int K, bool bf16_operands, bool a_kc) {
  if (t == 3 && !bf16_operands) return tiles <= 256 ? 8.0 + 27.0 * K * 1e-3 : 1e30;
  if (t == 4 && !bf16_operands) {
    const long full = tiles / 512, rest = tiles % 512;   // rounds of two workgroups a unit; behind them up to one a unit, or on the way to two
    const double round = 18.0 + 88.0 * K * 1e-3, single = 10.5 + 60.0 * K * 1e-3;
    return 3.0 + (double)full * round + (rest == 0 ? 0.0 : single + std::max(0L, rest - 256) / 256.0 * (round - single));
  }
  const double f = bf16_operands ? BF16_FIXED[t] : t == 1 ? 4.0 : 3.6, k = bf16_operands ? BF16_PER_K[t] : t == 1 ? 8.7 : 32.5;
  const long rounds = t == 2 && !a_kc && tiles > 256 ? (tiles + 511) / 512 * 2 : (tiles + 255) / 256;
  if (t == 2 && a_kc && bf16_operands) return 4.9 + (double)rounds * (1.6 + k * K * 1e-3);
  return 3.0 + (double)rounds * (f + k * K * 1e-3);
}

// The same for one fp32 product that is not cut over K, close enough (rel. error 5 %) to tell the two ways of multiplying apart where they
// lie near each other: 1, 2 on the fp32 instruction, 3, 4 in bf16 parts.  Fitted to 3144 products of 16 - 1280 tiles of 128 x 128, K 32 -
// 8192, of all three layouts.  Up to 128 of K tile 1 is gemm_direct_kernel; its stages are 256 of K, tile 3's 128; two workgroups of 2
// and 4 share a unit, so that a second round costs less than the first; A.B^T is the slowest layout in parts of 128 x 128.  Tile 4, and
// 3 in more than one round, have to be ahead by 3 and 7 %: then 5 of the 3144 are more than 3 % behind what the fp32 instruction took with
// its rule above (with the prices above for all four, 375: 4036 x 512 x 264 14.8 us in tile 2, 18.0 in 3; 2564 x 2056 x 136 23.4, 26.6 in
// 4; 1476 x 2048 x 896 A.B^T 56.7, 61.8 in 4), and all together take 0.95 of its time.
double f32_cost(int t, long tiles, int K, bool a_kc, bool b_kc) {
  const double rounds = (double)((tiles + 255) / 256);
  auto up = [&](int stage) { return (double)((K + stage - 1) / stage * stage); };
  if (t == 1) {
    if (K <= DIRECT_K) return std::max(7.5, 5.5 + rounds * (0.6 + 7.8e-3 * K));
    return 1.04 * (2.5 + rounds * (3.2 + (!a_kc ? 7.7e-3 : b_kc ? 6.9e-3 : 7.3e-3) * 0.5 * (K + up(256))));
  }
  if (t == 2) return std::max(7.7, 2.8 + rounds * (2.7 + 28.8e-3 * K));
  if (t == 3) return (rounds > 1.0 ? 1.07 : 1.0) * (3.0 + rounds * (4.5 + 24.7e-3 * up(128)) + 2.0 * ((double)tiles / 256.0 - (rounds - 1.0)));
  const long full = tiles / 512, rest = tiles % 512;
  const double single = (!a_kc ? 52.2e-3 : b_kc ? 54.5e-3 : 50.5e-3) * K;
  double c = 4.0 + (double)full * (12.8 + 75.6e-3 * K);
  if (rest > 256) c += 12.4 + 61.8e-3 * K + (double)(rest - 256) / 256.0 * (0.4 + 13.8e-3 * K);
  else if (rest) c += 7.5 + single + 2.0 * (double)rest / 256.0;
  return 1.03 * c;
}

std::atomic<int> g_forced_fit{0};
int pick_fit(int M, int N, int K, int splits, bool bf16_operands, bool a_kc, bool b_kc) {
  if (g_forced_fit) {
    int t = g_forced_fit;
    while (!fit_built(t, bf16_operands, a_kc)) --t;
    return t;
  }
  auto cost = [&](int t) { return shape_cost(t, shape_tiles(t, M, N, bf16_operands) * splits, K, bf16_operands, a_kc); };
  const bool by_parts = !bf16_operands && splits == 1;   // 3 and 4 against the better of 1 and 2
  int best = 1;
  for (int t = 2; t <= (by_parts ? 2 : 5); ++t)
    if (fit_built(t, bf16_operands, a_kc) && cost(t) < cost(best)) best = t;
  if (by_parts) {
    auto f32 = [&](int t) { return f32_cost(t, shape_tiles(t, M, N, false), K, a_kc, b_kc); };
    double least = f32(best);
    for (int t = 3; t <= 4; ++t)
      if (f32(t) < least) { least = f32(t); best = t; }
  }
  return best;
}

// fp32 tiles of 32 x 32 while one round of 256 compute units holds them: the eight waves' matrix instructions over 256 of K are 1.7 us of a
// launch of 7 in a 32 x 64 tile, while compute units idle.  500 x 256 x 768 10.7 -> 8.1 us, 1000 x 256 x 768 11.5 -> 8.4, 500 x 512 x 2048
// 21.7 -> 13.9, 512 x 512 x 4096 36.8 -> 22.7; the same sums, bit for bit.
long narrow_tiles(int M, int N) { return (long)((M + 31) / 32) * ((N + 31) / 32); }

template <typename T, typename TC, bool A_KC, bool B_KC> dipaco_status run_fit_shape(const GemmArgs& a, hipStream_t s) {
  const int splits = std::max(1, a.splits);
  const int t = a.raw_planes ? 1 : pick_fit(a.M, a.N, (a.K + splits - 1) / splits, splits, sizeof(T) == 2, A_KC, B_KC);
  if constexpr (sizeof(T) == 4) {
    const bool narrow = narrow_tiles(a.M, a.N) * splits <= 256;
    if (t == 1 && direct_takes(a, A_KC, B_KC, DIRECT_K))
      return narrow ? run_direct<A_KC, B_KC, 2, DIRECT_G>(a, s) : run_direct<A_KC, B_KC, 4, DIRECT_G>(a, s);
    if (t == 1 && narrow && direct_takes(a, A_KC, B_KC, 2 * DIRECT_K)) return run_direct<A_KC, B_KC, 2, 2 * DIRECT_G>(a, s);
    if (t == 1 && narrow) return run_fit<T, TC, A_KC, B_KC, 2, 2, 1, 1, 8, 3>(a, s);
  }
  if (t == 1) return run_fit<T, TC, A_KC, B_KC, 2, 4, 1, 1, 8, 3>(a, s);
  if constexpr (sizeof(T) == 4) {
    if (t == 3 || t == 4) {
      constexpr uint64_t most = 1ull << 32;   // 32-bit offsets there too
      if (fit_span(A_KC, 128, 32, a.M, a.K, a.lda, 4) < most && fit_span(B_KC, 128, 32, a.N, a.K, a.ldb, 4) < most)
        return launch_gemm_split(a, t == 3 ? 64 : 128, s);
    }
  } else {
    if constexpr (A_KC) {
      if (t == 3) return run_fit<T, TC, A_KC, B_KC, 3, 4, 2, 2, 2, 4>(a, s);
      if (t == 5) return run_fit<T, TC, A_KC, B_KC, 5, 4, 2, 2, 2, 4>(a, s);
    }
    if (t == 4) return run_fit<T, TC, A_KC, B_KC, 4, 4, 2, 2, 2, 4>(a, s);
  }
  return run_fit<T, TC, A_KC, B_KC, 2, 4, 2, 2, 2, 3>(a, s);
}

// both products in 32 x 64 tiles, uncut, on the compute units at once; 32-bit offsets
template <typename T> bool pair_fits(const GemmArgs& dw, const GemmArgs& dx) {
  using F = Fit<T, T, true, true, 2, 4, 1, 1, 8, 3>;
  constexpr uint64_t most = 1ull << 32;
  auto tiles = [](const GemmArgs& a) { return (long)((a.M + 31) / 32) * ((a.N + 63) / 64); };
  return dw.splits <= 1 && dx.splits <= 1 && pick_fit(dw.M, dw.N, dw.K, 1, sizeof(T) == 2, false, false) == 1 &&
         pick_fit(dx.M, dx.N, dx.K, 1, sizeof(T) == 2, true, true) == 1 && tiles(dw) + tiles(dx) <= 256 &&
         fit_span(false, F::BM, F::BK, dw.M, dw.K, dw.lda, sizeof(T)) < most && fit_span(false, F::BN, F::BK, dw.N, dw.K, dw.ldb, sizeof(T)) < most &&
         fit_span(true, F::BM, F::BK, dx.M, dx.K, dx.lda, sizeof(T)) < most && fit_span(true, F::BN, F::BK, dx.N, dx.K, dx.ldb, sizeof(T)) < most;
}

// Microseconds until `n` tiles of `us` and then `n2` of `us2` are done, dealt to 256 compute units as they come free
double dealt(long n, double us, long n2, double us2) {
  constexpr int MOST = 64;   // times at which some units come free; far more than a pair's tiles make
  double at[MOST];
  long units[MOST];
  int count = 1;
  at[0] = 0.0;
  units[0] = 256;
  double end = 0.0;
  for (int kind = 0; kind < 2; ++kind)
    for (long left = kind ? n2 : n; left > 0;) {
      int k = 0;
      for (int i = 1; i < count; ++i)
        if (at[i] < at[k]) k = i;
      const long take = std::min(left, units[k]);
      const double done = at[k] + (kind ? us2 : us);
      end = std::max(end, done);
      left -= take;
      if (take == units[k]) at[k] = done;
      else if (count == MOST) return 1e30;
      else { units[k] -= take; at[count] = done; units[count++] = take; }
    }
  return end;
}
GemmWidePair pick_wide(const GemmArgs& dw, const GemmArgs& dx) {   // the longer tiles first
  const long nw = shape_tiles(4, dw.M, dw.N, true);
  const double cw = BF16_FIXED[4] + BF16_PER_K[4] * dw.K * 1e-3;
  GemmWidePair best{0, true, 1e30};
  for (int t = 3; t <= 5; ++t) {
    const long nx = shape_tiles(t, dx.M, dx.N, true);
    if (nw + nx > 256 * 8) continue;
    const double cx = BF16_FIXED[t] + BF16_PER_K[t] * dx.K * 1e-3;
    const bool dw_first = cw >= cx;
    const double us = 3.0 + (dw_first ? dealt(nw, cw, nx, cx) : dealt(nx, cx, nw, cw));
    if (us < best.us) best = GemmWidePair{32 * t, dw_first, us};
  }
  return best;
}

}  // namespace

int gemm_fit_groups(int M, int N, int K, int splits) { return pick_fit(M, N, K, splits, true, false, false) == 1 ? 8 : 2; }

GemmWidePair gemm_fit_pair_wide(const GemmArgs& dw, const GemmArgs& dx) {
  constexpr uint64_t most = 1ull << 32;
  const GemmWidePair none{0, true, 1e30};
  if (g_forced_fit || dw.splits > 1 || dx.splits > 1 || dw.raw_planes || dx.raw_planes) return none;
  if (fit_span(false, 128, 64, dw.M, dw.K, dw.lda, 2) >= most || fit_span(false, 128, 64, dw.N, dw.K, dw.ldb, 2) >= most ||
      fit_span(true, 160, 64, dx.M, dx.K, dx.lda, 2) >= most || fit_span(true, 128, 64, dx.N, dx.K, dx.ldb, 2) >= most) return none;
  return pick_wide(dw, dx);
}
dipaco_status launch_gemm_fit_pair_wide(const GemmArgs& dw, const GemmArgs& dx, const GemmWidePair& p, hipStream_t s) {
  auto run = [&](auto TXc) -> dipaco_status {
    constexpr int TX = decltype(TXc)::value;
    using W = Fit<bf16, float, false, false, 4, 4, 2, 2, GEMM_WIDE_GROUPS, 4>;
    using X = Fit<bf16, bf16, true, true, TX, 4, 2, 2, GEMM_WIDE_GROUPS, 4>;
    constexpr int LDS = W::LDS > X::LDS ? W::LDS : X::LDS;
    auto kern = gemm_fit_pair_wide_kernel<TX>;
    static std::atomic<unsigned long long> lds_set{0};   // per instantiation
    if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), LDS, lds_set)) return e;
    const GemmDev w = fit_dev<W>(dw), x = fit_dev<X>(dx);
    const int nw = w.tiles_m * w.tiles_n, nx = x.tiles_m * x.tiles_n;
    kern<<<nw + nx, 64 * FIT_WAVES, LDS, s>>>(w, x, p.dw_first ? nw : nx, p.dw_first);
    DIPACO_LAUNCH_CHECK();
    if (dx.colsum) return launch_sum_rows(dx.colsum_partial, dx.colsum, x.tiles_m, dx.N, s, dx.sum_batch);
    return DIPACO_OK;
  };
  if (p.rows == 96) return run(std::integral_constant<int, 3>{});
  if (p.rows == 128) return run(std::integral_constant<int, 4>{});
  return run(std::integral_constant<int, 5>{});
}

template <typename T> bool gemm_fit_pair_takes(const GemmArgs& dw, const GemmArgs& dx) { return pair_fits<T>(dw, dx); }
template <typename T> dipaco_status launch_gemm_fit_pair(const GemmArgs& dw, const GemmArgs& dx, hipStream_t s) {
  auto run = [&](auto TNc) -> dipaco_status {
    constexpr int TN = decltype(TNc)::value;
    using W = Fit<T, float, false, false, 2, TN, 1, 1, 8, 3>;
    using X = Fit<T, T, true, true, 2, TN, 1, 1, 8, 3>;
    constexpr int LDS = W::LDS > X::LDS ? W::LDS : X::LDS;
    auto kern = gemm_fit_pair_kernel<T, TN>;
    static std::atomic<unsigned long long> lds_set{0};   // per instantiation
    if (dipaco_status e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), LDS, lds_set)) return e;
    const GemmDev w = fit_dev<W>(dw), x = fit_dev<X>(dx);
    const int first = w.tiles_m * w.tiles_n;
    kern<<<first + x.tiles_m * x.tiles_n, 64 * FIT_WAVES, LDS, s>>>(w, x, first);
    DIPACO_LAUNCH_CHECK();
    if (dx.colsum) return launch_sum_rows(dx.colsum_partial, dx.colsum, x.tiles_m, dx.N, s, dx.sum_batch);
    return DIPACO_OK;
  };
  if constexpr (sizeof(T) == 4) {
    const long narrow = narrow_tiles(dw.M, dw.N) + narrow_tiles(dx.M, dx.N);
    if (narrow <= 256 && direct_takes(dw, false, false, 2 * DIRECT_K) && direct_takes(dx, true, true, 2 * DIRECT_K)) {
      constexpr int G = 2 * DIRECT_G;
      const GemmDev w = fit_dev<DirectTile<2>>(dw), x = fit_dev<DirectTile<2>>(dx);
      const int first = w.tiles_m * w.tiles_n;
      gemm_direct_pair_kernel<G><<<first + x.tiles_m * x.tiles_n, 64 * G, fit_epilogue_bytes(2, 2, 1, 1, G), s>>>(w, x, first);
      DIPACO_LAUNCH_CHECK();
      if (dx.colsum) return launch_sum_rows(dx.colsum_partial, dx.colsum, x.tiles_m, dx.N, s, dx.sum_batch);
      return DIPACO_OK;
    }
    if (narrow <= 256) return run(std::integral_constant<int, 2>{});
  }
  return run(std::integral_constant<int, 4>{});
}
template bool gemm_fit_pair_takes<float>(const GemmArgs&, const GemmArgs&);
template bool gemm_fit_pair_takes<bf16>(const GemmArgs&, const GemmArgs&);
template dipaco_status launch_gemm_fit_pair<float>(const GemmArgs&, const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm_fit_pair<bf16>(const GemmArgs&, const GemmArgs&, hipStream_t);

void set_gemm_fit_shape(int t) { g_forced_fit = t; }

// 32 x 896 x 3584 is 14 workgroups of 32 x 64, each a serial walk over 14 stages (10 - 12 us, a few CUs' worth of bandwidth); cut
// into up to eight slices, two stages each, the chip reads the weights at once and the LayerNorm behind the product adds the planes.
int gemm_raw_splits(int M, int N, int K, bool bf16_operands) {
  const int bk = 8 * FIT_STEP / (bf16_operands ? 2 : 4);
  const int tiles = ((M + 31) / 32) * ((N + 63) / 64), steps = (K + bk - 1) / bk;
  const int want = std::min(std::min(8, steps), 256 / std::max(tiles, 1));
  if (want < 2) return 1;
  const int per = (steps + want - 1) / want;
  return (steps + per - 1) / per;
}

WeightTiles raw_product_weights(const bf16* W, int rows, int N, int K) {   // run_fit_shape's tile for planes
  using F = Fit<bf16, bf16, true, false, 2, 4, 1, 1, 8, 3>;
  const int splits = gemm_raw_splits(rows, N, K, true), steps = (K + F::BK - 1) / F::BK, tiles_m = (rows + F::BM - 1) / F::BM, tiles_n = (N + F::BN - 1) / F::BN;
  return WeightTiles{W, 2 * N, K, tiles_m * tiles_n * splits, tiles_m, (steps + splits - 1) / splits * F::BK, tiles_n};
}

// A product behind a LayerNorm in one launch with it: while one round of workgroups holds the product, each of which normalises its rows.  Where the
// 32 x 64 tile is the cheapest: above 16 of K.  Without column sums, which nothing behind it would add up.
bool gemm_norm_takes(const GemmArgs& a) {
  return !a.out_f32 && !a.colsum && !a.trans_a && !a.trans_b && a.lda == a.K && std::max(1, a.splits) == 1 && !g_forced_fit &&
         shape_tiles(1, a.M, a.N, false) <= 256 && direct_takes(a, true, false, DIRECT_K) && pick_fit(a.M, a.N, a.K, 1, false, true, false) == 1;
}
dipaco_status launch_gemm_norm(const GemmArgs& a, const RowNorm& ln, hipStream_t s) {
  auto run = [&](auto TNc) -> dipaco_status {
    constexpr int TN = decltype(TNc)::value;
    const GemmDev g = fit_dev<DirectTile<TN>>(a);
    gemm_direct_norm_kernel<TN><<<g.tiles_m * g.tiles_n, 64 * DIRECT_G, fit_epilogue_bytes(2, TN, 1, 1, DIRECT_G), s>>>(g, ln);
    DIPACO_LAUNCH_CHECK();
    return DIPACO_OK;
  };
  return narrow_tiles(a.M, a.N) <= 256 ? run(std::integral_constant<int, 2>{}) : run(std::integral_constant<int, 4>{});
}

size_t gemm_raw_plane_floats(int M, int N, int K, bool bf16_operands) {
  size_t most = 0;
  for (int m = std::min(M, 32);; m = std::min(M, m + 32)) {   // the split count depends on the rows in steps of 32
    if (256 / (((m + 31) / 32) * ((N + 63) / 64)) < 2) break;
    const int s = gemm_raw_splits(m, N, K, bf16_operands);
    if (s > 1) most = std::max(most, (size_t)s * m * N);
    if (m == M) break;
  }
  return most;
}

GemmFitTiles gemm_fit_tiles(int M, int N, bool bf16_operands, bool a_k_contiguous) {
  GemmFitTiles f{{}, bf16_operands, a_k_contiguous};
  for (int t = 1; t <= 5; ++t) f.tiles[t] = fit_built(t, bf16_operands, a_k_contiguous) ? shape_tiles(t, M, N, bf16_operands) : 0;
  return f;
}
double gemm_fit_cost(const GemmFitTiles& f, int K, int splits) {
  double best = 1e30;
#pragma unroll
  for (int t = 1; t <= 5; ++t)
    if (f.tiles[t]) best = std::min(best, shape_cost(t, f.tiles[t] * splits, K, f.bf16_operands, f.a_k_contiguous));
  return best;
}

template <typename T> dipaco_status launch_gemm_fit(const GemmArgs& a, hipStream_t s) {
  if (a.out_f32) return run_fit_shape<T, float, false, false>(a, s);
  if (!a.trans_b) return run_fit_shape<T, T, true, false>(a, s);
  return run_fit_shape<T, T, true, true>(a, s);
}
template dipaco_status launch_gemm_fit<float>(const GemmArgs&, hipStream_t);
template dipaco_status launch_gemm_fit<bf16>(const GemmArgs&, hipStream_t);

}  // namespace dipaco

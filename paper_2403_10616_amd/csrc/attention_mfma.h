// Causal attention on the matrix cores (bf16 operands, fp32 softmax and accumulation), head sizes 32, 64 and 128.
//
// Everything is arranged so that the probabilities never leave registers.  A 32x32 MFMA leaves its result with
// lane l holding column l%32 and rows 8*(e/4) + 4*(l/32) + e%4 (e = 0..15); the B operand of the next MFMA wants
// lane l to hold column l%32 and eight contraction indices.  So whatever must be contracted next is made the
// ROW index of the score tile:
//   forward, dQ:   S^T = K.Q^T  (rows = keys, columns = queries)  ->  O^T += V^T.P^T,   dQ^T += K^T.dS^T
//   dK, dV:        S   = Q.K^T  (rows = queries, columns = keys)  ->  dV^T += dO^T.P,   dK^T += Q^T.dS
// Softmax state (running max, sum, log-sum-exp, D = rowsum(dO*O)) is per query: per lane in the first family, per
// accumulator row in the second.  Exponentials are base 2 with log2(e) folded into the score scale.
// On this chip matrix-core and vector-ALU instructions of the waves of one SIMD do not run side by side (measured:
// 16 MFMAs + 256 FMAs take the sum of their times at two or more waves per SIMD), so every vector instruction of the
// inner loops is paid in full: the forward kernel adds its row sums two bf16 values per instruction on the packed
// probabilities, walks its two stages with compile-time LDS offsets, and leaves the sum over a lane pair to the end.
//
// One workgroup = 4 waves (or two groups of 4: below), each wave owns 32 queries (or 32 keys).  K / V (or Q / dO) tiles of 64 rows x 64
// columns go from global memory straight into LDS (16-byte global_load_lds: lane l of a wave-level load writes
// LDS bytes [16 l, 16 l + 16), so the swizzle is applied by choosing which 16 bytes a lane fetches) into a ring
// of stages that runs two or three tiles ahead of the arithmetic, one barrier per tile.  A tile is stored once,
// row-major, and read in both orientations:
//   * rows as the MFMA row index, contraction along the 64 columns: one ds_read_b128 per fragment;
//   * columns as the MFMA row index, contraction along the tile's rows (the V^T, K^T, dO^T, Q^T operands):
//     ds_read_b64_tr_b16, which transposes 4x4 halfword blocks across each group of 16 lanes.  Lane 4e+q of a
//     group points at columns 4q..4q+3 of tile row T(e); lane i then receives column i of rows T(0..3).  The
//     rows T are chosen in the order in which an accumulator holds them (4h + 0..3, then 8 + 4h + 0..3 of each
//     group of 16), so that accumulator elements 8g..8g+7, packed to bf16, are the matching B operand.
// Chunk c (16 bytes) of tile row r sits at chunk position c ^ swz(r), swz(r) = 4*bit1(r) + bits3:2(r): both kinds
// of read are then free of bank conflicts (rows two apart land in different 64-byte groups for the transposing
// read; the lane groups that a ds_read_b128 serves together see eight different swizzles per row parity).
// No atomics: every output element has exactly one writer and a fixed summation order.
//
// Head sizes.  A tile is kept as panels of 64 rows x 64 columns (128-byte rows), so one swizzle and one set of
// fragment offsets serve every head size: head size 128 is two panels side by side, head size 32 uses the first half
// of one panel's columns (the lanes whose 16 bytes fall into the other half fetch a valid chunk again, so that no
// load is conditional).  Head sizes 32 and 128 keep 16 bits of the probabilities and of dS in the second products and sum
// rows in fp32 (split_p below); head size 64 rounds them to bf16.  Measured on 8 sequences x 8 heads x 512 positions, head
// size 128: forward 19 us, backward 69 (with operands rounded to bf16 16 and 55, one-thread-per-row kernels 1470 and 22960).
//
// The kernels for head size 64 are compiled in attention_mfma.hip, those for 32 and 128 in attention_mfma_exact.hip: the latter
// honour NaN and keep non-finite values from rows that do not see them (attention_plain.h); with head size 64 such a value may
// reach earlier rows of its 64-row tile.
#pragma once
#include <type_traits>

#include "attention_plain.h"
#include "kernels.h"
#include "mma_tile.h"

namespace dipaco {

namespace {

constexpr int AT_THREADS = 256;
constexpr int PANEL_BYTES = 64 * TILE_ROW_BYTES;   // 64 rows x 64 columns of bf16
template <int DH> constexpr int panels() { return DH > 64 ? 2 : 1; }
template <int DH> constexpr int tile_bytes() { return panels<DH>() * PANEL_BYTES; }
// 1 / sqrt(d_head), the scale of the scores
template <int DH> constexpr float score_scale() { return DH == 32 ? 0.17677669529663689f : DH == 64 ? 0.125f : 0.088388347648318447f; }
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;

__device__ __forceinline__ f32x16 mfma16(const uint4& a, const uint4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ void zero(f32x16& v) {
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = 0.f;
}
// accumulator elements E0..E0+7 as a bf16 B fragment (contraction slots in accumulator order)
template <int E0> __device__ __forceinline__ uint4 pack8(const f32x16& v) {
  bf16x8 o = {(bf16)v[E0 + 0], (bf16)v[E0 + 1], (bf16)v[E0 + 2], (bf16)v[E0 + 3],
              (bf16)v[E0 + 4], (bf16)v[E0 + 5], (bf16)v[E0 + 6], (bf16)v[E0 + 7]};
  return __builtin_bit_cast(uint4, o);
}

// Probabilities (and dS) as the operand of a second product.  Head size 64: rounded to bf16.  Head sizes 32 and 128 (SPLIT): as the
// sum of two bf16 numbers, the value rounded and what the rounding left over, one product each, 16 significant bits in all.  The
// rounding of the bf16 output (2^-9) then hides the operand's (2^-18): over 17 .. 2048 positions the errors against 64 bits are
// those of fp32 operands (o 1.3e-3 .. 1.6e-3, dq, dk, dv 1.6e-3 .. 1.7e-3, lse below 1e-5; operands rounded to bf16: 1.3e-3 ..
// 2.1e-3, 2.0e-3 .. 2.6e-3, 1e-3 .. 4e-3).
template <int DH> constexpr bool split_p() { return DH != 64; }
template <bool SPLIT> struct PFrag { uint4 hi; };
template <> struct PFrag<true> { uint4 hi, lo; };
template <bool SPLIT, int E0> __device__ __forceinline__ PFrag<SPLIT> p_frag(const f32x16& v) {
  PFrag<SPLIT> p;
  p.hi = pack8<E0>(v);
  if constexpr (SPLIT) {
    const bf16x8 hi = __builtin_bit_cast(bf16x8, p.hi);
    bf16x8 lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) lo[e] = (bf16)(v[E0 + e] - (float)hi[e]);
    p.lo = __builtin_bit_cast(uint4, lo);
  }
  return p;
}
template <bool SPLIT> __device__ __forceinline__ f32x16 mfma_p(const uint4& a, const PFrag<SPLIT>& p, f32x16 c) {
  if constexpr (SPLIT) c = mfma16(a, p.lo, c);
  return mfma16(a, p.hi, c);
}

__device__ __forceinline__ int swz64(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

// ---- global memory -> LDS -----------------------------------------------------------------------------------
__device__ __forceinline__ void load4_to_lds(const float* gptr, uint32_t lds_addr) {   // lane l writes bytes [4 l, 4 l + 4)
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dword %0, off" ::"v"(gptr), "s"(lds_addr) : "memory");
}
// This wave's loads of every stage but the n newest have landed; LPW = loads per wave and stage.  (The loads are
// invisible to the compiler, so the count is kept by hand; loads the compiler issues itself only ever make these
// waits longer, never shorter, because the counter is decremented in issue order.)
template <int LPW> __device__ __forceinline__ void wait_stages_but(int n) {
  if (n >= 3) wait_vmcnt<3 * LPW>();
  else if (n == 2) wait_vmcnt<2 * LPW>();
  else if (n == 1) wait_vmcnt<LPW>();
  else wait_vmcnt<0>();
}

// This wave's share of the loads of a stage made of two tiles of 64 x DH: a panel is eight wave-level loads (each fills 8
// of its rows = 1024 LDS bytes).  Load i of wave w is number j = w + 4i: panel j / 8 (the first tile's panels, then the
// second's), rows 8 (j % 8) .. + 7 of it.
// A lane keeps a 32-bit byte offset (its row and 16-byte chunk inside a tile that starts at the operand's row 0) per
// operand and 32 rows: the tile's first row and the panel move the wave-uniform base, so a stage costs four vector
// registers whatever the head size.
template <int DH> struct StageLoader { uint32_t off[4]; };   // [operand][which of the wave's two row groups]
__device__ __forceinline__ int loader_row(int i, int wave, int lane) { return 8 * ((wave + 4 * i) & 7) + (lane >> 3); }
template <int DH> __device__ __forceinline__ uint32_t loader_column_bytes(int i, int wave, int lane) {
  int c = (lane & 7) ^ swz64(loader_row(i, wave, lane));
  if (DH == 32) c &= 3;
  return (uint32_t)(c * 16);
}
template <int DH> __device__ __forceinline__ StageLoader<DH> make_loader(long ld0, long ld1, int wave, int lane) {
  StageLoader<DH> L;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    L.off[i] = (uint32_t)(loader_row(i & 1, wave, lane) * (i < 2 ? ld0 : ld1) * 2) + loader_column_bytes<DH>(i & 1, wave, lane);
  return L;
}
// tile0 / tile1: the two operands (row 0 of this sequence and head), ld0 / ld1 their row strides in elements.
// Rows at or beyond rows_total re-read the last valid row: callers give such rows zero weight (masked
// probabilities, -inf statistics), so any finite value will do, and no branch surrounds a load.  Only the last
// tile of an operand can stick out; every other tile only moves the wave-uniform base.
// Byte offsets are 32-bit: rows_total * row stride * 2 stays below 2^32 (checked by the launchers).
template <int DH>
__device__ __forceinline__ void issue_stage(const StageLoader<DH>& L, const bf16* tile0, const bf16* tile1, int row0,
                                            int rows_total, long ld0, long ld1, int wave, int lane, uint32_t stage_addr) {
  constexpr int NP = panels<DH>();
  if (row0 + 64 <= rows_total) {   // wave-uniform
    const bf16* const b0 = tile0 + (long)row0 * ld0;
    const bf16* const b1 = tile1 + (long)row0 * ld1;
#pragma unroll
    for (int i = 0; i < 4 * NP; ++i) {
      const int second = i / (2 * NP), panel = (i >> 1) % NP;   // compile-time
      load16_to_lds_at((second ? b1 : b0) + 64 * panel, L.off[2 * second + (i & 1)], stage_addr + (uint32_t)((wave + 4 * i) * 1024));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4 * NP; ++i) {
      const int second = i / (2 * NP), panel = (i >> 1) % NP;
      const int r = min(row0 + loader_row(i, wave, lane), rows_total - 1);
      load16_to_lds_at((second ? tile1 : tile0) + 64 * panel,
                       (uint32_t)r * (uint32_t)((second ? ld1 : ld0) * 2) + loader_column_bytes<DH>(i, wave, lane),
                       stage_addr + (uint32_t)((wave + 4 * i) * 1024));
    }
  }
}

// ---- fragment reads -----------------------------------------------------------------------------------------
// Row-index reads.  Lane l reads row 32*t + r (r = l%32), chunk (2*ks + h) ^ swz(row), h = l/32; swz does not
// depend on t (it uses bits 1..3 of the row).  b[ks]: byte offset for t = 0; add 4096*t.
struct FragOff { int b[4]; };
__device__ __forceinline__ FragOff frag_offsets(int lane) {
  const int r = lane & 31, h = lane >> 5, s = swz64(r);
  FragOff f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) f.b[ks] = r * TILE_ROW_BYTES + (((2 * ks + h) ^ s) << 4);
  return f;
}
// K step ks (16 columns) of rows 32 t .. + 31 of a tile: panel ks / 4
__device__ __forceinline__ uint4 row_frag(const char* tile, const FragOff& fo, int ks, int t) {
  return *reinterpret_cast<const uint4*>(tile + (ks >> 2) * PANEL_BYTES + fo.b[ks & 3] + 4096 * t);
}

// Column-index (transposing) reads.  For output columns 32*dt .. + 31 and the 16 tile rows 32*t + 16*g2 .. + 15,
// read p (0 / 1) of lane l = 16*g4 + 4*e + q fetches columns 32*dt + 16*(g4 & 1) + 4q .. + 3 of tile row
// 32*t + 16*g2 + 8p + 4*(g4 >> 1) + e, and the two reads together give the lane its column's values in tile rows
// 4h + 0..3, 8 + 4h + 0..3 of the group (h = l/32): the order of accumulator elements 8*g2 .. 8*g2 + 7.
// b[dt][p]: byte offset for t = g2 = 0; add (32*t + 16*g2) * 128.
struct TrOff { int b[2][2]; };
__device__ __forceinline__ TrOff tr_offsets(int lane) {
  const int g4 = lane >> 4, e = (lane & 15) >> 2, q = lane & 3, h = g4 >> 1;
  TrOff t;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int row = 8 * p + 4 * h + e;
      const int chunk = (4 * dt + 2 * (g4 & 1) + (q >> 1)) ^ swz64(row);
      t.b[dt][p] = row * TILE_ROW_BYTES + (chunk << 4) + ((q & 1) << 3);
    }
  return t;
}
__device__ __forceinline__ uint4 tr_read(const char* tile, const TrOff& to, int dt, int rows16) {
  const char* base = tile + (dt >> 1) * PANEL_BYTES + rows16 * 16 * TILE_ROW_BYTES;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(uintptr_t)(uint32_t)(uintptr_t)(base + to.b[dt & 1][0]));
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(uintptr_t)(uint32_t)(uintptr_t)(base + to.b[dt & 1][1]));
  uint4 o;
  o.x = (uint16_t)lo[0] | ((uint32_t)(uint16_t)lo[1] << 16);
  o.y = (uint16_t)lo[2] | ((uint32_t)(uint16_t)lo[3] << 16);
  o.z = (uint16_t)hi[0] | ((uint32_t)(uint16_t)hi[1] << 16);
  o.w = (uint16_t)hi[2] | ((uint32_t)(uint16_t)hi[3] << 16);
  return o;
}
// The same offsets formed anew from one of each kind (an XOR apiece) instead of kept: seven registers less through a
// loop that has none to spare.  The opaque copies keep the compiler from forming them once, in front of the loop.
__device__ __forceinline__ void rederive_offsets(FragOff& fo, TrOff& to) {
  int f = fo.b[0], t = to.b[0][0];
  asm volatile("" : "+v"(f), "+v"(t));
#pragma unroll
  for (int ks = 1; ks < 4; ++ks) fo.b[ks] = f ^ (32 * ks);
  fo.b[0] = f;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int p = 0; p < 2; ++p) to.b[dt][p] = (t ^ (64 * dt) ^ (32 * p)) + 8 * TILE_ROW_BYTES * p;
}
// acc^T[dt] += (tile^T)[columns 32 dt.., rows 32 (T0 + t)..] . src[t]   for NT accumulator tiles src of 32 tile rows each
template <int DT, int NT>
__device__ __forceinline__ void mma_transposed(f32x16 (&acc)[DT], const char* tile, const TrOff& to, const f32x16 (&src)[NT], int t0) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if constexpr (split_p<32 * DT>()) {   // half a fragment at a time: a packed half takes the registers of the values it came from
      const auto p0 = p_frag<true, 0>(src[t]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * (t0 + t)), p0, acc[dt]);
      const auto p1 = p_frag<true, 8>(src[t]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * (t0 + t) + 1), p1, acc[dt]);
    } else {
      const auto p0 = p_frag<false, 0>(src[t]), p1 = p_frag<false, 8>(src[t]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * (t0 + t)), p0, acc[dt]);
        acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * (t0 + t) + 1), p1, acc[dt]);
      }
    }
  }
}

// The same with the probabilities already packed: pk[t][0 / 1] = p_frag<.., 0 / 8>(src[t]).
template <int DT>
__device__ __forceinline__ void mma_transposed_packed(f32x16 (&acc)[DT], const char* tile, const TrOff& to,
                                                      const PFrag<split_p<32 * DT>()> (&pk)[2][2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * t), pk[t][0], acc[dt]);
      acc[dt] = mfma_p(tr_read(tile, to, dt, 2 * t + 1), pk[t][1], acc[dt]);
    }
}
// acc + the eight bf16 values of v, two per instruction (v_dot2c_f32_bf16 with a vector of ones: products with 1 and
// the fp32 additions are exact operations on the rounded values, the ones the matrix core then multiplies)
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float add8_bf16(float acc, const uint4& v) {
  const bf16x2 ones = {(bf16)1.0f, (bf16)1.0f};
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.x), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.y), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.z), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.w), ones, acc, false);
  return acc;
}

// l + this lane's sixteen probabilities: what the second product multiplies with
template <bool SPLIT>
__device__ __forceinline__ float add_row_sum(float l, const f32x16& p, const PFrag<SPLIT>& p0, const PFrag<SPLIT>& p1) {
  if constexpr (SPLIT) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) s += p[e];
    return l + s;
  } else {
    return add8_bf16(add8_bf16(l, p0.hi), p1.hi);
  }
}

// store 4 consecutive head columns (accumulator elements 4g..4g+3 of a transposed-output tile) as bf16
__device__ __forceinline__ void store4(bf16* dst, const f32x16& v, int g, float scale) {
  bf16x4 o = {(bf16)(v[4 * g + 0] * scale), (bf16)(v[4 * g + 1] * scale), (bf16)(v[4 * g + 2] * scale),
              (bf16)(v[4 * g + 3] * scale)};
  *reinterpret_cast<bf16x4*>(dst) = o;
}
// out^T tiles ot[dt] hold head column 32*dt + 8*g + 4*h + (0..3) for this lane's row
template <int DT> __device__ __forceinline__ void store_transposed_out(bf16* row_ptr, const f32x16 (&ot)[DT], int h, float scale) {
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) store4(row_ptr + 32 * dt + 8 * g + 4 * h, ot[dt], g, scale);
}

// v + (v of the lane that the DPP control selects); rows outside row_mask add 0.  Pure VALU: no LDS traffic.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_add(float v) {
  const int t = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false);
  return v + __builtin_bit_cast(float, t);
}
// Sum over each half of the wave (lanes 0..31, lanes 32..63); the result is valid in lanes 16..31 and 48..63.
__device__ __forceinline__ float half_wave_sum(float v) {
  v = dpp_add<0xb1, 0xf>(v);    // quad_perm [1,0,3,2]
  v = dpp_add<0x4e, 0xf>(v);    // quad_perm [2,3,0,1]: every lane holds its quad's sum
  v = dpp_add<0x141, 0xf>(v);   // row_half_mirror: sums of 8
  v = dpp_add<0x140, 0xf>(v);   // row_mirror: sums of 16
  v = dpp_add<0x142, 0xa>(v);   // row_bcast15 into rows 1 and 3: sums of 32
  return v;
}

// Column sums of a block's 128 rows of a transposed-output tile pair (the bias gradient of the projection whose
// output gradient the block is): every lane adds scale * its values over the 32 rows of its wave, the four waves'
// sums are added in wave order, and the 32 DT sums go to out.
// red: LDS [4][32 DT].  All waves of the workgroup call it; rows with valid = false count as zero.
template <int DT> __device__ __forceinline__ void block_column_sums(const f32x16 (&ot)[DT], float scale, bool valid, float (*red)[32 * DT],
                                                  float* __restrict__ out, int grp, int wave, int lane) {
  const int h = lane >> 5;
#pragma unroll
  for (int dt = 0; grp == 0 && dt < DT; ++dt)   // the second group has handed its sums over
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float v = half_wave_sum(valid ? ot[dt][k] * scale : 0.f);
      if ((lane & 31) == 31) red[wave][32 * dt + 8 * (k >> 2) + 4 * h + (k & 3)] = v;
    }
  __syncthreads();
  if (threadIdx.x < 32 * DT) {
    const int c = threadIdx.x;
    out[c] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
  }
  __syncthreads();   // red is reused by the workgroup's next block
}

// ---- two groups of waves -----------------------------------------------------------------------------------------
// Where a launch has few blocks, the causal triangle's longest one is its length, on four waves of a compute unit that holds
// little else.  There a block gets two groups of four waves (NG = 2), each with a ring of its own, that take its tiles in turn;
// at the end the second group hands its sums over through LDS.  A workgroup then fills its compute unit, so the blocks' tiles
// (nqb + 1 on the mean, 2 nqb in the longest) have to be fewer than 0.9 of the chip's in that time, and four blocks long or more to repay the
// hand-over.  Us forward | backward with one -> two groups, head size 64: 42 heads x 1000 (336 blocks) 21.0 -> 18.5 | 57.9 -> 52.7, 28 x 1900
// (420) 39.0 -> 29.6 | 95.7 -> 81.0, 4 x 2048 30.0 -> 22.9 | 81 -> 63, 64 x 512 (256) 11.3 -> 10.7 | 31.5 -> 30.1; head size 128: 42 x 1000
// 34.6 -> 32.1 | 136 -> 109, 64 x 512 18.7 -> 18.3 | 70 -> 63, 14 x 2048 55 -> 46 | 226 -> 159.  Beyond the rule: 112 x 512 (448) 13.4 -> 15.8 |
// 38.8 -> 45.0, 42 x 1900 (630) 37.3 -> 43.9 | 114 -> 125, 56 x 256 8.0 -> 8.1 | 20.0 -> 20.4.
inline bool two_groups(int B, int H, int S) {
  const long nqb = (S + 127) / 128, blocks = (long)B * H * nqb;
  return nqb >= 4 && 10 * blocks * (nqb + 1) <= 9 * 512 * nqb;
}
// dQ and dK / dV in one launch, behind one that takes their statistics (4 us): each alone ends with its longest blocks, on
// compute units that hold little else; together the one's blocks run beside the other's.  us, two launches -> one: 42 heads x 1000 x 64 50.7 -> 42.0, 64 x 512 x
// 128 62.6 -> 53.0, 16 x 900 x 64 36.1 -> 24.2, 24 x 180 x 64 15.5 -> 12.0, 512 x 512 x 64 146 -> 130, 1792 x 256 x 64 215 -> 195, x 32 136 -> 133.
// Ahead up to 1152 blocks at every head size and 5 to 32 blocks a sequence (1 - 23 %), and up to four blocks a sequence.  Above, dQ and dK / dV fill
// the chip alone, and long sequences of narrow heads are behind (dQ alone has three waves a SIMD, not two; head size 32 has three for dK / dV too):
// 1536 | 2048 | 2560 blocks of sequences of 16 at head size 32 +1.6 | +4.4 | +5.1 %, 64 +3.7 | +6.1 | +5.5, 128 -1.4 | -1.5 | +0.5; of 12 at 64 +2.1 | -0.2 |
// -1.1; of 8 at 32 -0.7 | +0.1 | -0.1, 64 -2.2 | +2.6 | -3.4, 128 -6.1 | -6.5 | -3.3; of 5 at 32 -4.0 | -1.3 | -0.8; 3072 of 8 at 64 -1.6, 128 -2.2.
template <int DH> inline bool bwd_one_launch(int B, int H, int S) {
  const long nqb = (S + 127) / 128, blocks = (long)B * H * nqb;
  return nqb <= 4 || blocks <= 1280 || (blocks <= 3072 && nqb <= (DH == 32 ? 5 : DH == 64 ? 8 : 16));
}
// Two groups a block there while that is less than a workgroup of each kind a compute unit: one | two groups 14 x 1900 x 64 54.9 | 44.0, 14 x 2048 x 128
// 135 | 105, 16 x 900 x 64 28.0 | 24.2, 32 x 384 x 32 14.3 | 13.1; 64 x 512 (256 blocks) x 64 22.0 | 23.3, x 128 53.2 | 53.8; 42 x 1000 42.0 | 48.0; of two
// blocks 24 x 180 x 64 12.0 | 12.3.
inline bool one_launch_two_groups(int B, int H, int S) {
  const long nqb = (S + 127) / 128;
  return nqb >= 3 && (long)B * H * nqb < 256;
}
template <int N> __device__ __forceinline__ void hand_over(const f32x16 (&v)[N], float* at, int lane) {   // at: this wave's 16 N x 64 floats
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(at + ((n * 4 + g) * WAVE + lane) * 4) = make_float4(v[n][4 * g], v[n][4 * g + 1], v[n][4 * g + 2], v[n][4 * g + 3]);
}
// v = a v + b (what was handed over)
template <int N> __device__ __forceinline__ void take_over(f32x16 (&v)[N], const float* at, float a, float b, int lane) {
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 w = *reinterpret_cast<const float4*>(at + ((n * 4 + g) * WAVE + lane) * 4);
      v[n][4 * g] = v[n][4 * g] * a + w.x * b;
      v[n][4 * g + 1] = v[n][4 * g + 1] * a + w.y * b;
      v[n][4 * g + 2] = v[n][4 * g + 2] * a + w.z * b;
      v[n][4 * g + 3] = v[n][4 * g + 3] * a + w.w * b;
    }
}

// ---- forward ---------------------------------------------------------------------------------------------------
constexpr int FWD_STAGES = 2, DQ_STAGES = 2, DKV_STAGES = 2;   // three stages measured: forward level, backward 4 % slower

template <int DH, int NG>
__global__ void __launch_bounds__(AT_THREADS * NG, NG == 2 || DH == 128 ? 2 : 3) attn_fwd_mfma(const bf16* __restrict__ qkv, bf16* __restrict__ o,
                                                               float* __restrict__ lse, int S, int H, int single) {
  constexpr int NS = FWD_STAGES, KS = DH / 16, DT = DH / 32, TILE_BYTES = tile_bytes<DH>(), LPW = 4 * panels<DH>();
  extern __shared__ __attribute__((aligned(16))) char fwd_smem[];   // [group][stage][K | V]
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = NG == 1 ? 0 : wave_all >> 2, wave = NG == 1 ? wave_all : wave_all & 3;
  char (*smem)[2][TILE_BYTES] = reinterpret_cast<char (*)[2][TILE_BYTES]>(fwd_smem) + grp * NS;
  const int r = lane & 31, h = lane >> 5;
  const int bh = single ? blockIdx.x : blockIdx.y, b = bh / H, hd = bh % H;
  const int bx = single ? (int)blockIdx.y : (int)blockIdx.x;   // single: one block per workgroup, longest first
  const int A = H * DH;
  const long ld = 3L * A;
  const bf16* base = qkv + (long)b * S * ld + hd * DH;
  const FragOff fo = frag_offsets(lane);
  const TrOff to = tr_offsets(lane);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)fwd_smem + grp * NS * 2 * TILE_BYTES;
  const StageLoader<DH> L = make_loader<DH>(ld, ld, wave, lane);
  const bf16* const ktile = base + A;
  const bf16* const vtile = base + 2 * A;
  // A workgroup takes a long and a short query block (block x from the end, then block x from the start), so that
  // every workgroup walks the same number of tiles whatever the causal triangle gives its blocks.
  const int nqb = (S + 127) / 128;
  for (int pass = 0; pass < 2; ++pass) {
  const int qb = pass == 0 ? nqb - 1 - bx : bx;
  if (pass == 1) {
    if (single || qb >= nqb - 1 - bx) break;      // the middle block of an odd count was done in the first pass
    __syncthreads();                              // the stages are reused
  }
  const int q0 = qb * 128, qw0 = q0 + 32 * wave, q = qw0 + r;

  uint4 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = q < S ? *reinterpret_cast<const uint4*>(base + (long)q * ld + 8 * (2 * ks + h)) : make_uint4(0, 0, 0, 0);

  const int kv_end = min(S, q0 + 128);
  const int ntiles = (kv_end + 63) / 64;
  f32x16 ot[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) zero(ot[dt]);
  float m = -INFINITY, l = 0.f;
  const float sc = score_scale<DH>() * LOG2E;   // base-2 exponentials

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (grp + NG * s < ntiles) issue_stage(L, ktile, vtile, (grp + NG * s) * 64, S, ld, ld, wave, lane, smem_addr + s * 2 * TILE_BYTES);
  static_assert(NS == 2 || NS == 3, "the tile loop below is unrolled over the stages, so that every LDS offset is a constant");
  // one key / value tile; CUR: the stage it sits in
  auto tile = [&](auto CUR, int kt) {
    constexpr int cur = decltype(CUR)::value;
    wait_stages_but<LPW>(min(NS - 2, (ntiles - 1 - kt) / NG));
    __syncthreads();   // tile kt is in LDS; nobody still reads the stage of tile kt - 1, which is refilled now
    if (kt + NG * (NS - 1) < ntiles)
      issue_stage(L, ktile, vtile, (kt + NG * (NS - 1)) * 64, S, ld, ld, wave, lane, smem_addr + (cur == 0 ? NS - 1 : cur - 1) * 2 * TILE_BYTES);
    const int kv0 = kt * 64;
    if (kv0 <= qw0 + 31 && (NG == 1 || kt < ntiles)) {   // wave-uniform: at least one query of this wave sees this tile
      const char* k_ = smem[cur][0];
      const char* v_ = smem[cur][1];
      f32x16 st[2];
      zero(st[0]); zero(st[1]);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < 2; ++t) st[t] = mfma16(row_frag(k_, fo, ks, t), qf[ks], st[t]);
      if (kv0 + 63 > qw0) {   // wave-uniform: the tile crosses the diagonal of some query
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (kv0 + 32 * t + acc_row(e, lane) > q) st[t][e] = -INFINITY;
      }
      float mx = fmaxf(st[0][0], st[1][0]);
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(fmaxf(mx, st[0][e]), st[1][e]);   // one three-input maximum each
      mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
      // The reference exponent m only has to stay within 2^8 of the true running maximum (probabilities then stay
      // below 256, harmless in fp32 sums and in bf16 operands, and the final O / l and lse do not depend on the
      // reference): the accumulators are rescaled only when some query's maximum outgrows it by more than that.
      const float mn = fmaxf(m, mx * sc);   // finite: key 0 is visible to every query
      if (__builtin_amdgcn_ballot_w64(mn > m + 8.0f) != 0) {   // wave-uniform
        const float corr = __builtin_amdgcn_exp2f(m - mn);
        l *= corr;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) ot[dt][e] *= corr;
        m = mn;
      }
      // probabilities.  Head size 64: rounded to bf16 once: the rounded values are both what the matrix core multiplies with V
      // and what the row sum adds up (two per instruction), so numerator and denominator of the softmax agree exactly.
      // l is this lane's half of the row (keys 4h + 0..3 of every eight); the halves meet after the last tile.
      PFrag<split_p<DH>()> pk[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int e = 0; e < 16; ++e) st[t][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][e], sc, -m));
        pk[t][0] = p_frag<split_p<DH>(), 0>(st[t]);
        pk[t][1] = p_frag<split_p<DH>(), 8>(st[t]);
        l = add_row_sum(l, st[t], pk[t][0], pk[t][1]);
      }
      mma_transposed_packed(ot, v_, to, pk);
    }
  };
  for (int kt = 0; kt < ntiles; kt += NG * NS) {   // both groups walk as often as the first: the barriers are the workgroup's
    tile(std::integral_constant<int, 0>{}, kt + grp);
    if (kt + NG < ntiles) tile(std::integral_constant<int, 1>{}, kt + NG + grp);
    if (NS > 2 && kt + 2 * NG < ntiles) tile(std::integral_constant<int, NS - 1>{}, kt + 2 * NG + grp);
  }
  if constexpr (NG == 2) {
    constexpr int PER = (16 * DT + 2) * WAVE;   // floats a wave hands over: O^T, the reference exponent, the half row sum
    static_assert(4 * PER * 4 <= NG * NS * 2 * TILE_BYTES, "the sums fit in the rings");
    float* const at = reinterpret_cast<float*>(fwd_smem) + wave * PER;
    __syncthreads();   // the rings have been read
    if (grp == 1) {
      hand_over(ot, at, lane);
      at[16 * DT * WAVE + lane] = m;
      at[(16 * DT + 1) * WAVE + lane] = l;
    }
    __syncthreads();
    if (grp == 1) continue;
    const float m1 = at[16 * DT * WAVE + lane], mn = fmaxf(m, m1);   // m is finite: key 0 is the first group's
    const float c0 = __builtin_amdgcn_exp2f(m - mn), c1 = __builtin_amdgcn_exp2f(m1 - mn);
    l = l * c0 + at[(16 * DT + 1) * WAVE + lane] * c1;
    take_over(ot, at, c0, c1, lane);
    m = mn;
  }
  l += __shfl_xor(l, 32, WAVE);
  if constexpr (split_p<DH>()) {
    if (__any(q < S && plain::not_finite(ot)) && q < S)
      plain::attend<DH>(ot, base, ld, A, q, h, [&](float s) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, sc, -m)); });
  }
  // the output addresses are formed from here on (an opaque copy of the row index: formed before the loop they would
  // sit in sixteen registers through it)
  int q_out = q;
  asm volatile("" : "+v"(q_out));
  if (q_out < S) {
    store_transposed_out(o + ((long)b * S + q_out) * A + hd * DH, ot, h, 1.0f / l);
    if (h == 0) lse[(long)bh * S + q_out] = (m + __builtin_amdgcn_logf(l)) * LN2;   // v_log_f32 is log2
  }
  }
}

// ---- forward, sequences of up to 32 positions (routing prefixes) ---------------------------------------------------
// One query block of the kernel above is 128 queries of four waves: with 32 positions three of them idle, 64 rows are
// staged and a barrier waits for every tile.  Here a wave owns one sequence and head: it brings its Q, K and V rows into
// its own part of LDS (whole 128-byte lines; no barrier), multiplies, and sends O back through LDS so that it leaves in
// 16-byte row-contiguous stores.  Same arithmetic in the same order.  Bound by the bytes of qkv and o: 8192 documents x 14
// heads x 32 x 64 (1.88 GB) 601 us in the kernel above, 355 here (5.3 TB/s).
constexpr int SHORT_ROWS = 32;
constexpr int SHORT_TILE = SHORT_ROWS * TILE_ROW_BYTES;   // 32 rows of one panel
template <int DH> constexpr int short_wave_bytes() { return panels<DH>() == 1 ? 3 * SHORT_TILE : 2 * PANEL_BYTES + PANEL_BYTES + SHORT_TILE; }

template <int DH>
__global__ void __launch_bounds__(AT_THREADS, DH == 128 ? 1 : 3) attn_fwd_short_mfma(const bf16* __restrict__ qkv, bf16* __restrict__ o,
                                                                      float* __restrict__ lse, int S, int H, int n_bh) {
  constexpr int KS = DH / 16, DT = DH / 32, NP = panels<DH>();
  extern __shared__ __attribute__((aligned(16))) char short_smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bh = blockIdx.x * (AT_THREADS / WAVE) + wave;
  if (bh >= n_bh) return;   // whole waves leave; nothing below involves another wave
  const int r = lane & 31, h = lane >> 5, b = bh / H, hd = bh % H, A = H * DH;
  const long ld = 3L * A;
  const bf16* const base = qkv + (long)b * S * ld + hd * DH;
  // panel p of K, V and Q at PANEL_BYTES p + 0, SHORT_TILE and (behind both panels of K and V) NP PANEL_BYTES
  char* const k_ = short_smem + wave * short_wave_bytes<DH>();
  char* const v_ = k_ + SHORT_TILE;
  char* const q_ = k_ + NP * PANEL_BYTES;
  // load i of an operand's panel: rows 8 i .. 8 i + 7; rows beyond S re-read the last one (masked keys, unstored queries)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * i + (lane >> 3);
    int c = (lane & 7) ^ swz64(row);
    if (DH == 32) c &= 3;
    const uint32_t off = (uint32_t)((min(row, S - 1) * ld + c * 8) * 2);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)k_ + p * PANEL_BYTES + i * 1024);
      load16_to_lds_at(base + 64 * p, off, at + NP * PANEL_BYTES);
      load16_to_lds_at(base + A + 64 * p, off, at);
      load16_to_lds_at(base + 2 * A + 64 * p, off, at + SHORT_TILE);
    }
  }
  const FragOff fo = frag_offsets(lane);
  const TrOff to = tr_offsets(lane);
  wait_vmcnt<0>();
  asm volatile("" ::: "memory");

  f32x16 st;
  zero(st);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) st = mfma16(row_frag(k_, fo, ks, 0), row_frag(q_, fo, ks, 0), st);
#pragma unroll
  for (int e = 0; e < 16; ++e)
    if (acc_row(e, lane) > r) st[e] = -INFINITY;
  float mx = st[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) mx = fmaxf(mx, st[e]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
  const float sc = score_scale<DH>() * LOG2E, m = mx * sc;
#pragma unroll
  for (int e = 0; e < 16; ++e) st[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[e], sc, -m));
  const auto p0 = p_frag<split_p<DH>(), 0>(st), p1 = p_frag<split_p<DH>(), 8>(st);
  float l = add_row_sum(0.f, st, p0, p1);
  f32x16 ot[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    zero(ot[dt]);
    ot[dt] = mfma_p(tr_read(v_, to, dt, 0), p0, ot[dt]);
    ot[dt] = mfma_p(tr_read(v_, to, dt, 1), p1, ot[dt]);
  }
  l += __shfl_xor(l, 32, WAVE);
  if constexpr (split_p<DH>()) {
    if (__any(r < S && plain::not_finite(ot)) && r < S)
      plain::attend<DH>(ot, base, ld, A, r, h, [&](float s) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, sc, -m)); });
  }
  // O^T to LDS as rows of O, in K's place (its reads are done: the scores above needed them), under the tiles' swizzle
  const float scale = 1.0f / l;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int chunk = (4 * dt + g) & 7;
      store4(reinterpret_cast<bf16*>(k_ + (dt >> 1) * PANEL_BYTES + r * TILE_ROW_BYTES + ((chunk ^ swz64(r)) << 4) + 8 * h), ot[dt], g, scale);
    }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * i + (lane >> 3), c = (lane & 7) ^ swz64(row);
    if (row < S && (DH > 32 || c < 4)) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<uint4*>(o + ((long)b * S + row) * A + hd * DH + 64 * p + 8 * c) =
            *reinterpret_cast<const uint4*>(k_ + p * PANEL_BYTES + row * TILE_ROW_BYTES + 16 * (lane & 7));
    }
  }
  if (h == 0 && r < S) lse[(long)bh * S + r] = (m + __builtin_amdgcn_logf(l)) * LN2;   // v_log_f32 is log2
}

// ---- backward: D = rowsum(dO * O) and -lse log2(e) of every query ------------------------------------------------------
// For the dQ and the dK / dV blocks, in rows padded to whole query blocks: D is 0 and -lse log2(e) is -inf (probability 0) beyond S, so that those
// need neither a bounds check nor a rescale.  One workgroup a block of 128 queries of a head.
template <int DH>
__global__ void __launch_bounds__(AT_THREADS) attn_stats_mfma(const bf16* __restrict__ o, const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                             float* __restrict__ dsum, int S, int H) {
  constexpr int LANES = DH / 8, ROWS = WAVE / LANES;   // lanes of a query, queries of a wave at a time
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, bh = blockIdx.x, b = bh / H, hd = bh - b * H;
  const long Sp = (long)gridDim.y * 128;
  const int c = 8 * (lane % LANES);
#pragma unroll
  for (int i = 0; i < 32 / ROWS; ++i) {
    const int q = blockIdx.y * 128 + 32 * wave + ROWS * i + lane / LANES;
    float D = 0.f;
    if (q < S) {
      const size_t at = ((size_t)b * S + q) * H * DH + hd * DH + c;
      const uint4 gv = *reinterpret_cast<const uint4*>(d_o + at), ov = *reinterpret_cast<const uint4*>(o + at);
      const bf16* gp = reinterpret_cast<const bf16*>(&gv);
      const bf16* op = reinterpret_cast<const bf16*>(&ov);
#pragma unroll
      for (int e = 0; e < 8; ++e) D += (float)gp[e] * (float)op[e];
    }
#pragma unroll
    for (int m = 1; m < LANES; m <<= 1) D += __shfl_xor(D, m, WAVE);
    if (lane % LANES == 0) {
      dsum[bh * Sp + q] = D;
      dsum[(gridDim.x + bh) * Sp + q] = q < S ? -lse[(long)bh * S + q] * LOG2E : -INFINITY;
    }
  }
}

// ---- backward, dQ ---------------------------------------------------------------------------------------------------
// STATS: attn_stats_mfma has written dsum; else this takes D itself and leaves both for the dK / dV kernel
template <int DH, int NG, bool STATS>
__device__ __forceinline__ void dq_blocks(const bf16* __restrict__ qkv, const bf16* __restrict__ o, const bf16* __restrict__ d_o,
                                          const float* __restrict__ lse, bf16* __restrict__ dqkv, float* __restrict__ dsum,
                                          float* __restrict__ colsum, int S, int H, int single, int bh, int n_bh, int bx) {
  constexpr int NS = DQ_STAGES, KS = DH / 16, DT = DH / 32, TILE_BYTES = tile_bytes<DH>(), LPW = 4 * panels<DH>();
  __shared__ float cs_red[4][DH];
  extern __shared__ __attribute__((aligned(16))) char dq_smem[];   // [group][stage][K | V]
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = NG == 1 ? 0 : wave_all >> 2, wave = NG == 1 ? wave_all : wave_all & 3;
  char (*smem)[2][TILE_BYTES] = reinterpret_cast<char (*)[2][TILE_BYTES]>(dq_smem) + grp * NS;
  const int r = lane & 31, h = lane >> 5;
  const int b = bh / H, hd = bh % H;
  const int A = H * DH;
  const long ld = 3L * A;
  const bf16* base = qkv + (long)b * S * ld + hd * DH;
  const FragOff fo = frag_offsets(lane);
  const TrOff to = tr_offsets(lane);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)dq_smem + grp * NS * 2 * TILE_BYTES;
  const StageLoader<DH> L = make_loader<DH>(ld, ld, wave, lane);
  const bf16* const ktile = base + A;
  const bf16* const vtile = base + 2 * A;
  const int nqb = (S + 127) / 128;
  for (int pass = 0; pass < 2; ++pass) {   // a long and a short query block per workgroup (see the forward kernel)
  const int qb = pass == 0 ? nqb - 1 - bx : bx;
  if (pass == 1) {
    if (single || qb >= nqb - 1 - bx) break;
    __syncthreads();
  }
  const int q0 = qb * 128, qw0 = q0 + 32 * wave, q = qw0 + r;

  uint4 qf[KS], gf[KS];
  float D = 0.f;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int c = 8 * (2 * ks + h);
    if (q < S) {
      qf[ks] = *reinterpret_cast<const uint4*>(base + (long)q * ld + c);
      gf[ks] = *reinterpret_cast<const uint4*>(d_o + ((long)b * S + q) * A + hd * DH + c);
      if constexpr (!STATS) {
        const uint4 ov = *reinterpret_cast<const uint4*>(o + ((long)b * S + q) * A + hd * DH + c);
        const bf16* gp = reinterpret_cast<const bf16*>(&gf[ks]);
        const bf16* op = reinterpret_cast<const bf16*>(&ov);
#pragma unroll
        for (int i = 0; i < 8; ++i) D += (float)gp[i] * (float)op[i];
      }
    } else {
      qf[ks] = make_uint4(0, 0, 0, 0);
      gf[ks] = make_uint4(0, 0, 0, 0);
    }
  }
  const long Sp = (long)nqb * 128;
  float nlse2;
  if constexpr (STATS) {
    D = dsum[bh * Sp + q];
    nlse2 = dsum[(n_bh + bh) * Sp + q];
  } else {
    D += __shfl_xor(D, 32, WAVE);
    nlse2 = q < S ? -lse[(long)bh * S + q] * LOG2E : -INFINITY;
    if (h == 0 && grp == 0) {
      dsum[bh * Sp + q] = q < S ? D : 0.f;
      dsum[(n_bh + bh) * Sp + q] = nlse2;
    }
  }

  const int kv_end = min(S, q0 + 128);
  const int ntiles = (kv_end + 63) / 64;
  f32x16 dqt[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) zero(dqt[dt]);
  const float sc = score_scale<DH>() * LOG2E;

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (grp + NG * s < ntiles) issue_stage(L, ktile, vtile, (grp + NG * s) * 64, S, ld, ld, wave, lane, smem_addr + s * 2 * TILE_BYTES);
  int cur = 0;
  for (int kt = grp; kt - grp < ntiles; kt += NG, cur = cur + 1 == NS ? 0 : cur + 1) {
    wait_stages_but<LPW>(min(NS - 2, (ntiles - 1 - kt) / NG));
    __syncthreads();   // tile kt is in LDS; nobody still reads the stage of tile kt - 1, which is refilled now
    if (kt + NG * (NS - 1) < ntiles)
      issue_stage(L, ktile, vtile, (kt + NG * (NS - 1)) * 64, S, ld, ld, wave, lane, smem_addr + (cur == 0 ? NS - 1 : cur - 1) * 2 * TILE_BYTES);
    const int kv0 = kt * 64;
    if (kv0 <= qw0 + 31 && (NG == 1 || kt < ntiles)) {
      const char* k_ = smem[cur][0];
      const char* v_ = smem[cur][1];
      f32x16 st[2], dp[2];
      zero(st[0]); zero(st[1]); zero(dp[0]); zero(dp[1]);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          st[t] = mfma16(row_frag(k_, fo, ks, t), qf[ks], st[t]);
          dp[t] = mfma16(row_frag(v_, fo, ks, t), gf[ks], dp[t]);
        }
      // dS^T without the 1/sqrt(d_head) factor (applied once when dQ is stored)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          st[t][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][e], sc, nlse2)) * (dp[t][e] - D);
      if (kv0 + 63 > qw0) {   // wave-uniform: the tile crosses the diagonal
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (kv0 + 32 * t + acc_row(e, lane) > q) st[t][e] = 0.f;
      }
      mma_transposed<DT, 2>(dqt, k_, to, st, 0);
    }
  }
  if constexpr (NG == 2) {
    static_assert(4 * 16 * DT * WAVE * 4 <= NG * NS * 2 * TILE_BYTES, "the sums fit in the rings");
    float* const at = reinterpret_cast<float*>(dq_smem) + wave * 16 * DT * WAVE;
    __syncthreads();   // the rings have been read
    if (grp == 1) hand_over(dqt, at, lane);
    __syncthreads();
    if (grp == 0) take_over(dqt, at, 1.0f, 1.0f, lane);
  }
  if constexpr (split_p<DH>()) {
    if (grp == 0 && __any(q < S && plain::not_finite(dqt)) && q < S)
      plain::query_grad<DH>(dqt, base, d_o + ((long)b * S + q) * A + hd * DH, D, ld, A, q, h,
                            [&](float s) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, sc, nlse2)); });
  }
  if (grp == 0 && q < S) store_transposed_out(dqkv + ((long)b * S + q) * ld + hd * DH, dqt, h, score_scale<DH>());
  // one row of partial column sums per (document, query block): [b * nqb + qb][3 A], this head's 64 dQ columns
  if (colsum) block_column_sums(dqt, score_scale<DH>(), q < S, cs_red, colsum + ((long)b * nqb + qb) * ld + hd * DH, grp, wave, lane);
  }
}

// ---- backward, dK and dV ------------------------------------------------------------------------------------------
template <int DH> constexpr int dkv_stage() { return 2 * tile_bytes<DH>() + 2 * 64 * (int)sizeof(float); }   // Q | dO | -lse2 | D

template <int DH, int NG>
__device__ __forceinline__ void dkv_blocks(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o, const float* __restrict__ dsum,
                                           bf16* __restrict__ dqkv, float* __restrict__ colsum, int S, int H, int single, int bh, int n_bh, int bx) {
  constexpr int NS = DKV_STAGES, KS = DH / 16, DT = DH / 32, TILE_BYTES = tile_bytes<DH>(), LPW = 4 * panels<DH>();
  constexpr int DKV_STAGE = dkv_stage<DH>();
  __shared__ float cs_red[4][DH];
  extern __shared__ __attribute__((aligned(16))) char dkv_rings[];   // NS stages of DKV_STAGE bytes per group
  const int tid = threadIdx.x, lane = tid & 63, wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = NG == 1 ? 0 : wave_all >> 2, wave = NG == 1 ? wave_all : wave_all & 3;
  char* const dkv_smem = dkv_rings + grp * NS * DKV_STAGE;
  const int r = lane & 31, h = lane >> 5;
  const int b = bh / H, hd = bh % H;
  const int A = H * DH;
  const long ld = 3L * A;
  const bf16* base = qkv + (long)b * S * ld + hd * DH;
  const bf16* gbase = d_o + (long)b * S * A + hd * DH;
  FragOff fo = frag_offsets(lane);
  TrOff to = tr_offsets(lane);
  const uint32_t smem_addr = (uint32_t)(uintptr_t)dkv_rings + grp * NS * DKV_STAGE;
  const int nkb = (S + 127) / 128;
  const int ntiles = (S + 63) / 64;
  // Statistics of a tile's 64 queries (in rows padded to whole query blocks): waves 0
  // and 2 fetch -lse*log2(e), waves 1 and 3 fetch D, one float per lane; the duplicates keep every wave's count of
  // outstanding loads the same.
  const long Sp = (long)nkb * 128;
  const float* stat_src = dsum + ((wave & 1) ? 0 : (long)n_bh * Sp) + bh * Sp + lane;
  const uint32_t stat_dst = 2 * TILE_BYTES + ((wave & 1) ? 256 : 0);
  const StageLoader<DH> L = make_loader<DH>(ld, A, wave, lane);
  auto issue = [&](int qt, int stage) {
    issue_stage(L, base, gbase, qt * 64, S, ld, A, wave, lane, smem_addr + stage * DKV_STAGE);
    load4_to_lds(stat_src + qt * 64, smem_addr + stage * DKV_STAGE + stat_dst);
  };
  for (int pass = 0; pass < 2; ++pass) {   // an early (long) and a late (short) key block per workgroup
  const int kb = pass == 0 ? bx : nkb - 1 - bx;
  if (pass == 1) {
    if (single || kb <= bx) break;
    __syncthreads();
  }
  const int k0 = kb * 128, kw0 = k0 + 32 * wave, key = kw0 + r;

  uint4 kf[KS], vf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int c = 8 * (2 * ks + h);
    kf[ks] = key < S ? *reinterpret_cast<const uint4*>(base + (long)key * ld + A + c) : make_uint4(0, 0, 0, 0);
    vf[ks] = key < S ? *reinterpret_cast<const uint4*>(base + (long)key * ld + 2 * A + c) : make_uint4(0, 0, 0, 0);
  }
  f32x16 dkt[DT], dvt[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) { zero(dkt[dt]); zero(dvt[dt]); }
  const float sc = score_scale<DH>() * LOG2E;

  const int first = k0 / 64;               // first query tile that can see a key of this block
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (first + grp + NG * s < ntiles) issue(first + grp + NG * s, s);
  int cur = 0;
  for (int qt = first + grp; qt - grp < ntiles; qt += NG, cur = cur + 1 == NS ? 0 : cur + 1) {
    wait_stages_but<LPW + 1>(min(NS - 2, (ntiles - 1 - qt) / NG));
    __syncthreads();
    if (qt + NG * (NS - 1) < ntiles) issue(qt + NG * (NS - 1), cur == 0 ? NS - 1 : cur - 1);
    const int q0 = qt * 64;
    if (q0 + 63 >= kw0 && (NG == 1 || qt < ntiles)) {   // wave-uniform: some query of this tile sees a key of this wave
      const char* q_ = dkv_smem + cur * DKV_STAGE;
      const char* g_ = q_ + TILE_BYTES;
      const float* nlse2s = reinterpret_cast<const float*>(q_ + 2 * TILE_BYTES);
      const float* Ds = nlse2s + 64;
      // TG blocks of 32 queries at a time: with head size 128 the two accumulators and the K / V fragments leave room
      // for one
      constexpr int TG = DH == 128 ? 1 : 2;
#pragma unroll
      for (int t0 = 0; t0 < 2; t0 += TG) {
        if constexpr (TG == 1) rederive_offsets(fo, to);
        f32x16 st[TG], dp[TG];
#pragma unroll
        for (int t = 0; t < TG; ++t) { zero(st[t]); zero(dp[t]); }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int t = 0; t < TG; ++t) {
            st[t] = mfma16(row_frag(q_, fo, ks, t0 + t), kf[ks], st[t]);
            dp[t] = mfma16(row_frag(g_, fo, ks, t0 + t), vf[ks], dp[t]);
          }
        // accumulator elements 4g..4g+3 are queries 32t + 8g + 4h + (0..3): their statistics are 16 contiguous bytes
#pragma unroll
        for (int t = 0; t < TG; ++t)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const float4 Lq = *reinterpret_cast<const float4*>(nlse2s + 32 * (t0 + t) + 8 * g + 4 * h);
            const float4 Dv = *reinterpret_cast<const float4*>(Ds + 32 * (t0 + t) + 8 * g + 4 * h);
            const float Ls[4] = {Lq.x, Lq.y, Lq.z, Lq.w}, Dd[4] = {Dv.x, Dv.y, Dv.z, Dv.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int e = 4 * g + i;
              const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(st[t][e], sc, Ls[i]));
              st[t][e] = p;
              dp[t][e] = p * (dp[t][e] - Dd[i]);   // dS without 1/sqrt(d_head) (applied when dK is stored)
            }
          }
        if (q0 < kw0 + 31) {   // wave-uniform: the tile crosses the diagonal of some key
#pragma unroll
          for (int t = 0; t < TG; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (q0 + 32 * (t0 + t) + acc_row(e, lane) < key) { st[t][e] = 0.f; dp[t][e] = 0.f; }
        }
        mma_transposed<DT, TG>(dvt, g_, to, st, t0);
        mma_transposed<DT, TG>(dkt, q_, to, dp, t0);
      }
    }
  }
  if constexpr (NG == 2) {
    constexpr int PER = 2 * 16 * DT * WAVE;
    static_assert(4 * PER * 4 <= NG * NS * DKV_STAGE, "the sums fit in the rings");
    float* const at = reinterpret_cast<float*>(dkv_rings) + wave * PER;
    __syncthreads();   // the rings have been read
    if (grp == 1) {
      hand_over(dkt, at, lane);
      hand_over(dvt, at + PER / 2, lane);
    }
    __syncthreads();
    if (grp == 0) {
      take_over(dkt, at, 1.0f, 1.0f, lane);
      take_over(dvt, at + PER / 2, 1.0f, 1.0f, lane);
    }
  }
  int key_out = grp == 0 ? key : S;   // as in the forward kernel: output addresses are formed behind the loop
  asm volatile("" : "+v"(key_out));
  if constexpr (split_p<DH>()) {
    const float* const D = dsum + bh * Sp;
    if (__any(key_out < S && (plain::not_finite(dkt) || plain::not_finite(dvt))) && key_out < S)
      plain::key_grads<DH>(dkt, dvt, base, gbase, ld, A, key_out, S, h,
                           [&](float s, int i) { return __builtin_amdgcn_exp2f(__builtin_fmaf(s, sc, D[(long)n_bh * Sp + i])); },
                           [&](int i) { return D[i]; });
  }
  if (key_out < S) {
    bf16* out = dqkv + ((long)b * S + key_out) * ld + hd * DH;
    store_transposed_out(out + A, dkt, h, score_scale<DH>());
    store_transposed_out(out + 2 * A, dvt, h, 1.0f);
  }
  if (colsum) {
    float* cs = colsum + ((long)b * nkb + kb) * ld + hd * DH;
    block_column_sums(dkt, score_scale<DH>(), key < S, cs_red, cs + A, grp, wave, lane);
    block_column_sums(dvt, 1.0f, key < S, cs_red, cs + 2 * A, grp, wave, lane);
  }
  }
}

// one block per workgroup, longest first (single), or a long and a short one
template <int DH, int NG>
__global__ void __launch_bounds__(AT_THREADS * NG, 2) attn_bwd_dq_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ o, const bf16* __restrict__ d_o,
                                                                  const float* __restrict__ lse, bf16* __restrict__ dqkv, float* __restrict__ dsum,
                                                                  float* __restrict__ colsum, int S, int H, int single) {
  dq_blocks<DH, NG, false>(qkv, o, d_o, lse, dqkv, dsum, colsum, S, H, single, single ? blockIdx.x : blockIdx.y, single ? gridDim.x : gridDim.y,
                           single ? (int)blockIdx.y : (int)blockIdx.x);
}
template <int DH, int NG>
__global__ void __launch_bounds__(AT_THREADS * NG, NG == 1 && DH == 32 ? 3 : 2) attn_bwd_dkv_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                                                   const float* __restrict__ dsum, bf16* __restrict__ dqkv,
                                                                   float* __restrict__ colsum, int S, int H, int single) {
  dkv_blocks<DH, NG>(qkv, d_o, dsum, dqkv, colsum, S, H, single, single ? blockIdx.x : blockIdx.y, single ? gridDim.x : gridDim.y,
                     single ? (int)blockIdx.y : (int)blockIdx.x);
}
// Both in one launch, behind attn_stats_mfma: grid (heads, 2 x blocks), longest first
template <int DH, int NG>
__global__ void __launch_bounds__(AT_THREADS * NG, 2) attn_bwd_both_mfma(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o, float* __restrict__ dsum,
                                                                    bf16* __restrict__ dqkv, float* __restrict__ colsum, int S, int H) {
  if (blockIdx.y & 1) dq_blocks<DH, NG, true>(qkv, nullptr, d_o, nullptr, dqkv, dsum, colsum, S, H, 1, blockIdx.x, gridDim.x, blockIdx.y >> 1);
  else dkv_blocks<DH, NG>(qkv, d_o, dsum, dqkv, colsum, S, H, 1, blockIdx.x, gridDim.x, blockIdx.y >> 1);
}

}  // namespace

template <int DH>
dipaco_status launch_attention_fwd_mfma(const bf16* qkv, bf16* o, float* lse, int B, int S, int H, hipStream_t s) {
  if (S <= SHORT_ROWS) {   // whatever the batch: one document 4.2 -> 3.1 us, 8192 documents 601 -> 355 us
    constexpr int LDS = (AT_THREADS / WAVE) * short_wave_bytes<DH>();
    static std::atomic<unsigned long long> lds_set{0};
    if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_fwd_short_mfma<DH>), LDS, lds_set)) return st;
    const int n_bh = B * H;
    attn_fwd_short_mfma<DH><<<(n_bh + 3) / 4, AT_THREADS, LDS, s>>>(qkv, o, lse, S, H, n_bh);
    DIPACO_LAUNCH_CHECK();
    return DIPACO_OK;
  }
  const int single = attention_single_block();
  const int nqb = (S + 127) / 128;   // more than 32 positions: at most 2^32 / (33 * 3 * 32) sequences x heads, one launch
  dim3 grid = single ? dim3(B * H, nqb) : dim3((nqb + 1) / 2, B * H);   // one or two query blocks per workgroup
  auto run = [&](auto NGc) -> dipaco_status {
    constexpr int NG = decltype(NGc)::value, LDS = NG * FWD_STAGES * 2 * tile_bytes<DH>();
    static std::atomic<unsigned long long> lds_set{0};
    if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_fwd_mfma<DH, NG>), LDS, lds_set)) return st;
    attn_fwd_mfma<DH, NG><<<grid, AT_THREADS * NG, LDS, s>>>(qkv, o, lse, S, H, single);
    DIPACO_LAUNCH_CHECK();
    return DIPACO_OK;
  };
  return two_groups(B, H, S) ? run(std::integral_constant<int, 2>{}) : run(std::integral_constant<int, 1>{});
}

template <int DH>
dipaco_status launch_attention_bwd_mfma(const bf16* qkv, const bf16* o, const bf16* d_o, const float* lse, bf16* dqkv,
                                        float* dsum, float* colsum_out, float* colsum_partial, int B, int S, int H,
                                        hipStream_t s, SumBatch* batch) {
  const int single = attention_single_block();
  const int nqb = (S + 127) / 128;
  const bool one = single && bwd_one_launch<DH>(B, H, S);
  const size_t A = (size_t)H * DH;
  const int step = attention_launch_batch(B, H);
  auto run = [&](auto NGc) -> dipaco_status {
    constexpr int NG = decltype(NGc)::value, DQ_LDS = NG * DQ_STAGES * 2 * tile_bytes<DH>(), DKV_LDS = NG * DKV_STAGES * dkv_stage<DH>();
    static std::atomic<unsigned long long> dq_lds{0}, dkv_lds{0};
    if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_dq_mfma<DH, NG>), DQ_LDS, dq_lds)) return st;
    if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_dkv_mfma<DH, NG>), DKV_LDS, dkv_lds)) return st;
    for (int b = 0; b < B; b += step) {
      const size_t row = (size_t)b * S;
      const int n_bh = std::min(step, B - b) * H;
      dim3 grid = single ? dim3(n_bh, nqb) : dim3((nqb + 1) / 2, n_bh);   // one or two query (key) blocks per workgroup
      float* const cs = colsum_out ? colsum_partial + (size_t)b * nqb * 3 * A : nullptr;
      if (one) {
        constexpr int LDS = DQ_LDS > DKV_LDS ? DQ_LDS : DKV_LDS;
        static std::atomic<unsigned long long> both_lds{0};
        if (dipaco_status st = ensure_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_both_mfma<DH, NG>), LDS, both_lds)) return st;
        attn_stats_mfma<DH><<<grid, AT_THREADS, 0, s>>>(o + row * A, d_o + row * A, lse + row * H, dsum, S, H);
        DIPACO_LAUNCH_CHECK();
        attn_bwd_both_mfma<DH, NG><<<dim3(n_bh, 2 * nqb), AT_THREADS * NG, LDS, s>>>(qkv + row * 3 * A, d_o + row * A, dsum, dqkv + row * 3 * A, cs, S, H);
        DIPACO_LAUNCH_CHECK();
        continue;
      }
      attn_bwd_dq_mfma<DH, NG><<<grid, AT_THREADS * NG, DQ_LDS, s>>>(qkv + row * 3 * A, o + row * A, d_o + row * A, lse + row * H,
                                                                     dqkv + row * 3 * A, dsum, cs, S, H, single);
      DIPACO_LAUNCH_CHECK();
      attn_bwd_dkv_mfma<DH, NG><<<grid, AT_THREADS * NG, DKV_LDS, s>>>(qkv + row * 3 * A, d_o + row * A, dsum, dqkv + row * 3 * A, cs, S, H, single);
      DIPACO_LAUNCH_CHECK();
    }
    return DIPACO_OK;
  };
  if (dipaco_status st = (one ? one_launch_two_groups(B, H, S) : two_groups(B, H, S)) ? run(std::integral_constant<int, 2>{}) : run(std::integral_constant<int, 1>{})) return st;
  if (colsum_out) return launch_sum_rows(colsum_partial, colsum_out, B * nqb, 3 * H * DH, s, batch);
  return DIPACO_OK;
}

}  // namespace dipaco

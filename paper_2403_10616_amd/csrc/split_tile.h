// fp32 operands on the bf16 matrix cores: every number is taken apart into three bf16 parts, x = h + m + l (each part the
// rounded rest of the ones before: 24 bits, the subtractions are exact), and a product is the six part products h h, h m, m h,
// m m, h l, l h in fp32 accumulators.  The three left out are below 2^-25 of it.  v_mfma_f32_16x16x32_bf16 contracts 32 of K in the time
// v_mfma_f32_16x16x4_f32 takes for two, so six of them do 2.7 times the work of the fp32 instruction.  The instruction cuts what falls
// below its accumulator's last bit: the six are chained from zero over 32 of K and added to the running sum on the vector ALU, which rounds.
// Limits: a third part ends at 2^-133, the smallest bf16 (conversions and products keep subnormal numbers), so a number below
// SPLIT_LEAST errs by up to 2^-134, more than 2^-24 of it; infinities and numbers that round to one make a part NaN.  Callers look
// for both and take what depends on them again in fp32.
// The split and the sum of part products are those of G. Henry, P. T. P. Tang, A. Heinecke, Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations, ARITH 2019.
//
// Operand tiles in LDS: three planes (h, m, l) of rows of 32 K = 64 bytes.  Within a plane, row R lies at row slot
// 4 (R / 4) + ((R ^ (R / 4)) & 3), and its 16-byte chunk c (K 8 c .. 8 c + 7) at chunk c ^ 2 (R / 8 & 1) ^ (R / 16 & 1): what the LDS
// serves together then lies in different slots of its 256-byte bank space, for the 16-byte fragment reads (lane l: row l % 16, chunk
// l / 16) and for the 8-byte stores of both kinds of operand below (see mma_tile.h for the lane sets).
#pragma once
#include "common.h"

namespace dipaco {

constexpr int SPLIT_ROW = 64;    // bytes of a plane's row: 32 of K
constexpr float SPLIT_LEAST = 0x1p-110f;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));

// the parts of two numbers, the first in the low half of each word
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& h, uint32_t& m, uint32_t& l) {
  auto pack = [](float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  };
  auto low = [](uint32_t p) { return __uint_as_float(p << 16); };
  auto high = [](uint32_t p) { return __uint_as_float(p & 0xffff0000u); };
  h = pack(x, y);
  x -= low(h); y -= high(h);
  m = pack(x, y);
  x -= low(m); y -= high(m);
  l = pack(x, y);
}

// s + the squares of a word's two bf16 numbers
__device__ __forceinline__ float add_squares(uint32_t p, float s) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), __builtin_bit_cast(bf16x2, p), s, false);
}

// byte offset of 8-byte piece p (K 4 p .. 4 p + 3) of row R in a plane
__device__ __forceinline__ int split_offset(int R, int p) {
  return ((R & ~3) | ((R ^ (R >> 2)) & 3)) * SPLIT_ROW + (((p >> 1) ^ ((R >> 2) & 2) ^ ((R >> 4) & 1)) << 4) + ((p & 1) << 3);
}
// A unit is 32 rows x 32 of K that a wave stages at a time, four rows of four K per lane:
//   operand contiguous along K: four 16-byte vectors, K 4 (l % 8) .. + 3 of rows l / 8 + 8 j;
//   operand contiguous along its rows: four 16-byte vectors, rows 4 (l % 8) .. + 3 of K 4 (l / 8) + j.
// Eight adjacent lanes read one 128-byte line either way.
template <bool KC> struct SplitUnit {
  float v[4][4];   // [row][K]
  static __device__ __forceinline__ int row(int lane, int j) { return KC ? (lane >> 3) + 8 * j : 4 * (lane & 7); }   // of load j
  static __device__ __forceinline__ int k(int lane, int j) { return KC ? 4 * (lane & 7) : 4 * (lane >> 3) + j; }
  static __device__ __forceinline__ int piece(int lane) { return KC ? lane & 7 : lane >> 3; }   // the lane's four K
  static __device__ __forceinline__ int store_offset(int lane, int q) {   // of row q
    return split_offset(KC ? (lane >> 3) + 8 * q : 4 * (lane & 7) + q, piece(lane));
  }
  __device__ __forceinline__ void load(const char* base, uint32_t off, int j) {
    const float4 x = *reinterpret_cast<const float4*>(base + off);
    if constexpr (KC) {
      v[j][0] = x.x; v[j][1] = x.y; v[j][2] = x.z; v[j][3] = x.w;
    } else {
      v[0][j] = x.x; v[1][j] = x.y; v[2][j] = x.z; v[3][j] = x.w;
    }
  }
  __device__ __forceinline__ void cut(int lane, int left) {   // zeroes the K from `left` on
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (4 * piece(lane) + j >= left) v[0][j] = v[1][j] = v[2][j] = v[3][j] = 0.f;
  }
  __device__ __forceinline__ void least(float& m, int q) const {   // m = min(m, |row q|); by hand: fminf would first quiet its operands
    asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(v[q][0]), "v"(v[q][1]));
    asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(v[q][2]), "v"(v[q][3]));
  }
  __device__ __forceinline__ bool tiny(int q) const {
    auto is = [](float x) { return fabsf(x) < SPLIT_LEAST && x != 0.f; };
    return is(v[q][0]) || is(v[q][1]) || is(v[q][2]) || is(v[q][3]);
  }
  // row q, taken apart, into the planes at p, p + PLANE, p + 2 PLANE; returns the first parts
  template <int PLANE> __device__ __forceinline__ uint2 store(char* p, int q) const {
    uint2 h, m, l;
    split_pair(v[q][0], v[q][1], h.x, m.x, l.x);
    split_pair(v[q][2], v[q][3], h.y, m.y, l.y);
    *reinterpret_cast<uint2*>(p) = h;
    *reinterpret_cast<uint2*>(p + PLANE) = m;
    *reinterpret_cast<uint2*>(p + 2 * PLANE) = l;
    return h;
  }
};

// This lane's byte offsets of a fragment (16 rows x 32 of K) within a plane, from the plane's row 16 b on: b even, odd
struct SplitFragments {
  int at[2];
  __device__ __forceinline__ explicit SplitFragments(int lane)
      : at{split_offset(lane & 15, 2 * (lane >> 4)), split_offset(16 + (lane & 15), 2 * (lane >> 4)) - 16 * SPLIT_ROW} {}
};

// acc[i][j] += A_i . B_j over 32 of K for the blocks of 16 rows at pa, pb (rows of multiples of 32 of their planes)
template <int TM, int TN, int PLANE_A, int PLANE_B>
__device__ __forceinline__ void split_multiply(f32x4 (&acc)[TM][TN], const char* pa, const char* pb, const SplitFragments& f) {
  auto fragment = [&](const char* p, int block) { return *reinterpret_cast<const bf16x8*>(p + f.at[block & 1] + block * 16 * SPLIT_ROW); };
  bf16x8 b[3][TN];
#pragma unroll
  for (int p = 2; p >= 0; --p)
#pragma unroll
    for (int j = 0; j < TN; ++j) b[p][j] = fragment(pb + p * PLANE_B, j);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    bf16x8 a[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) a[p] = fragment(pa + p * PLANE_A, i);
    f32x4 t[TN];
#pragma unroll
    for (int q = 0; q < 6; ++q) {   // small part products first
      constexpr int P[6] = {0, 2, 1, 0, 1, 0}, Q[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
      for (int j = 0; j < TN; ++j)
        t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[P[q]], b[Q[q]][j], q ? t[j] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += t[j];
  }
}

}  // namespace dipaco

// LDS operand tiles for the gfx950 matrix cores and the loaders that fill them.
//
// An operand tile is ROWS rows (the M or N index) by 128 bytes of the contraction index K (32 fp32),
// K-contiguous: that is the order in which v_mfma_f32_32x32x2_f32 wants both operands (lane l supplies row l%32, K-group l/32).  A row is 8 chunks of 16 bytes; chunk c of row r lives at
// chunk position c ^ swz(r), swz(r) = (r >> 1) & 7.
//
// Why this swizzle.  LDS has 64 banks of 4 bytes (addresses 256 bytes apart share a bank).  Measured on gfx950
// with two-lane probes and the SQ_LDS_BANK_CONFLICT counter, the lanes of a wave are served together in these
// sets:  ds_read_b128: {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31} and the same +32;  ds_read_b64: 32 consecutive
// lanes;  ds_write_b128: 8 consecutive lanes;  ds_write_b64: 16 consecutive lanes.  An access is free of conflicts
// when the lanes of a set touch different 16-byte (8-byte) slots of the 256-byte bank space.  A fragment read has
// lane l on row l%32: the rows of either read set, split by parity (odd rows sit 128 bytes higher), take every
// value of (r >> 1) & 7 once, so XOR-ing it into the chunk spreads them over the 8 chunk positions.  Row-major
// 16-byte stores put 8 consecutive lanes on the 8 chunks of one row.
//
// Loaders move global memory -> registers -> LDS, so that loads of later tiles are in flight during the MFMAs
// of the current one.  Loads are unconditional: a tile row beyond the operand reads the operand's last row (it only
// feeds output rows / columns that are never stored), K beyond the range reads the last valid K index instead and is
// zeroed when the tile is written to LDS.
#pragma once
#include "common.h"

namespace dipaco {

constexpr int TILE_ROW_BYTES = 128;

// Global memory straight into LDS: lane l of the wave fetches 16 bytes at gptr into LDS bytes [lds_addr + 16 l, + 16).
// Counted in vmcnt; the wave waits for it with wait_vmcnt (other waves' reads also need the barrier behind that).
template <typename T> __device__ __forceinline__ void load16_to_lds(const T* gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_addr) : "memory");
}
// the same with a wave-uniform base address (scalar registers) and a 32-bit per-lane byte offset
template <typename T> __device__ __forceinline__ void load16_to_lds_at(const T* base, uint32_t byte_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vmcnt() {   // vmcnt only: expcnt and lgkmcnt fields at maximum
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <typename T> struct MmaTraits;
template <> struct MmaTraits<float> { static constexpr int VEC = 4; static constexpr int BK = 32; };

// v if keep, else zero -- as a bitwise AND, so that the compiler cannot turn the load of v into a conditional one
__device__ __forceinline__ uint4 keep_or_zero(const uint4& v, bool keep) {
  const uint32_t m = keep ? 0xffffffffu : 0u;
  return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
}

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

__device__ __forceinline__ char* tile_chunk(char* tile, int row, int chunk) {
  return tile + row * TILE_ROW_BYTES + ((chunk ^ swz(row)) << 4);
}

// One K-group step of a 32x32 MFMA tile.  a, b: this lane's 16-byte fragments (row l%32 of the A / B tile,
// chunk 2*ks + l/32).  fp32: four 32x32x2 MFMAs; MFMA s contracts element s of the two lane halves' chunks (the same K on both operands, so the order of K inside the step does not matter).
template <typename T> __device__ __forceinline__ void mma_step(f32x16& acc, const uint4& a, const uint4& b);
template <> __device__ __forceinline__ void mma_step<float>(f32x16& acc, const uint4& a, const uint4& b) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// Accumulator element e (0..15) of a 32x32 tile held by lane l: row 8*(e/4) + 4*(l/32) + e%4, column l%32.
__device__ __forceinline__ int acc_row(int e, int lane) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }

// ---------------------------------------------------------------------------------------------------------
// TileLoader<T, ROWS, NT>: NT threads fill a tile from a K-contiguous source, element (row, k) at src[row * ld + k]
//   load_tail(r, src, ld, row0, rows_total, k0, k_end, tid)    any tile (K indices clamped to the last valid one)
//   store(r, tile, tid, k0, k_end)            registers -> LDS (zeroing K >= k_end)
template <typename T, int ROWS, int NT> struct TileLoader {
  static constexpr int NLD = ROWS * 8 / NT;
  static constexpr int VEC = MmaTraits<T>::VEC;
  __device__ static __forceinline__ void load_tail(uint4 (&r)[NLD], const T* __restrict__ src, long ld, int row0,
                                                   int rows_total, int k0, int k_end, int tid) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int idx = tid + NT * i;
      const int row = min(row0 + (idx >> 3), rows_total - 1);
      const int k = min(k0 + (idx & 7) * VEC, k_end - VEC);
      r[i] = *reinterpret_cast<const uint4*>(src + (long)row * ld + k);
    }
  }
  __device__ static __forceinline__ void store_full(const uint4 (&r)[NLD], char* tile, int tid) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int idx = tid + NT * i;
      *reinterpret_cast<uint4*>(tile_chunk(tile, idx >> 3, idx & 7)) = r[i];
    }
  }
  __device__ static __forceinline__ void store(const uint4 (&r)[NLD], char* tile, int tid, int k0, int k_end) {
    if (k0 + MmaTraits<T>::BK <= k_end) {   // whole tile inside the K range (uniform branch)
      store_full(r, tile, tid);
    } else {
      const bool keep = k0 + (tid & 7) * VEC < k_end;
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int idx = tid + NT * i;
        *reinterpret_cast<uint4*>(tile_chunk(tile, idx >> 3, idx & 7)) = keep_or_zero(r[i], keep);
      }
    }
  }
};

// Fragments of K group ks (chunk 2*ks + l/32) for a wave that owns TM x TN 32x32 tiles starting at rows
// a_row0 / b_row0 of the A / B tile.
template <int TM, int TN>
__device__ __forceinline__ void load_frags(uint4 (&af)[TM], uint4 (&bfr)[TN], char* a_tile, char* b_tile, int a_row0,
                                           int b_row0, int lane, int ks) {
  const int r = lane & 31, h = lane >> 5;
#pragma unroll
  for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const uint4*>(tile_chunk(a_tile, a_row0 + 32 * i + r, 2 * ks + h));
#pragma unroll
  for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const uint4*>(tile_chunk(b_tile, b_row0 + 32 * j + r, 2 * ks + h));
}
template <typename T, int TM, int TN>
__device__ __forceinline__ void mma_group(f32x16 (&acc)[TM][TN], const uint4 (&af)[TM], const uint4 (&bfr)[TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) mma_step<T>(acc[i][j], af[i], bfr[j]);
}
// All MFMAs of one K tile (fragments of group ks+1 are read while the MFMAs of group ks run).
template <typename T, int TM, int TN>
__device__ __forceinline__ void mma_ktile(f32x16 (&acc)[TM][TN], char* a_tile, char* b_tile, int a_row0, int b_row0,
                                          int lane) {
  uint4 af[2][TM], bfr[2][TN];
  load_frags<TM, TN>(af[0], bfr[0], a_tile, b_tile, a_row0, b_row0, lane, 0);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    if (ks < 3) load_frags<TM, TN>(af[(ks + 1) & 1], bfr[(ks + 1) & 1], a_tile, b_tile, a_row0, b_row0, lane, ks + 1);
    mma_group<T, TM, TN>(acc, af[ks & 1], bfr[ks & 1]);
  }
}

}  // namespace dipaco

// LDS operand tiles for the gfx950 matrix cores, and the loads that fill them.
//
// An operand tile is ROWS rows (the M or N index) by 128 bytes of the contraction index K (32 fp32),
// K-contiguous, as the matrix instructions want both operands.  A row is 8 chunks of 16 bytes; chunk c of row r lives at
// chunk position c ^ swz(r), swz(r) = (r >> 1) & 7.
//
// Why this swizzle.  LDS has 64 banks of 4 bytes (addresses 256 bytes apart share a bank).  Measured on gfx950
// with two-lane probes and the SQ_LDS_BANK_CONFLICT counter, the lanes of a wave are served together in these
// sets:  ds_read_b128: {0-3, 12-15, 20-27}, {4-11, 16-19, 28-31} and the same +32;  ds_read_b64: 32 consecutive
// lanes;  ds_write_b128: 8 consecutive lanes;  ds_write_b64: 16 consecutive lanes.  An access is free of conflicts
// when the lanes of a set touch different 16-byte (8-byte) slots of the 256-byte bank space.  A fragment read of 32 rows has
// lane l on row l%32: the rows of either read set, split by parity (odd rows sit 128 bytes higher), take every
// value of (r >> 1) & 7 once, so XOR-ing it into the chunk spreads them over the 8 chunk positions.  Row-major
// 16-byte stores put 8 consecutive lanes on the 8 chunks of one row.
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

// v if keep, else zero -- as a bitwise AND, so that the compiler cannot turn the load of v into a conditional one
__device__ __forceinline__ uint4 keep_or_zero(const uint4& v, bool keep) {
  const uint32_t m = keep ? 0xffffffffu : 0u;
  return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
}

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

__device__ __forceinline__ char* tile_chunk(char* tile, int row, int chunk) {
  return tile + row * TILE_ROW_BYTES + ((chunk ^ swz(row)) << 4);
}

// Accumulator element e (0..15) of a 32x32 tile held by lane l: row 8*(e/4) + 4*(l/32) + e%4, column l%32.
__device__ __forceinline__ int acc_row(int e, int lane) { return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3); }

}  // namespace dipaco

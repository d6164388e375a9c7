// The order in which the blocks of a causal triangle are dealt to workgroups (fp32 attention).
//
// One block a workgroup, longest first, is as good as it gets where workgroups wait for room: the next one goes to the unit that is done
// first.  A launch whose workgroups are all resident at once is dealt in one go, workgroup i to compute unit i mod 256 (measured with the
// hardware's ids: in 256, 336, 512 and 768 workgroups of 256 and 512 threads, every one), and then longest first puts long blocks with
// long ones: 64 heads of 8 blocks give one unit 8 + 4, another 5 + 1.  Such a launch pairs its rounds of 256 instead, so that a unit's blocks
// add up to about the same.  Forward | backward, us, longest first -> paired: 64 heads x 500 x 64 40.3 -> 36.3 | 113.8 -> 102.6, x 128 67.1 ->
// 58.7 | 205.0 -> 177.5, 128 heads x 500 x 64 57.3 -> 53.4 | 172.4 -> 168.9, 32 x 2000 x 64 209 -> 183 | 583 -> 547.  A multiple of 256 heads has
// nothing to pair, each round being one block of every head, and keeps a head's blocks on one unit: 256 heads x 70 x 128 forward 18.0 us longest first,
// 19.7 paired, x 130 x 64 19.5 | 20.5, x 250 x 32 20.1 | 20.7, backward level.  The bf16 kernels, which wait more and multiply less, gain nothing (42 x 1900 forward 38.3 -> 38.6)
// or lose (64 x 700 x 64 backward 60.2 -> 62.5): they stay longest first.
#pragma once
#include "common.h"

namespace dipaco {

constexpr int CAUSAL_UNITS = 256, CAUSAL_MOST_ROUNDS = 4;

// Rank by length, longest first, of the block that workgroup i of n takes: two to CAUSAL_MOST_ROUNDS rounds
__host__ __device__ __forceinline__ int causal_rank(int i, int n) {
  constexpr int U = CAUSAL_UNITS;
  const int rounds = (n + U - 1) / U, r = i / U, c = i % U, m = n - (rounds - 1) * U;   // m workgroups in the last round
  if (r == rounds - 1) return i;                                   // the shortest blocks, on units 0 .. m - 1
  if (r == rounds - 2) return r * U + (c < m ? U - 1 - c : c - m);   // there the shorter ones of the round before, in reverse
  if (rounds == 3) return c < m ? c : U - 1 - (c - m);             // the other units hold one block more length as c falls
  return r == 0 ? c : 2 * U - 1 - c;                               // four rounds: the first two are pairs of their own
}
struct CausalPlace { int bh, order; };   // sequence and head; block, longest first
// grid (sequences x heads, blocks)
__device__ __forceinline__ CausalPlace causal_place(bool paired) {
  const int n_bh = gridDim.x;
  if (!paired) return {(int)blockIdx.x, (int)blockIdx.y};
  const int rank = causal_rank(blockIdx.x + n_bh * blockIdx.y, n_bh * gridDim.y), order = rank / n_bh;
  return {rank - order * n_bh, order};
}

// whether a launch of n workgroups, blocks of n_bh heads, pairs its rounds: they are resident at once.  `seen`: the kernel's own, workgroups to a unit + 1
inline dipaco_status causal_paired(const void* kernel, int threads, int lds, long n_bh, long n, std::atomic<int>& seen, bool& paired) {
  paired = false;
  if (n_bh % CAUSAL_UNITS == 0 || n <= CAUSAL_UNITS || n > CAUSAL_UNITS * CAUSAL_MOST_ROUNDS) return DIPACO_OK;
  int resident = seen.load(std::memory_order_relaxed) - 1;
  if (resident < 0) {
    DIPACO_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&resident, kernel, threads, lds));
    seen.store(resident + 1, std::memory_order_relaxed);
  }
  paired = n <= (long)CAUSAL_UNITS * resident;
  return DIPACO_OK;
}

}  // namespace dipaco

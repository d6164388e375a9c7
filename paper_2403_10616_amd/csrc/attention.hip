// Causal self-attention, forward and backward, on the packed QKV buffer: dispatch by element type.
//
// Layout: qkv is [B*S, 3A] with A = H*dh; row t holds q (columns 0..A), k (A..2A), v (2A..3A); head h owns
// columns h*dh..(h+1)*dh of each third.  o and d_o are [B*S, A].  lse[b,h,i] = log sum_j exp(s_ij).
// bf16 runs in attention_mfma.hip, fp32 in attention_f32.hip: both on the matrix cores, for head sizes 32, 64 and 128.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace dipaco {

template <typename T>
dipaco_status launch_attention_fwd(const T* qkv, T* o, float* lse, int B, int S, int H, int dh, hipStream_t s) {
  if constexpr (std::is_same<T, bf16>::value) return launch_attention_fwd_mfma(qkv, o, lse, B, S, H, dh, s);
  else return launch_attention_fwd_f32(qkv, o, lse, B, S, H, dh, s);
}

// one row of partial column sums per (document, block of 128 positions), in fp32 also of 64
size_t attention_bwd_colsum_floats(int B, int S, int H, int dh) {
  return std::max((size_t)B * ((S + 127) / 128), attention_bwd_colsum_rows_f32(B, S, H)) * 3 * H * dh;
}

template <typename T>
dipaco_status launch_attention_bwd(const T* qkv, const T* o, const T* d_o, const float* lse, T* dqkv, float* dsum,
                                   float* colsum_out, float* colsum_partial, int B, int S, int H, int dh,
                                   hipStream_t s, SumBatch* batch, bool coarse) {
  if constexpr (std::is_same<T, bf16>::value)
    return launch_attention_bwd_mfma(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, dh, s, batch);
  else
    return launch_attention_bwd_f32(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, dh, s, batch, coarse);
}

template dipaco_status launch_attention_fwd<float>(const float*, float*, float*, int, int, int, int, hipStream_t);
template dipaco_status launch_attention_fwd<bf16>(const bf16*, bf16*, float*, int, int, int, int, hipStream_t);
template dipaco_status launch_attention_bwd<float>(const float*, const float*, const float*, const float*, float*,
                                                   float*, float*, float*, int, int, int, int, hipStream_t, SumBatch*, bool);
template dipaco_status launch_attention_bwd<bf16>(const bf16*, const bf16*, const bf16*, const float*, bf16*, float*,
                                                  float*, float*, int, int, int, int, hipStream_t, SumBatch*, bool);

}  // namespace dipaco

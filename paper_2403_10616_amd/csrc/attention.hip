// Causal self-attention, forward and backward, on the packed QKV buffer: dispatch by element type.
//
// Layout: qkv is [B*S, 3A] with A = H*dh; row t holds q (columns 0..A), k (A..2A), v (2A..3A); head h owns
// columns h*dh..(h+1)*dh of each third.  o and d_o are [B*S, A].  lse[b,h,i] = log sum_j exp(s_ij).
// bf16 runs in attention_mfma.h, fp32 in attention_f32.hip: both on the matrix cores, for head sizes 32, 64 and 128.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "kernels.h"

namespace dipaco {

static std::atomic<int> g_attn_single_block{1};   // test / tuning hook; measured 3-5 % faster than pairing a long with a short block
void set_attention_single_block(int on) { g_attn_single_block = on ? 1 : 0; }
int attention_single_block() { return g_attn_single_block; }

template <typename T>
dipaco_status launch_attention_fwd(const T* qkv, T* o, float* lse, int B, int S, int H, int dh, hipStream_t s) {
  if constexpr (std::is_same<T, bf16>::value) {
    if (dh == 32) return launch_attention_fwd_mfma<32>(qkv, o, lse, B, S, H, s);
    if (dh == 64) return launch_attention_fwd_mfma<64>(qkv, o, lse, B, S, H, s);
    if (dh == 128) return launch_attention_fwd_mfma<128>(qkv, o, lse, B, S, H, s);
    return fail(DIPACO_ESHAPE, "attention: d_head must be 32, 64 or 128");
  } else {
    return launch_attention_fwd_f32(qkv, o, lse, B, S, H, dh, s);
  }
}

// one row of partial column sums per (document, block of 128 positions), in fp32 also of 64
size_t attention_bwd_colsum_floats(int B, int S, int H, int dh) {
  return std::max((size_t)B * ((S + 127) / 128), attention_bwd_colsum_rows_f32(B, S, H)) * 3 * H * dh;
}

template <typename T>
dipaco_status launch_attention_bwd(const T* qkv, const T* o, const T* d_o, const float* lse, T* dqkv, float* dsum,
                                   float* colsum_out, float* colsum_partial, int B, int S, int H, int dh,
                                   hipStream_t s, SumBatch* batch, bool coarse) {
  if constexpr (std::is_same<T, bf16>::value) {
    if (dh == 32) return launch_attention_bwd_mfma<32>(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, s, batch);
    if (dh == 64) return launch_attention_bwd_mfma<64>(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, s, batch);
    if (dh == 128) return launch_attention_bwd_mfma<128>(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, s, batch);
    return fail(DIPACO_ESHAPE, "attention: d_head must be 32, 64 or 128");
  } else {
    return launch_attention_bwd_f32(qkv, o, d_o, lse, dqkv, dsum, colsum_out, colsum_partial, B, S, H, dh, s, batch, coarse);
  }
}

template dipaco_status launch_attention_fwd<float>(const float*, float*, float*, int, int, int, int, hipStream_t);
template dipaco_status launch_attention_fwd<bf16>(const bf16*, bf16*, float*, int, int, int, int, hipStream_t);
template dipaco_status launch_attention_bwd<float>(const float*, const float*, const float*, const float*, float*,
                                                   float*, float*, float*, int, int, int, int, hipStream_t, SumBatch*, bool);
template dipaco_status launch_attention_bwd<bf16>(const bf16*, const bf16*, const bf16*, const float*, bf16*, float*,
                                                  float*, float*, int, int, int, int, hipStream_t, SumBatch*, bool);

}  // namespace dipaco

// bf16 attention with head sizes 32 and 128 (attention_mfma.h); NaN is honoured.
#include "attention_mfma.h"

namespace dipaco {

template dipaco_status launch_attention_fwd_mfma<32>(const bf16*, bf16*, float*, int, int, int, hipStream_t);
template dipaco_status launch_attention_bwd_mfma<32>(const bf16*, const bf16*, const bf16*, const float*, bf16*, float*, float*,
                                                      float*, int, int, int, hipStream_t, SumBatch*);
template dipaco_status launch_attention_fwd_mfma<128>(const bf16*, bf16*, float*, int, int, int, hipStream_t);
template dipaco_status launch_attention_bwd_mfma<128>(const bf16*, const bf16*, const bf16*, const float*, bf16*, float*, float*,
                                                      float*, int, int, int, hipStream_t, SumBatch*);

}  // namespace dipaco

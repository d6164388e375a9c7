// bf16 attention with head size 64 (attention_mfma.h); compiled with -fno-honor-nans (build.py).
#include "attention_mfma.h"

namespace dipaco {

template dipaco_status launch_attention_fwd_mfma<64>(const bf16*, bf16*, float*, int, int, int, hipStream_t);
template dipaco_status launch_attention_bwd_mfma<64>(const bf16*, const bf16*, const bf16*, const float*, bf16*, float*, float*,
                                                      float*, int, int, int, hipStream_t, SumBatch*);

}  // namespace dipaco

// The FP32 decoder on the vector ALU, one query per lane, its activations in the lane's own
// column of an LDS table: the pieces shared by decode_f32_kernel and by the few queries that the
// split decode (decode_split.h) hands back to full FP32.
#pragma once

#include "frames.h"
#include "latent_fetch.h"

namespace nam {

__device__ __forceinline__ float softplus_f32(float q) {
    // max(q, 0) + log(1 + exp(-|q|)), exact for every q without a threshold
    return fmaxf(q, 0.0f) + log1pf(expf(-fabsf(q)));
}

// out[o] = sum_j Wt[j][o] * col[j S] + bias[o], j < IN, o < OUT; Wt and bias wave-uniform, S the
// row stride of the table.
template <int IN, int OUT, int S>
__device__ __forceinline__ void dense_from_lds(const float* __restrict__ Wt, const float* col, float* out) {
    const float* bias = Wt + IN * OUT;
    #pragma unroll
    for (int o = 0; o < OUT; ++o) out[o] = bias[o];
    #pragma unroll 2
    for (int j = 0; j < IN; ++j) {
        const float aj = col[j * S];
        const float* wj = Wt + j * OUT;
        #pragma unroll
        for (int o = 0; o < OUT; ++o) out[o] = fmaf(wj[o], aj, out[o]);
    }
}

}  // namespace nam

// Sample-mode launches of the transformer (transformer.hpp).
#include "transformer.hpp"

namespace nnqs {

__global__ void __launch_bounds__(64 * kTfWaves) k_transformer_bf16(Bf16View M, TfArgs A) {
    transformer<false, false, false>(M, A, nullptr, 0);
}

__global__ void __launch_bounds__(64 * kTfWaves) k_transformer_fp8(Bf16View M, TfArgs A) {
    transformer<false, true, false>(M, A, nullptr, 0);
}

void tf_launch_sample(bool fp8, unsigned grid, hipStream_t st, const Bf16View &M, const TfArgs &A) {
    if (fp8) hipLaunchKernelGGL(k_transformer_fp8, dim3(grid), dim3(64 * kTfWaves), 0, st, M, A);
    else hipLaunchKernelGGL(k_transformer_bf16, dim3(grid), dim3(64 * kTfWaves), 0, st, M, A);
}

}  // namespace nnqs

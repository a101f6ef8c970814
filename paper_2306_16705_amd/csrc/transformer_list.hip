// BF16 list-mode launch of the transformer (transformer.hpp).
#include "transformer.hpp"

namespace nnqs {

__global__ void __launch_bounds__(64 * kTfWaves) k_transformer_bf16_list(Bf16View M, TfArgs A) {
    transformer<true, false, false>(M, A, nullptr, 0);
}

void tf_launch_list_fp8(unsigned grid, hipStream_t st, const Bf16View &M, const TfArgs &A);

void tf_launch_list(bool fp8, unsigned grid, hipStream_t st, const Bf16View &M, const TfArgs &A) {
    if (fp8) tf_launch_list_fp8(grid, st, M, A);
    else hipLaunchKernelGGL(k_transformer_bf16_list, dim3(grid), dim3(64 * kTfWaves), 0, st, M, A);
}

}  // namespace nnqs

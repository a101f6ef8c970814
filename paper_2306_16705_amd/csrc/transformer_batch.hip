// Many systems in one persistent launch of the transformer
// (transformer.hpp): the list-mode work of every item as one tile space, each
// tile run with its item's model.
#include "transformer.hpp"

namespace nnqs {

__global__ void __launch_bounds__(64 * kTfWaves) k_transformer_bf16_batch(Bf16View M0, const TfItem *items, int n_items) {
    transformer<true, false, true>(M0, items[0].A, items, n_items);
}

void tf_launch_batch(unsigned grid, hipStream_t st, const Bf16View &M0, const TfItem *items, int n_items) {
    hipLaunchKernelGGL(k_transformer_bf16_batch, dim3(grid), dim3(64 * kTfWaves), 0, st, M0, items, n_items);
}

}  // namespace nnqs

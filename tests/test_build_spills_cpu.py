"""Private memory of the kernels that the other build guard does not name, from
the compiler's own report: the scans, batch sampling's rows, the phase network
and the gradient's attention keep everything in registers; the whole-wave
transformers, at 256 registers for two waves per SIMD, spill no more than they
were measured with."""
from concurrent.futures import ThreadPoolExecutor

import pytest

from tests.test_build_cpu import _resource_usage

# file: {kernel (a part of its name): bytes a lane at most}
LIMITS = {
    "eloc_sa.hip": {"k_eloc_scanI": 0, "k_eloc_scan_batch": 0},
    "model_bf16.hip": {"k_phase_bf16": 0, "k_bf16_refresh": 0},
    "model_f64.hip": {"k64x_attention_back": 0},
    "transformer_f64.hip": {"k64_transformerE": 224, "k64_transformer_list": 264},
    "transformer_sample.hip": {"k_transformer_bf16E": 148, "k_transformer_fp8E": 12},
    "transformer_list.hip": {"k_transformer_bf16_list": 340},
    "transformer_list_fp8.hip": {"k_transformer_fp8_list": 64},
    "transformer_batch.hip": {"k_transformer_bf16_batch": 540},
    "transformer_rows.hip": {"k_transformer_rows": 0},
}


@pytest.fixture(scope="module")
def usage():
    with ThreadPoolExecutor(4) as pool:
        return dict(zip(LIMITS, pool.map(_resource_usage, LIMITS)))


@pytest.mark.parametrize("src", list(LIMITS))
def test_private_memory_is_bounded(usage, src):
    for part, most in LIMITS[src].items():
        names = [k for k in usage[src] if part in k]
        assert names, part
        for k in names:
            assert usage[src][k] <= most, (k, usage[src][k])

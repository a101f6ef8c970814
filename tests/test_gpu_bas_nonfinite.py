"""Batch sampling when some prefixes have no finite conditionals: the embedding
of one token is NaN, so every prefix that holds it (before its last position)
is dropped, and no other.

The BF16 network draws 16 prefixes of a wave together; the FP64 one evaluates
each by itself and drops the same prefixes.  Their conditionals differ by about
1 %, so the numbers of unique samples agree to a few per cent: 5 %.  A NaN that
reached the prefixes of its wave would drop most of them."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import keys_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("K,nu,ns", [(20, 8, 400000), (36, 8, 400000)])
def test_a_dropped_prefix_takes_no_other_with_it(nn, K, nu, ns):
    print(f"[case] bas with NaN prefixes K={K} n_samples={ns}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=1, n_unique=2, model=True, beta=0.1)
    w = dict(d["weights"])
    w["tok_emb"] = w["tok_emb"].copy()
    w["tok_emb"][2] = np.nan  # a down electron alone on its orbital
    M = nn.Model(d["model_shape"], nu, 1, w)
    k, c, la, _ = nn.bas(M, ns, 5, nn.NNQS_BF16)
    ref, _, _, _ = nn.bas(M, ns, 5, nn.NNQS_FP64, with_phase=False)
    print(f"{len(k)} unique in BF16, {len(ref)} in FP64", flush=True)
    assert len(ref) > 3000  # more than one prefix per wave
    occ = synth.unpack_keys(keys_np(k), K)
    assert not np.any(occ[:, 1, 1:] & ~occ[:, 0, 1:])  # orbital 0 is the last position
    la2, _ = nn.model_logpsi(M, k.contiguous(), nn.NNQS_BF16)
    assert torch.all((la - la2).abs() <= 1e-6 * la2.abs().clamp(min=1.0))
    assert abs(len(k) - len(ref)) <= 0.05 * len(ref)

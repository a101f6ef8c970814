"""Sizes at which the gradient's kernels change path: row blocks and splits
part filled, more than one pass, hidden sizes off the tiles, more layers than
one grouped launch holds; and the reduced-precision copies after a step.

The bar is that of the other gradient tests: 1e-9 of the largest entry of each
tensor.  A copy refreshed by a step and one made from the same weights are the
same bits, so their outputs are equal."""
import numpy as np
import pytest
import torch

import oracle.vmc as vmc
import synth
from tests.gpu_util import dev
from tests.test_gpu_vmc import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("K,n,L,F,P", [(15, 1, 1, 64, 1), (16, 300, 4, 256, 512), (17, 47, 2, 192, 63),
                                       (33, 5, 2, 128, 70), (49, 3, 5, 1024, 1000), (64, 25, 6, 64, 65)])
def test_gradient_shapes(nn, K, n, L, F, P):
    print(f"[case] gradient K={K} n={n} L={L} F={F} P={P}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=3, n_dn=2, n_unique=n)
    shape = synth.TransformerShape(K=K, n_layers=L, d_ff=F, phase_hidden=P)
    rng = np.random.default_rng([K, n])
    w = synth.transformer_weights(shape, 3, 2, rng)
    cl, cp = rng.normal(size=n), rng.normal(size=n)
    M = nn.Model(shape, 3, 2, w)
    g = nn.model_grad(M, dev(d["keys"]), dev(cl), dev(cp))
    assert torch.equal(g, nn.model_grad(M, dev(d["keys"]), dev(cl), dev(cp))), "two calls differ"
    ora = vmc.logpsi_vjp(w, shape, 3, 2, d["keys"], cl, cp)
    _compare(g.cpu().numpy(), ora, shape, 1e-9, f"K={K}")


@pytest.mark.parametrize("K,L", [(5, 1), (64, 4)])
def test_refreshed_copies_equal_new_ones(nn, K, L):
    print(f"[case] refreshed copies K={K} L={L}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=3, n_dn=2, n_unique=40)
    shape = synth.TransformerShape(K=K, n_layers=L)
    rng = np.random.default_rng(K)
    M = nn.Model(shape, 3, 2, synth.transformer_weights(shape, 3, 2, rng))
    nw = nn.model_get_weights(M).numel()
    m1, m2 = (torch.zeros(nw, dtype=torch.float64, device="cuda") for _ in range(2))
    nn.model_adamw_step(M, dev(rng.normal(size=nw)), 1, 0.01, m1, m2)
    wd = vmc.unpack(nn.model_get_weights(M).cpu().numpy(), synth.transformer_weights(shape, 3, 2, rng), shape)
    M2 = nn.Model(shape, 3, 2, {k: v.astype(np.float32) for k, v in wd.items()})
    for prec in (nn.NNQS_BF16, nn.NNQS_FP8):
        for a, b in zip(nn.model_logpsi(M, dev(d["keys"]), prec), nn.model_logpsi(M2, dev(d["keys"]), prec)):
            assert torch.equal(a, b)

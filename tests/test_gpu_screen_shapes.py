"""The screen's training kernels at the edges of their tiles: hidden sizes and
example counts around 16, 64 and 256, systems on either side of one key word.

Against the FP64 oracle with the bars of the other screen tests: FP64 1e-12 of
max(1, |y|) and 1e-11 of the largest gradient entry, FP32 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev
from tests.test_gpu_screen import _connection_inputs, _weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("K,H,n", [(4, 1, 1), (7, 15, 16), (8, 16, 17), (31, 63, 63), (32, 64, 64), (33, 65, 65),
                                   (48, 255, 513), (60, 257, 127), (64, 1024, 129), (64, 256, 1100)])
@pytest.mark.parametrize("fp32", [False, True])
def test_shapes_match_oracle(nn, K, H, n, fp32):
    N = 2 * K
    print(f"[case] screen shapes K={K} H={H} n={n} fp32={fp32}", flush=True)
    prec, fb, gb = (nn.NNQS_FP32, 1e-4, 1e-4) if fp32 else (nn.NNQS_FP64, 1e-12, 1e-11)
    keys, exc, target = _connection_inputs(K, n, seed=K + H)
    exc[n // 2] = 255  # absent codes add nothing
    w = _weights(N, H, seed=n) / max(1.0, np.sqrt(H / 64.0))
    S = nn.Screen(N, H, w)
    pred = S.forward(dev(keys), dev(exc), prec).cpu().numpy()
    ref = oracle.screen_forward(N, H, w, keys, exc)
    assert np.max(np.abs(pred - ref) / np.maximum(1.0, np.abs(ref))) < fb
    g, loss = S.gradient(dev(keys), dev(exc), dev(target), prec)
    oloss, og = oracle.screen_loss_grad(N, H, w, keys, exc, target)
    assert abs(loss.item() - oloss) <= fb * max(1.0, abs(oloss))
    assert np.max(np.abs(g.cpu().numpy() - og)) <= gb * np.abs(og).max()

"""Batch sampling in BF16 with cached rows: lengths on either side of every
block of 16 positions, from fewer prefixes than waves to several per wave.

A path's log-probability is the FP64 sum of the conditionals; the network's
own log|psi| rounds the sum of each 16 positions to FP32 (16 additions, 2^-24
each), so they agree to 1e-6 of max(1, |log psi|).  A wrong key or value would
show at 1e-3."""
import threading

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


def _model(nn, K, nu, nd):
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=2, model=True)
    return nn.Model(d["model_shape"], nu, nd, d["weights"])


@pytest.mark.parametrize("ns", [1, 300, 120000])
@pytest.mark.parametrize("K,nu,nd", [(2, 1, 1), (15, 4, 3), (16, 5, 5), (17, 4, 5), (31, 6, 6), (33, 5, 6), (48, 8, 8),
                                     (49, 8, 7), (64, 10, 10)])
def test_paths_agree_with_the_network(nn, K, nu, nd, ns):
    print(f"[case] bas rows K={K} n_samples={ns}", flush=True)
    M = _model(nn, K, nu, nd)
    k, c, la, ph = nn.bas(M, ns, 11, nn.NNQS_BF16)
    assert int(c.cpu().numpy().view(np.uint32).astype(np.int64).sum()) == ns
    assert len(torch.unique(k, dim=0)) == len(k)
    la2, ph2 = nn.model_logpsi(M, k.contiguous(), nn.NNQS_BF16)
    print(f"{len(k)} unique, max difference {float((la - la2).abs().max()):.2e}")
    assert torch.all((la - la2).abs() <= 1e-6 * la2.abs().clamp(min=1.0))
    assert torch.equal(ph, ph2)
    again = nn.bas(M, ns, 11, nn.NNQS_BF16)
    assert all(torch.equal(a, b) for a, b in zip((k, c, la, ph), again))


def test_two_threads_share_a_model(nn):
    print("[case] bas from two threads", flush=True)
    M = _model(nn, 24, 6, 6)
    want = [nn.bas(M, 20000, seed, nn.NNQS_BF16) for seed in (1, 2)]
    torch.cuda.synchronize()
    got = [None, None]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                got[i] = nn.bas(M, 20000, i + 1, nn.NNQS_BF16)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(want, got):
        assert all(torch.equal(x, y) for x, y in zip(a, b))

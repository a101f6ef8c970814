"""Row-block and configuration counts, and activation sizes, at which the
one-launch FP64 transformer changes path.

Against the FP64 oracle: 1e-12 of max(1, |log psi|) (about 10^3 roundings of
1e-16 per row, 64 rows).  Weights scaled up take the FFN's GELU through its
three ranges (|v| below 1, below 4, beyond).  The prefix-reusing list path,
with every term refined, against the whole forward of every x': 1e-12 of the
sum of |terms| (log psi to 1e-14, compensated sums)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import dev, eloc_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("scale", [1.0, 12.0, 60.0])
@pytest.mark.parametrize("K,n", [(15, 1), (16, 5), (17, 3), (32, 9), (33, 2), (48, 1), (49, 3), (64, 2)])
def test_against_the_oracle(nn, K, n, scale):
    print(f"[case] FP64 transformer K={K} n={n} scale={scale}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=3, n_dn=2, n_unique=n, model=True)
    w = {k: v * np.float32(scale) if k.endswith((".w1", ".b1", ".wq", ".wk")) else v for k, v in d["weights"].items()}
    M = nn.Model(d["model_shape"], 3, 2, w)
    la, ph = nn.model_logpsi(M, dev(d["keys"]), nn.NNQS_FP64)
    ola, oph = oracle.net_logpsi(w, d["model_shape"], 3, 2, d["keys"])
    assert np.all(np.abs(la.cpu().numpy() - ola) <= 1e-12 * np.maximum(1.0, np.abs(ola)))
    assert np.all(np.abs(ph.cpu().numpy() - oph) <= 1e-12)


def test_part_filled_tiles(nn):
    """Every configuration of a long list gives what it gives alone, bit for bit."""
    for K, n in ((12, 1030), (40, 517)):
        print(f"[case] FP64 part-filled tiles K={K}", flush=True)
        d = synth.config_inputs(2, K=K, n_up=4, n_dn=4, n_unique=n, model=True)
        M = nn.Model(d["model_shape"], 4, 4, d["weights"])
        keys = dev(d["keys"])
        la, ph = nn.model_logpsi(M, keys, nn.NNQS_FP64)
        for a, b in ((0, 1), (2, 5), (9, 300), (n - 3, n)):
            sa, sp = nn.model_logpsi(M, keys[a:b].contiguous(), nn.NNQS_FP64)
            assert torch.equal(sa, la[a:b]) and torch.equal(sp, ph[a:b]), (K, a, b)


@pytest.mark.parametrize("dedup", [False, True])
@pytest.mark.parametrize("K,nu,nd,n", [(16, 2, 3, 4), (17, 3, 3, 3), (33, 2, 3, 2), (48, 2, 3, 3), (64, 2, 2, 5)])
def test_refinement_equals_the_whole_forward(nn, K, nu, nd, n, dedup):
    print(f"[case] FP64 refinement K={K} n={n} dedup={dedup}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=n, model=True)
    S = nn.System(d["N"], nu, nd, d["h"], d["g"], d["e_core"])
    M = nn.Model(d["model_shape"], nu, nd, d["weights"])
    keys = dev(d["keys"])
    e = eloc_complex(nn.eloc_model(S, M, keys, precision=nn.NNQS_BF16, with_energy=False, refine_nats=200.0,
                                   dedup=dedup)[0])
    c = nn.connections(S, keys)
    la, ph = (t.reshape(n, -1) for t in nn.model_logpsi(M, c["xprime"].reshape(-1, 2), nn.NNQS_FP64))
    la0, ph0 = nn.model_logpsi(M, keys, nn.NNQS_FP64)
    amp = c["hxx"] * torch.exp(la - la0[:, None])
    dphi = ph - ph0[:, None]
    ref = torch.complex((amp * dphi.cos()).sum(1), (amp * dphi.sin()).sum(1)).cpu().numpy()
    scale = amp.abs().sum(1).cpu().numpy()
    assert np.all(np.abs(e - ref) <= 1e-12 * scale), np.max(np.abs(e - ref) / scale)

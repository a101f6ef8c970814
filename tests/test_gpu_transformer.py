"""Row-block and configuration counts at which the register-resident BF16 /
FP8 transformer changes path: every (own row blocks, first block) pair of the
prefix-reusing forward, part-filled waves and tiles.

The prefix-reusing forward does for each row what the whole forward does, in
the same order, so the full local energy must equal the sum over exported
connections with log|psi| and phase of the whole forward: FP64 sums of the
same terms in another order, 1e-13 of the sum of |terms| (about 10^4 terms of
rounding 1e-16 each)."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import dev, eloc_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
@pytest.mark.parametrize("K,nu,nd,n", [(15, 3, 2, 5), (16, 2, 3, 4), (17, 3, 3, 3), (32, 3, 2, 9), (33, 2, 3, 2),
                                       (48, 2, 3, 3), (49, 3, 2, 2), (64, 2, 2, 5)])
def test_prefix_classes_equal_the_whole_forward(nn, precision, K, nu, nd, n):
    print(f"[case] prefix classes {precision} K={K} n={n}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=n, model=True)
    p = nn.NNQS_BF16 if precision == "bf16" else nn.NNQS_FP8
    S = nn.System(d["N"], nu, nd, d["h"], d["g"], d["e_core"])
    M = nn.Model(d["model_shape"], nu, nd, d["weights"])
    keys = dev(d["keys"])
    e = eloc_complex(nn.eloc_model(S, M, keys, precision=p, with_energy=False)[0])
    c = nn.connections(S, keys)
    la, ph = (t.reshape(n, -1) for t in nn.model_logpsi(M, c["xprime"].reshape(-1, 2), p))
    la0, ph0 = nn.model_logpsi(M, keys, p)
    amp = c["hxx"] * torch.exp(la - la0[:, None])
    dphi = ph - ph0[:, None]
    ref = torch.complex((amp * dphi.cos()).sum(1), (amp * dphi.sin()).sum(1)).cpu().numpy()
    scale = amp.abs().sum(1).cpu().numpy()
    assert np.all(np.abs(e - ref) <= 1e-13 * scale), np.max(np.abs(e - ref) / scale)


@pytest.mark.parametrize("K", [7, 32, 40, 60])
def test_part_filled_tiles(nn, K):
    """Every configuration of a long list gives what it gives alone, bit for bit."""
    print(f"[case] part-filled tiles K={K}", flush=True)
    nu = nd = max(2, K // 4)
    n = 2051 if K > 7 else 300
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=n, model=True)
    M = nn.Model(d["model_shape"], nu, nd, d["weights"])
    keys = dev(d["keys"])
    la, ph = nn.model_logpsi(M, keys, nn.NNQS_BF16)
    for a, b in ((0, 1), (1, 4), (5, 12), (17, 274), (n - 9, n)):
        sa, sp = nn.model_logpsi(M, keys[a:b].contiguous(), nn.NNQS_BF16)
        assert torch.equal(sa, la[a:b]) and torch.equal(sp, ph[a:b]), (a, b)


def test_phase_groups_agree(nn):
    """The phase of a configuration is the same bits whatever the call's size:
    lists on either side of each change of the group size (256 CUs) against
    the configurations in calls of at most 16."""
    K = 20
    d = synth.config_inputs(2, K=K, n_up=5, n_dn=5, n_unique=16401, model=True)
    M = nn.Model(d["model_shape"], 5, 5, d["weights"])
    keys = dev(d["keys"])
    cut = [(0, 16), (4080, 4096), (4095, 4097), (8190, 8195), (16380, 16390)]
    few = {c: nn.model_logpsi(M, keys[c[0]:c[1]].contiguous(), nn.NNQS_BF16)[1] for c in cut}
    for n in (4096, 4097, 8192, 8193, 16384, 16385):
        print(f"[case] phase groups n={n}", flush=True)
        ph = nn.model_logpsi(M, keys[:n].contiguous(), nn.NNQS_BF16)[1]
        for (a, b), want in few.items():
            m = min(b, n) - a
            assert m <= 0 or torch.equal(ph[a:a + m], want[:m]), (n, a)

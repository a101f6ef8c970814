"""Memory of the refinement's FP64 cache: keys and values of the row blocks of
16 positions that the system has."""
import pytest
import torch

import synth
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("K,ne,blocks", [(8, 4, 1), (20, 2, 2)])
def test_refinement_cache_follows_the_sequence_length(nn, K, ne, blocks):
    """4,096 samples of four layers: 64 KiB a sample and row block, 256 MiB a
    block in all; 64 MB of other scratch (the FP64 phase's 32 MiB) allowed for."""
    print(f"[case] refinement cache K={K}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=ne, n_dn=ne, n_unique=4096, model=True)
    S = nn.System(d["N"], ne, ne, d["h"], d["g"], d["e_core"])
    M = nn.Model(d["model_shape"], ne, ne, d["weights"])
    keys = dev(d["keys"])
    nn.eloc_model(S, M, keys, precision=nn.NNQS_BF16, with_energy=False)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    nn.eloc_model(S, M, keys, precision=nn.NNQS_BF16, with_energy=False, refine_nats=1.0)
    torch.cuda.synchronize()
    grown = before - torch.cuda.mem_get_info()[0]
    print(f"{grown / MB:.0f} MB", flush=True)
    assert grown <= (256 * blocks + 64) * MB

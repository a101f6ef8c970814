"""Calls of more than 2^26 rows, where 64 threads a row no longer fit one
launch: rows that repeat give results that repeat, bit for bit."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

N_ROWS = 36 * 1864136  # 2^26 + 32


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


def _repeat(t):
    return t.repeat((N_ROWS // 36,) + (1,) * (t.dim() - 1))


def test_samples_of_a_scanned_table(nn):
    print("[case] scan of 2^26 + 32 samples", flush=True)
    d = synth.config_inputs(1)
    S = nn.System(d["N"], d["n_up"], d["n_dn"], d["h"], d["g"], d["e_core"])
    keys, la, ph = dev(d["keys"]), dev(d["logabs"]), dev(d["phase"])
    T = nn.Table(S, 36).build(keys, la, ph, validate=True)
    few, _ = nn.eloc_table(S, T, keys, None, la, ph, with_energy=False)
    e, _ = nn.eloc_table(S, T, _repeat(keys), None, _repeat(la), _repeat(ph), with_energy=False)
    assert torch.equal(e[:36], few)  # fewer than 256 members: never split
    assert bool((e.view(-1, 36, 2) == few).all())


def test_examples_of_a_screen(nn):
    print("[case] screen of 2^26 + 32 examples", flush=True)
    d = synth.config_inputs(1)
    keys = dev(d["keys"])
    exc = torch.randint(0, 9, (36, 4), generator=torch.Generator().manual_seed(3)).to(torch.uint8).cuda()
    scr = nn.Screen(8, 1, np.random.default_rng([16705, 96]).normal(0, 0.3, 5 * 8 + 5))
    few = scr.forward(keys, exc, nn.NNQS_FP64)
    y = scr.forward(_repeat(keys), _repeat(exc), nn.NNQS_FP64)
    assert torch.equal(y[:36], few)
    assert bool((y.view(-1, 36) == few).all())

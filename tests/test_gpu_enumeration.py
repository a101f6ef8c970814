"""The enumeration of connections (k_eloc_sa and its exact and batched forms)
at table sizes for which it is the path taken, which every call is checked to
have used: dense hits in two-word keys, both searches, schedules, samples far
below the largest amplitude, the autotuners and batches.

Against the oracle at the bar of the other sample-aware tests; schedules
against one another at 1e-12 of max(1, |E|) (rounding order)."""
import os

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import assert_eloc_close, dev, eloc_complex
from tests.test_gpu_parity_allhit import _all_hit_table
from tests.test_gpu_sa_paths import launches

pytestmark = pytest.mark.gpu

SINGLE, BATCH = ("k_eloc_scan", "k_eloc_sa"), ("k_eloc_scan_batch", "k_eloc_sa_batch")
CORES = len(os.sched_getaffinity(0))


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


def _system(nn, d):
    return nn.System(d["N"], d["n_up"], d["n_dn"], d["h"], d["g"], d["e_core"])


def _enumerated(nn, call, names=SINGLE):
    r, got = launches(nn, names, call)
    assert got[0] == 0 and got[1] > 0, got
    return r


def _oracle(d, keys, la, ph, idx):
    return oracle.eloc_table(d["K"], d["n_up"], d["n_dn"], d["h"], d["g"], d["e_core"], keys, la, ph, keys[idx], la[idx],
                             ph[idx], with_absum=True, nthreads=CORES)


@pytest.mark.parametrize("K,nu,nd,take", [(24, 6, 6, 12), (40, 3, 3, 20), (33, 4, 3, 20), (64, 3, 2, 12), (60, 20, 20, 3)])
def test_all_hit_tables(nn, K, nu, nd, take):
    """Every connection of the checked samples is a member: a connection that
    the loops drop, repeat or sign wrongly changes E_loc by a whole term.  Other
    members make up the 2,100 samples of the call: fewer would scan the table."""
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=take)
    keys, la, ph, pos = _all_hit_table(d, take, 3)
    smp = np.concatenate([pos, np.setdiff1d(np.arange(len(keys)), pos)[:2100]])
    assert len(smp) > 2100
    print(f"[case] all-hit enumeration K={K}, {len(keys)} members", flush=True)
    S = _system(nn, d)
    T = nn.Table(S, len(keys))
    ora, absum = _oracle(d, keys, la, ph, pos)
    for tune in (dict(search=1, splitter_levels=10), dict(search=2, splitter_levels=12),
                 dict(search=2, waves_per_block=16, filter_log2_bits=14, splitter_levels=3)):
        T.set_tune(**tune)
        T.build(dev(keys), dev(la), dev(ph), validate=True)
        e, _ = _enumerated(nn, lambda: nn.eloc_table(S, T, dev(keys[smp]), None, dev(la[smp]), dev(ph[smp]),
                                                     with_energy=False, validate=True))
        assert_eloc_close(eloc_complex(e)[:len(pos)], ora, absum, label=f"all-hit K={K} {tune}")


@pytest.mark.parametrize("search", [1, 2])
def test_whole_sector(nn, search):
    """K = 12, 4 up and 3 down: the whole sector of 108,900 members, every
    connection a hit, in a call of as many samples."""
    d = synth.config_inputs(1, K=12, n_up=4, n_dn=3)
    n = len(d["keys"])
    print(f"[case] whole sector of {n}, search {search}", flush=True)
    S = _system(nn, d)
    T = nn.Table(S, n)
    T.set_tune(search=search, splitter_levels=8 if search == 1 else 12)
    keys, la, ph = dev(d["keys"]), dev(d["logabs"]), dev(d["phase"])
    T.build(keys, la, ph, validate=True)
    e, en = _enumerated(nn, lambda: nn.eloc_table(S, T, keys, dev(d["counts"], torch.int32), la, ph, validate=True))
    g, chk = eloc_complex(e), np.arange(0, n, 53)
    ora, absum = _oracle(d, d["keys"], d["logabs"], d["phase"], chk)
    assert_eloc_close(g[chk], ora, absum, label="whole sector")
    ref = oracle.energy(d["counts"], g)
    assert abs(en[0].item() - ref[0]) <= 1e-12 * abs(ref[0])


@pytest.fixture(scope="module")
def n48():
    return synth.config_inputs(2, n_unique=40000)


def test_schedules_agree(nn, n48):
    print("[case] schedules of an enumerated table", flush=True)
    d, S = n48, _system(nn, n48)
    T = nn.Table(S, 40000)
    keys, la, ph = dev(d["keys"]), dev(d["logabs"]), dev(d["phase"])
    T.build(keys, la, ph)
    call = lambda: nn.eloc_table(S, T, keys, None, la, ph, with_energy=False)[0]
    base = _enumerated(nn, call)
    assert torch.equal(base, call())
    base = eloc_complex(base)
    chk = np.arange(0, 40000, 401)
    ora, absum = _oracle(d, d["keys"], d["logabs"], d["phase"], chk)
    assert_eloc_close(base[chk], ora, absum, label="default schedule")
    for tune in (dict(filter_log2_bits=12), dict(waves_per_block=4, blocks_per_cu=3),
                 dict(filter_log2_bits=20, splitter_levels=13), dict(search=2, splitter_levels=7),
                 dict(search=2, splitter_levels=12), dict(waves_per_block=16),
                 dict(waves_per_block=16, search=1, splitter_levels=12)):
        T.set_tune(**tune)
        T.build(keys, la, ph)
        g = eloc_complex(_enumerated(nn, call))
        assert np.all(np.abs(g - base) <= 1e-12 * np.maximum(1.0, np.abs(base))), tune


def test_autotuned_schedule(nn, n48):
    print("[case] autotuner on an enumerated table", flush=True)
    d, S = n48, _system(nn, n48)
    T = nn.Table(S, 40000)
    keys, la, ph = dev(d["keys"]), dev(d["logabs"]), dev(d["phase"])
    T.build(keys, la, ph)
    base = eloc_complex(nn.eloc_table(S, T, keys, None, la, ph, with_energy=False)[0])
    tune, ms = _enumerated(nn, lambda: T.autotune(keys, la, ph, reps=1))
    assert tune["waves_per_block"] in (8, 12, 16) and tune["splitter_levels"] in (8, 10, 12) and tune["search"] in (1, 2)
    assert T.get_tune() == tune and ms > 0.0
    g = eloc_complex(_enumerated(nn, lambda: nn.eloc_table(S, T, keys, None, la, ph, with_energy=False))[0])
    assert np.all(np.abs(g - base) <= 1e-12 * np.maximum(1.0, np.abs(base)))


@pytest.mark.parametrize("K,nu,nd,n", [(12, 4, 3, 60000), (40, 2, 2, 100000)])
def test_samples_far_below_the_largest_amplitude(nn, K, nu, nd, n):
    print(f"[case] exact pass of an enumerated table K={K}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=n)
    la = d["logabs"].copy()
    la[::7] -= 650.0
    S = _system(nn, d)
    T = nn.Table(S, n)
    T.build(dev(d["keys"]), dev(la), dev(d["phase"]), validate=True)
    m = 4200  # samples of the call
    e, _ = _enumerated(nn, lambda: nn.eloc_table(S, T, dev(d["keys"][:m]), None, dev(la[:m]), dev(d["phase"][:m]),
                                                 with_energy=False))
    chk = np.arange(0, m, 3)
    ora, absum = _oracle(d, d["keys"], la, d["phase"], chk)
    assert np.abs(ora[::7]).max() > 1e200
    assert_eloc_close(eloc_complex(e)[chk], ora, absum, label="far below")


def test_batch(nn, n48):
    """Systems of one- and two-word keys, all enumerated: two schedules, the
    autotuner and graph replays."""
    print("[case] enumerated batch", flush=True)
    ds = [n48, synth.config_inputs(2, K=12, n_up=3, n_dn=3, n_unique=12000),
          synth.config_inputs(2, K=33, n_up=2, n_dn=2, n_unique=16000)]
    items = []
    for d in ds:
        S, n = _system(nn, d), len(d["keys"])
        items.append(dict(system=S, table=nn.Table(S, n), keys=dev(d["keys"]), logabs=dev(d["logabs"]),
                          phase=dev(d["phase"]), counts=dev(d["counts"], torch.int32),
                          eloc=torch.full((n, 2), np.nan, dtype=torch.float64, device="cuda"),
                          energy=torch.zeros(4, dtype=torch.float64, device="cuda")))
    B = nn.Batch(items)
    chk = [np.arange(0, len(d["keys"]), 97) for d in ds]
    refs = [_oracle(d, d["keys"], d["logabs"], d["phase"], c) for d, c in zip(ds, chk)]

    def check(label):
        for it, c, (ora, absum) in zip(items, chk, refs):
            assert_eloc_close(eloc_complex(it["eloc"])[c], ora, absum, label=label)

    for tune in (dict(search=1, splitter_levels=10, tile_samples=64), dict(search=2, splitter_levels=12, tile_samples=1024)):
        B.set_tune(**tune)
        _enumerated(nn, B.run, BATCH)
        check(str(tune))
    tune, ms = _enumerated(nn, lambda: B.autotune(reps=1), BATCH)
    assert tune["waves_per_block"] in (8, 12) and tune["tile_samples"] in (64, 256, 1024) and B.get_tune() == tune
    st = torch.cuda.Stream()
    B.run(st)
    st.synchronize()
    want = [it["eloc"].clone() for it in items]
    B.capture(st)
    for _ in range(3):
        for it in items:
            it["eloc"].fill_(np.nan)
        torch.cuda.synchronize()
        B.launch(st)
        st.synchronize()
        assert all(torch.equal(it["eloc"], w) for it, w in zip(items, want))
    check("replayed")

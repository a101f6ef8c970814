"""Which of the two sample-aware paths a call takes, by the launches the
library's timing records, and the result of either against the oracle.

Few samples against a table that is large for their number of connections are
enumerated: a scan is spread over no more than four waves per sample.  With many
connections and a table that fills the filter they are scanned all the same."""
import functools

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import assert_eloc_close, dev, eloc_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


def launches(nn, names, call):
    """What `call` returns, and the recorded launches of each name."""
    nn.timing_enable(True)
    try:
        r = call()
        torch.cuda.synchronize()
        return r, [nn.timing_read(k)[1] for k in names]
    finally:
        nn.timing_enable(False)


@pytest.fixture(scope="module")
def sector():
    """Every determinant of K = 12, 4 up and 4 down (C = 1,425), in random order."""
    d = synth.config_inputs(1, K=12, n_up=4, n_dn=4)
    p = np.random.default_rng([16705, 95]).permutation(len(d["keys"]))
    for k in ("keys", "logabs", "phase", "counts"):
        d[k] = np.ascontiguousarray(d[k][p])
    return d


def _check_path(nn, d, members, n, scans, checked):
    K, nu, nd = d["K"], d["n_up"], d["n_dn"]
    S = nn.System(d["N"], nu, nd, d["h"], d["g"], d["e_core"])
    T = nn.Table(S, members)
    keys, la, ph = d["keys"], d["logabs"], d["phase"]
    T.build(dev(keys[:members]), dev(la[:members]), dev(ph[:members]))
    (e, _), got = launches(nn, ("k_eloc_scan", "k_eloc_sa"), lambda: nn.eloc_table(
        S, T, dev(keys[:n]), None, dev(la[:n]), dev(ph[:n]), with_energy=False))
    assert got == ([1, 0] if scans else [0, 1])
    chk = np.linspace(0, n - 1, min(n, checked)).astype(np.int64)
    ora, absum = oracle.eloc_table(K, nu, nd, d["h"], d["g"], d["e_core"], keys[:members], la[:members], ph[:members],
                                   keys[chk], la[chk], ph[chk], with_absum=True)
    assert_eloc_close(eloc_complex(e)[chk], ora, absum, label=f"{n} of {members}")


@pytest.mark.parametrize("members,n,scans", [(1, 1, True), (40000, 1, True), (40000, 256, True), (150000, 1, False),
                                             (240000, 3, False), (150000, 256, False), (12000, 2048, True),
                                             (24000, 2048, False), (60000, 2048, False), (7000, 2049, True),
                                             (7000, 20000, True), (14000, 2049, False), (20000, 14000, False)])
def test_the_rule(nn, sector, members, n, scans):
    print(f"[case] path of {n} samples, {members} members", flush=True)
    _check_path(nn, sector, members, n, scans, 100)


@functools.lru_cache(maxsize=1)
def _inputs(K, nu, nd, members):
    return synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=members)


@pytest.mark.parametrize("K,nu,nd,members,n,scans", [(24, 6, 6, 120000, 1, True), (24, 6, 6, 120000, 300, True),
                                                     (24, 6, 6, 120000, 2049, False), (36, 4, 4, 100000, 1, True),
                                                     (36, 4, 4, 100000, 2048, True), (36, 4, 4, 100000, 2049, False)])
def test_many_connections(nn, K, nu, nd, members, n, scans):
    d = _inputs(K, nu, nd, members)
    print(f"[case] path of K={K}, {n} samples, {members} members", flush=True)
    _check_path(nn, d, members, n, scans, 20)


def test_autotuners_keep_a_schedule_that_changes_nothing(nn):
    """Scanned tables: timing schedules would pick one by chance."""
    d = synth.config_inputs(2, K=24, n_up=6, n_dn=6, n_unique=3000)
    print("[case] autotuners on scanned tables", flush=True)
    S = nn.System(d["N"], 6, 6, d["h"], d["g"], d["e_core"])
    keys, la, ph = dev(d["keys"]), dev(d["logabs"]), dev(d["phase"])
    T = nn.Table(S, 3000)
    T.set_tune(waves_per_block=5, splitter_levels=9, search=2, filter_log2_bits=15)
    before = T.get_tune()
    (tune, ms), got = launches(nn, ("k_eloc_scan", "k_eloc_sa"), lambda: T.autotune(keys, la, ph, reps=2))
    assert tune == before and T.get_tune() == before and 0.0 < ms < 1e3
    assert got == [3, 0]
    item = dict(system=S, table=T, keys=keys, logabs=la, phase=ph, counts=dev(d["counts"], torch.int32),
                eloc=torch.empty((3000, 2), dtype=torch.float64, device="cuda"),
                energy=torch.empty(4, dtype=torch.float64, device="cuda"))
    B = nn.Batch([item])
    B.set_tune(waves_per_block=6, splitter_levels=7, tile_samples=33)
    before = B.get_tune()
    (tune, ms), got = launches(nn, ("k_eloc_scan_batch", "k_eloc_sa_batch"), lambda: B.autotune(reps=2))
    assert tune == before and B.get_tune() == before and 0.0 < ms < 1e3
    assert got == [3, 0]

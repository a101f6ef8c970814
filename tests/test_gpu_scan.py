"""Sample-aware energies by scanning the table against the enumeration: the
same table and samples in a call of few samples (scanned) and of many
(enumerated), with members of other sectors among them, and samples that are
not members or lie far below the largest amplitude.

Both add the same FP64 terms with compensated sums in another order: 1e-12 of
max(1, |E|).  Small tables on either side of 64 and 256 members against the
oracle, as the other sample-aware tests."""
import numpy as np
import pytest
import torch

import oracle
import synth
from synth.gen import sector_size
from tests.gpu_util import assert_eloc_close, dev, eloc_complex, keys_np
from tests.test_gpu_batch import _items
from tests.test_gpu_sample_aware import _eloc_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


@pytest.mark.parametrize("tune", [{}, dict(search=2), dict(waves_per_block=16), dict(waves_per_block=8, search=2, filter_log2_bits=12,
                                                                                splitter_levels=3)])
@pytest.mark.parametrize("K,nu,nd,n", [(12, 3, 3, 16000), (40, 2, 2, 24000)])
def test_scan_equals_enumeration(nn, K, nu, nd, n, tune):
    print(f"[case] scan vs enumeration K={K} n={n} {tune}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=n)
    keys, la, ph = d["keys"][:n].copy(), d["logabs"][:n].copy(), d["phase"][:n]
    la[7::501] -= 650.0  # the exact ratio's samples
    S = nn.System(d["N"], nu, nd, d["h"], d["g"], d["e_core"])
    T = nn.Table(S, n + 4)
    T.set_tune(**tune)
    # members one spin flip away from a sample: other sectors, never connected
    other = keys[:4].copy()
    for r in range(4):
        x = int(other[r, 0]) | int(other[r, 1]) << 64
        up = next(p for p in range(0, 2 * K, 2) if x >> p & 1)
        dn = next(p for p in range(1, 2 * K, 2) if not x >> p & 1)
        x ^= 1 << up | 1 << dn
        other[r] = np.uint64(x & (1 << 64) - 1), np.uint64(x >> 64)
    tk = np.concatenate([keys[n // 10:], other])  # the first tenth of the samples are no members
    T.build(dev(tk), dev(np.concatenate([la[n // 10:], la[:4]])), dev(np.concatenate([ph[n // 10:], ph[:4]])))
    many, _ = nn.eloc_table(S, T, dev(keys), None, dev(la), dev(ph), with_energy=False)
    many = eloc_complex(many)
    for a, b in ((0, 1), (0, 65), (n // 10 - 9, n // 10 + 40), (n - 700, n)):
        few, _ = nn.eloc_table(S, T, dev(keys[a:b]), None, dev(la[a:b]), dev(ph[a:b]), with_energy=False)
        few = eloc_complex(few)
        assert np.all(np.abs(few - many[a:b]) <= 1e-12 * np.maximum(1.0, np.abs(many[a:b]))), (a, b)


@pytest.mark.parametrize("search", [1, 2])
def test_batch_of_scanned_and_enumerated_systems(nn, search):
    print(f"[case] mixed batch search={search}", flush=True)
    specs = [dict(K=12, n_up=3, n_dn=3, n_unique=16000), dict(K=24, n_up=6, n_dn=6, n_unique=500),
             dict(K=40, n_up=2, n_dn=2, n_unique=24000)]
    items = _items(nn, specs)
    B = nn.Batch(items)
    B.set_tune(search=search)
    B.run()
    for it in items:
        whole = eloc_complex(it["eloc"])
        for a in (0, 8000, 15900):
            k, l, p = (it[key][a:a + 64].contiguous() for key in ("keys", "logabs", "phase"))
            if len(k) == 0:
                continue
            few, _ = nn.eloc_table(it["system"], it["table"], k, None, l, p, with_energy=False)
            want = whole[a:a + len(k)]
            assert np.all(np.abs(eloc_complex(few) - want) <= 1e-12 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("K,nu,nd", [(6, 2, 3), (33, 3, 2)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257])
def test_small_tables_match_the_oracle(nn, K, nu, nd, n):
    print(f"[case] scan K={K} n={n}", flush=True)
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=min(n, sector_size(K, nu, nd)))
    S, T, g, ora, absum, ci, en = _eloc_case(nn, d)
    assert_eloc_close(g, ora, absum, label=f"K={K} n={n}")


@pytest.mark.parametrize("n", [1, 2, 64, 65, 1000, 8191, 8192, 8193])
def test_table_order_on_both_sorts(nn, n):
    """Tables on either side of the largest that is sorted by counting, with a
    key given twice from n = 64 on (the first given comes first)."""
    print(f"[case] table order n={n}", flush=True)
    d = synth.config_inputs(2, K=40, n_up=4, n_dn=3, n_unique=n)
    keys, la, ph = d["keys"].copy(), d["logabs"], d["phase"]
    if n >= 64:
        keys[n - 1] = keys[3]
    T = nn.Table(nn.System(d["N"], 4, 3, d["h"], d["g"], d["e_core"]), n)
    T.build(dev(keys), dev(la), dev(ph))
    k, l, p = T.export()
    order = np.lexsort((np.arange(n), keys[:, 0], keys[:, 1]))
    assert (keys_np(k) == keys[order]).all()
    assert (l.cpu().numpy() == la[order]).all() and (p.cpu().numpy() == ph[order]).all()
    if n < 64:
        assert oracle.sort_table(keys, la, ph)[3] and T.status() == 0
    else:
        assert T.status() != 0

"""Memory of batch sampling: what models keep between calls, what is left after
a call that ran out, and sampling without cached rows where memory is short
(the rest of the GPU's memory is held by a tensor meanwhile)."""
import ctypes

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module")
def nn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2306_16705_amd as nn
    return nn


def _model(nn, K, nu, nd):
    d = synth.config_inputs(2, K=K, n_up=nu, n_dn=nd, n_unique=2, model=True, beta=0.05)
    return nn.Model(d["model_shape"], nu, nd, d["weights"])


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_models_together_keep_eight_gib(nn):
    """Each of the three calls takes about 3 GiB; afterwards the three models
    hold 8 GiB at most (and 64 MB of other growth is allowed for)."""
    print("[case] workspaces of three models", flush=True)
    models = [_model(nn, 40, 10, 10) for _ in range(3)]
    nn.bas(models[0], 100, 1, nn.NNQS_BF16)
    before = _free()
    got = []
    for M in models:
        r = nn.bas(M, 100000, 3, nn.NNQS_BF16, capacity=100000)
        got.append([t.cpu() for t in r])
        del r
        print(f"{len(got[-1][0])} unique, {(before - _free()) / MB:.0f} MB held", flush=True)
    assert before - _free() <= 8192 * MB + 64 * MB
    for r in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(r, got[0]))
    for M in models:
        M.close()
    assert before - _free() <= 64 * MB


def test_nothing_is_held_after_running_out(nn):
    """20 million samples of a flat model with 2 GB free: the levels of their
    prefixes do not fit, and the call leaves what it found."""
    print("[case] sampling out of memory", flush=True)
    M = _model(nn, 24, 8, 8)
    nn.model_logpsi(M, nn.bas(M, 5000, 1, nn.NNQS_BF16)[0], nn.NNQS_BF16)  # both forwards have run
    ns = 20_000_000
    keys = torch.empty((ns, 2), dtype=torch.int64, device="cuda")
    cnt = torch.empty(ns, dtype=torch.int32, device="cuda")
    la = torch.empty(ns, dtype=torch.float64, device="cuda")
    hold = torch.empty(_free() - 2048 * MB, dtype=torch.uint8, device="cuda")
    before = _free()
    from paper_2306_16705_amd import _lib as L
    n = ctypes.c_int64()
    p = [ctypes.c_void_p(t.data_ptr()) for t in (keys, cnt, la)]
    with pytest.raises(nn.NNQSError) as ei:
        L.check(L.load().nnqs_bas(M.handle, nn.NNQS_BF16, 1, ns, ns, *p, None, ctypes.byref(n), None))
    after = _free()
    print(f"{before / MB:.0f} MB free before, {after / MB:.0f} after", flush=True)
    assert ei.value.code == -5 and before - after <= 64 * MB
    del hold
    _free()
    k, c, _, _ = nn.bas(M, 5000, 1, nn.NNQS_BF16)
    assert int(c.sum()) == 5000


def test_whole_prefixes_where_rows_do_not_fit(nn):
    """The same samples, counts and log-amplitudes, bit for bit, with rows and
    (4 GB free) with whole prefixes from the position on at which the paths or
    rows would take more than a quarter of what is free."""
    print("[case] sampling without rows", flush=True)
    ns = 2_000_000
    args = (ns, 7, nn.NNQS_BF16)

    def run(M):
        nn.timing_enable(True)
        r = [t.cpu() for t in nn.bas(M, *args, capacity=ns)]
        n = [nn.timing_read(k)[1] for k in ("k_transformer_rows", "k_transformer_bf16")]
        nn.timing_enable(False)
        return r, n

    first, n = run(_model(nn, 17, 8, 8))
    assert n == [17, 0]
    M = _model(nn, 17, 8, 8)
    nn.model_logpsi(M, nn.bas(M, 100, 1, nn.NNQS_BF16)[0], nn.NNQS_BF16)
    hold = torch.empty(_free() - 4096 * MB, dtype=torch.uint8, device="cuda")
    short, n = run(M)
    del hold
    _free()
    print(f"{len(first[0])} unique, {n} launches", flush=True)
    assert n[0] >= 5 and n[1] >= 1 and sum(n) == 17
    assert all(torch.equal(a, b) for a, b in zip(first, short))

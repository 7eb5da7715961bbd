"""The selection of the attention-free policy from a list of the positions that can be retained, against the oracle.

ta_evict takes this form for rows of more than 4096 positions where no score ranks the plain ones, ta_select for more than 8192.
Its edges: rows whose length does not divide into loads of flags, words with every flag set, a list that just holds and one that does not hold what is
flagged (the whole row is then taken), budgets that leave no plain slot, lengths below the budget, and ties.
"""
import numpy as np
import pytest
import torch

import paper_2604_11288_amd as ta
from oracle import ta_oracle as ora

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TABLE = (np.array([[1, -1, -1, -1], [2, 3, -1, -1]], np.int32), np.array([1, 2], np.int32))


def _tokens(n, share, rng):
    """Filler with about `share` anchors, single tokens and pairs."""
    tok = rng.integers(10, 1000, n).astype(np.int32)
    hit = rng.random(n) < share
    tok[hit] = rng.choice(np.array([1, 2, 3], np.int32), int(hit.sum()))
    return tok


@pytest.mark.parametrize("n,K,share,kw", [
    (16, 6, 0.1, {}), (17, 8, 0.2, {}), (31, 12, 0.05, {}), (33, 12, 0.0, {}),
    (4096, 64, 0.002, {}), (4097, 300, 0.01, {}), (8191, 512, 0.003, {}), (8193, 64, 0.05, {}),    # 0.05: more sponsored than slots
    (16385, 1024, 0.001, {}), (32768, 512, 0.001, {}), (32767, 2048, 0.002, {}), (32768, 4000, 0.0, {}),
    (32768, 512, 0.02, {}), (32768, 512, 0.0185, {}),                                  # about as many flagged as the list holds
    (20000, 700, 1.0, {}), (32768, 512, 0.5, {}), (4096, 64, 1.0, {}),                 # far more
    (32769, 512, 0.001, {}), (65537, 1024, 0.002, {}), (98304, 300, 0.0, {}), (131072, 1024, 0.001, {}), (131071, 64, 0.005, {}),     # two to four segments
    (131072, 512, 0.2, {}), (131072, 512, 0.0047, {}), (131073, 512, 0.001, {}),       # more than the list holds, about as many; a longer row
    (5000, 100, 0.004, dict(n_recent=96)), (5000, 100, 0.004, dict(n_sink=0, n_recent=0)),
    (5000, 200, 0.004, dict(beta=0.0)), (5000, 200, 0.004, dict(beta=0.0, gamma=0.0)),             # ties: the position decides
    (5000, 200, 0.004, dict(beta=-0.5)), (5000, 200, 0.004, dict(gamma=-0.1)),                     # taken by the whole row
])
def test_attention_free_selection(n, K, share, kw):
    rng = np.random.default_rng(n + K)
    lens = np.array([n, max(1, n - 5), max(1, n // 3), min(n, K), 3], np.int32)
    tok = np.stack([_tokens(n, share, rng) for _ in lens])
    prm = ta.Params(alpha=0.0, **{**dict(n_sink=min(4, K // 2), n_recent=min(4, K // 2)), **kw})
    rows = [torch.randn((1, len(lens), 1, n, 128), generator=torch.Generator().manual_seed(s)).to(torch.bfloat16).to(DEV) for s in (1, 2)]
    plan = ta.EvictPlan(torch.from_numpy(tok).to(DEV), *TABLE, None, *rows, K, prm, seq_len=torch.from_numpy(lens).to(DEV))
    plan.run()
    torch.cuda.synchronize()
    idx, cnt = plan.idx.cpu().numpy().reshape(len(lens), K), plan.cnt.cpu().numpy().reshape(len(lens))
    for b, nb in enumerate(lens):
        a, s, v = ora.evict_sequence(tok[b, :nb], *TABLE)
        ref = ora.select(None, a, s, v, K, prm.n_sink, prm.n_recent, alpha=0.0, beta=prm.beta, gamma=prm.gamma)
        assert cnt[b] == len(ref) == min(K, nb)
        assert np.array_equal(idx[b, :len(ref)], ref), (b, nb)
        keep = torch.from_numpy(ref.astype(np.int64)).to(DEV)
        for got, src in ((plan.Kout, rows[0]), (plan.Vout, rows[1])):
            assert torch.equal(got[0, b, 0, :len(ref)].view(torch.int16), src[0, b, 0].index_select(0, keep).view(torch.int16))


@pytest.mark.parametrize("n,K,layers,hkv", [
    (257, 40, 2, 3), (8193, 300, 1, 2), (16387, 64, 2, 1), (20001, 512, 1, 1), (32768, 4000, 1, 1), (32771, 512, 1, 2), (131072, 1024, 1, 1),
])
@pytest.mark.parametrize("vouchers", ["sparse", "below zero in front", "below zero at the end", "none at the end", "everywhere", "at the ends"])
def test_selection_with_any_vouchers(n, K, layers, hkv, vouchers):
    """ta_select without scores, on vouchers that neither the match nor the expansion wrote."""
    rng = np.random.default_rng(n + K)
    lens = np.array([n, max(1, n - 3), max(1, n // 2)], np.int32)
    B = len(lens)
    a, s = (rng.random((B, n)) < p for p in (0.002, 0.004))
    v = np.where(rng.random((B, n)) < (0.9 if vouchers == "everywhere" else 0.003), rng.random((B, n)) * 2, 0.0).astype(np.float32)
    for b, nb in enumerate(lens):
        if vouchers == "below zero in front":
            v[b, : nb // 4 : 3 if n < 1000 else 97] = -0.5
        elif vouchers == "below zero at the end":
            v[b, nb - max(1, K // 2)] = -3.0
        elif vouchers == "none at the end":
            v[b, nb - max(1, K // 2)] = np.nan
        elif vouchers == "at the ends":
            v[b, [0, nb - 1, max(0, nb - K), max(0, nb - K - 1)]] = 5.0
    prm = ta.Params(alpha=0.0, n_sink=min(4, K // 3), n_recent=min(4, K // 3))
    dev = [torch.from_numpy(x).to(DEV) for x in (a.astype(np.uint8), s.astype(np.uint8), v)]
    idx, cnt = ta.ta_select(None, *dev, K, prm, layers, hkv, seq_len=torch.from_numpy(lens).to(DEV))
    idx, cnt = idx.cpu().numpy().reshape(layers, B, hkv, K), cnt.cpu().numpy().reshape(layers, B, hkv)
    if vouchers == "none at the end":                      # not a number: what the form without a list does (margin output asked for)
        full = ta.Params(alpha=0.0, n_sink=prm.n_sink, n_recent=prm.n_recent, margin=torch.zeros((layers, B, hkv, 2), device=DEV))
        ref = ta.ta_select(None, *dev, K, full, layers, hkv, seq_len=torch.from_numpy(lens).to(DEV))[0].cpu().numpy().reshape(layers, B, hkv, K)
    for b, nb in enumerate(lens):
        want = (ref[0, b, 0, :min(K, nb)] if vouchers == "none at the end" else
                ora.select(None, a[b, :nb], s[b, :nb], v[b, :nb], K, prm.n_sink, prm.n_recent, alpha=0.0, beta=prm.beta, gamma=prm.gamma))
        assert (cnt[:, b] == len(want)).all()
        assert (idx[:, b, :, :len(want)] == want).all(), (b, nb)


@pytest.mark.parametrize("n,K,flagged,vouchers", [
    (8193, 300, 0.9, 0.003), (16387, 64, 0.5, 0.003), (32768, 512, 0.2, 0.9), (131072, 64, 0.05, 0.003),     # the flags alone fill the list
    (32768, 512, 0.12, 0.0), (32768, 512, 0.11, 0.01), (32768, 512, 0.1, 0.1), (131071, 512, 0.03, 0.0),     # about as many; vouchers as well
])
def test_selection_with_many_flags_and_any_vouchers(n, K, flagged, vouchers):
    rng = np.random.default_rng(n + K)
    lens = np.array([n, n - 1, n // 2 + 1], np.int32)
    a, s = rng.random((3, n)) < flagged / 8, rng.random((3, n)) < flagged
    v = np.where(rng.random((3, n)) < vouchers, rng.random((3, n)) * 2, 0.0).astype(np.float32)
    prm = ta.Params(alpha=0.0)
    dev = [torch.from_numpy(x).to(DEV) for x in (a.astype(np.uint8), s.astype(np.uint8), v)]
    idx, cnt = (x.cpu().numpy().reshape(3, -1) for x in ta.ta_select(None, *dev, K, prm, 1, 1, seq_len=torch.from_numpy(lens).to(DEV)))
    for b, nb in enumerate(lens):
        want = ora.select(None, a[b, :nb], s[b, :nb], v[b, :nb], K, prm.n_sink, prm.n_recent, alpha=0.0, beta=prm.beta, gamma=prm.gamma)
        assert cnt[b, 0] == len(want) and np.array_equal(idx[b], want), (b, nb)

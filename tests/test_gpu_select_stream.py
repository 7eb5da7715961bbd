"""The streaming form of step 4 (one read of every input, candidate list in LDS) against the oracle.

ta_select picks that form for rows longer than a workgroup's registers hold and for launches of many units;
these cases reach it at sizes the oracle finishes in seconds, on inputs chosen to drive its
branches: repeated cuts of the list (utilities that grow towards the start of the sequence, so
every segment of the walk beats the threshold), thousands of exact ties (position passes), pool
overflow, no mandatory class, ragged lengths below and above the budget, per-layer budgets, and
budgets whose list does not fit (those fall back to the kernel that recomputes its keys and must agree as well).
The register form, which takes the shorter rows of fewer units, is tested at its limits further down.
"""
import numpy as np
import pytest
import torch

import paper_2604_11288_amd as ta
from oracle import ta_oracle as ora
from paper_2604_11288_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _inputs(n, batch, planted, ragged, seed):
    w = wl.scaled(wl.CONFIGS["c2_full_model"], n=n, batch=batch, planted=planted, ragged=ragged)
    td = wl.make_tokens(w, clean=False)
    seqs = []
    for b in range(batch):
        nb = int(td.seq_len[b])
        seqs.append(ora.evict_sequence(td.tok[b, :nb], td.tab_ids, td.tab_len))
    return w, td, seqs


def _scores(mode, shape, rng):
    n = shape[-1]
    if mode == "uniform":
        return (rng.random(shape) * 4).astype(np.float32)
    if mode == "ties":
        return np.round(rng.random(shape) * 4, 1).astype(np.float32)
    if mode == "zeros":
        return np.zeros(shape, np.float32)
    if mode == "early":                # large scores at the start: the walk from the end keeps finding better positions
        return (np.linspace(8.0, 0.0, n, dtype=np.float32)[None, None, None, :] + rng.random(shape).astype(np.float32) * 0.01).astype(np.float32)
    raise ValueError(mode)


def _check(layers, batch, hkv, n, K, ns, nr, mode, planted=8, ragged=None, beta=0.5, layer_K=None, sample=None, seed=0):
    w, td, seqs = _inputs(n, batch, planted, ragged, seed)
    rng = np.random.default_rng(1000 * n + K + seed)
    A = _scores(mode, (layers, batch, hkv, n), rng)
    lk = None if layer_K is None else _dev(np.asarray(layer_K, np.int32))
    margin = torch.full((layers, batch, hkv, 2), 123.0, device=DEV)
    prm = ta.Params(n_sink=ns, n_recent=nr, beta=beta, layer_K=lk, margin=margin)
    seq = _dev(td.seq_len) if ragged else None
    anchor, spons, vouch = ta.ta_match_anchors(_dev(td.tok), td.tab_ids, td.tab_len, prm, seq_len=seq)
    idx, cnt = ta.ta_select(_dev(A), anchor, spons, vouch, K, prm, layers, hkv, seq_len=seq)
    torch.cuda.synchronize()
    idx, cnt, margin = idx.cpu().numpy(), cnt.cpu().numpy(), margin.cpu().numpy()
    units = [(l, b, h) for l in range(layers) for b in range(batch) for h in range(hkv)]
    if sample is not None and sample < len(units):
        pick = np.random.default_rng(seed + 5).choice(len(units), size=sample, replace=False)
        units = [units[i] for i in sorted(pick)] + [units[0], units[-1]]
    for (l, b, h) in units:
        nb = int(td.seq_len[b])
        a, s, v = seqs[b]
        Kl = K if layer_K is None else min(K, max(int(layer_K[l]), ns + nr, 1))
        ref = ora.select(A[l, b, h, :nb], a, s, v, Kl, ns, nr, alpha=1.0, beta=beta, gamma=0.3)
        assert cnt[l, b, h] == len(ref) == min(Kl, nb), (l, b, h)
        assert np.array_equal(idx[l, b, h, :len(ref)], ref), (l, b, h)
        # the margin of the cut: the same two utilities, bit for bit
        want = ora.select_margin(A[l, b, h, :nb], a, s, v, Kl, ns, nr, alpha=1.0, beta=beta, gamma=0.3)
        assert margin[l, b, h].tolist() == want.tolist(), (l, b, h, margin[l, b, h], want)
    return len(units)


@pytest.mark.parametrize("n,K,ns,nr,mode,planted", [
    (1500, 64, 4, 4, "uniform", 8),
    (1500, 16, 4, 4, "uniform", 8),      # pool overflow: more sponsored positions than protected slots
    (2048, 256, 4, 8, "ties", 8),        # exact ties at the threshold: position passes
    (1028, 100, 0, 0, "zeros", 4),       # no mandatory class, recency alone decides
    (3000, 700, 4, 64, "early", 8),      # every segment of the walk beats the threshold: a cut per segment
])
def test_streaming_select_many_units(n, K, ns, nr, mode, planted):
    # 16 x 16 x 8 = 2048 units: ta_select takes the streaming form on short rows from 1024 on
    checked = _check(16, 16, 8, n, K, ns, nr, mode, planted=planted, sample=300)
    assert checked >= 300


def test_streaming_select_ragged_many_units():
    # lengths from below the budget (nothing to evict) to several segments, 4-aligned padded rows
    _check(16, 16, 8, 2600, 128, 4, 16, "uniform", ragged=(40, 2600), sample=400)


def test_streaming_select_negative_recency_weight():
    # beta < 0 reverses the recency order: the walk from the end meets the worst positions first
    _check(16, 16, 8, 2304, 200, 4, 4, "uniform", beta=-0.5, sample=200)


def test_streaming_select_per_layer_budgets():
    layers = 16
    lk = [max(12, 300 - 18 * l) for l in range(layers)]
    _check(layers, 16, 8, 1800, 300, 4, 8, "uniform", layer_K=lk, sample=300)


@pytest.mark.parametrize("n,K,mode", [
    (70000, 1024, "early"),              # long rows, dozens of cuts of the list
    (131072, 1024, "uniform"),           # the long-context row length
    (50000, 4000, "ties"),               # list of more than 4000 entries
    (40000, 7000, "uniform"),            # the list would not fit: keys recomputed in every pass, same answer
])
def test_streaming_select_long_rows(n, K, mode):
    _check(1, 2, 3, n, K, 4, 128, mode, planted=40)


@pytest.mark.parametrize("n,K,ns,nr,mode", [
    (2, 1, 0, 1, "uniform"), (3, 2, 1, 1, "zeros"), (5, 4, 0, 0, "ties"), (37, 9, 4, 4, "uniform"),   # rows of less than a quad and a few
    (1023, 300, 4, 4, "ties"),           # rows of a batch at every alignment
    (4095, 64, 4, 4, "uniform"), (4096, 4000, 4, 4, "zeros"), (4097, 1024, 4, 4, "early"),              # one round of quads and one position more
    (8193, 2000, 0, 64, "ties"), (16385, 512, 4, 4, "uniform"), (32767, 16, 4, 4, "zeros"), (32768, 1024, 4, 128, "uniform"),
    (33001, 700, 4, 4, "uniform"),       # streaming form, rows at odd addresses
])
def test_register_select_at_its_limits(n, K, ns, nr, mode):
    _check(1, 3, 2, n, K, ns, nr, mode, planted=3 if n > 300 else 0)


@pytest.mark.parametrize("n,layers", [(1337, 64), (2050, 64)])
def test_streaming_select_rows_at_odd_addresses(n, layers):
    _check(layers, 4, 4, n, 120, 4, 8, "uniform", ragged=(100, n), sample=150)     # 1024 units


@pytest.mark.parametrize("layers,n,K,low", [(32, 2049, 640, 100), (33, 2049, 640, 2049), (33, 4097, 900, 500), (34, 8192, 639, 8000), (64, 2303, 700, 600), (65, 2303, 700, 600)])
def test_many_units_with_lengths_on_both_sides_of_the_line(layers, n, K, low):
    """Larger budgets: registers up to 2048 units, the walk beyond; below 640 the walk from 1025 units on."""
    _check(layers, 4, 8, n, K, 4, 8, "ties" if n == 4097 else "uniform", ragged=(low, n), sample=60)


@pytest.mark.parametrize("spread", [1e-30, 1.0, 1e30])
def test_register_select_with_outliers_and_crowded_bins(spread):
    # nearly all keys in one bin of the first level (a few values far away), then exact ties among thousands
    rng = np.random.default_rng(7)
    n, K = 12000, 900
    A = (1.0 + rng.integers(0, 4, (1, 1, 4, n)) * 1e-6).astype(np.float32)
    A[0, 0, :, rng.integers(0, n, 5)] = spread
    A[0, 0, 1, 100:200] = -spread
    A[0, 0, 2] = np.float32(0.25)
    zero8, zerof = np.zeros((1, n), np.uint8), np.zeros((1, n), np.float32)
    prm = ta.Params(n_sink=2, n_recent=3, beta=0.0)
    idx, cnt = ta.ta_select(_dev(A), _dev(zero8), _dev(zero8), _dev(zerof), K, prm, 1, 4)
    idx = idx.cpu().numpy()
    for h in range(4):
        ref = ora.select(A[0, 0, h], zero8[0], zero8[0], zerof[0], K, 2, 3, alpha=1.0, beta=0.0, gamma=0.3)
        assert np.array_equal(idx[0, 0, h], ref)


@pytest.mark.parametrize("n,K", [(900, 40), (4097, 256), (20001, 512), (32768, 512), (40002, 512)])
@pytest.mark.parametrize("vouchers", ["sponsored", "any", "negative"])
def test_attention_free_select_with_any_vouchers(n, K, vouchers):
    # anchors and vouchers anywhere, on unsponsored positions too; negative vouchers turn the recency order round
    rng = np.random.default_rng(n + K)
    anchor = (rng.random((2, n)) < 0.004).astype(np.uint8)
    spons = (rng.random((2, n)) < 0.004).astype(np.uint8)
    vouch = np.where(spons != 0, rng.random((2, n)) * 9, 0.0).astype(np.float32)
    if vouchers == "any":
        vouch += np.where(rng.random((2, n)) < 0.002, 0.7, 0.0).astype(np.float32)
    if vouchers == "negative":
        vouch[1] -= np.where(rng.random(n) < 0.9, 0.9, 0.0).astype(np.float32)
    prm = ta.Params(n_sink=4, n_recent=8, alpha=0.0)
    idx, cnt = ta.ta_select(None, _dev(anchor), _dev(spons), _dev(vouch), K, prm, 1, 1)
    idx = idx.cpu().numpy()
    for b in range(2):
        ref = ora.select(None, anchor[b], spons[b], vouch[b], K, 4, 8, alpha=0.0)
        assert np.array_equal(idx[0, b, 0], ref)


@pytest.mark.parametrize("n,K,planted,beta,gamma", [(900, 40, 3, 0.5, 0.3), (4097, 256, 12, 0.5, 0.3), (20001, 512, 200, 0.5, 0.3),
                                                    (20001, 64, 200, 0.5, 0.3), (32768, 512, 30, 0.0, 0.0), (32767, 512, 30, 0.5, -0.4),
                                                    (9000, 512, 30, -0.5, 0.3)])
def test_attention_free_pass_skips_nothing_that_counts(n, K, planted, beta, gamma):
    # the pass does not rank plain positions that cannot be retained; anchors early in the sequence can be
    w, td, seqs = _inputs(n, 2, planted, (n // 2, n), 3)
    kv = torch.zeros((1, 2, 1, n, 128), dtype=torch.bfloat16, device=DEV)
    prm = ta.Params(n_sink=4, n_recent=8, alpha=0.0, beta=beta, gamma=gamma)
    plan = ta.ta_evict(_dev(td.tok), td.tab_ids, td.tab_len, None, kv, kv.clone(), K, prm, seq_len=_dev(td.seq_len))
    idx, cnt = plan.idx.cpu().numpy(), plan.cnt.cpu().numpy()
    for b in range(2):
        a, s, v = seqs[b]
        ref = ora.select(None, a, s, v, K, 4, 8, alpha=0.0, beta=beta, gamma=gamma)
        assert cnt[b] == len(ref) and np.array_equal(idx[b, :len(ref)], ref)


@pytest.mark.parametrize("K", [72, 73, 264, 265, 1032, 1033])     # slots beside the 8 mandatory ones: 64, 256, 1024 and one more
@pytest.mark.parametrize("n,mode,ragged", [
    (9000, "uniform", None), (20000, "ties", None), (16384, "early", None), (12000, "zeros", None),
    (30000, "uniform", (20, 30000)),                              # rows that leave most lanes without a position
])
def test_register_select_bound_of_the_cut(n, K, mode, ragged):
    """Rows of four and eight rounds leave out what lies below a bound taken from groups of 16, 4 and 1 lanes."""
    _check(2, 2, 3, n, K, 4, 4, mode, planted=6, ragged=ragged)


@pytest.mark.parametrize("layers,n,K,pool_k,mode,planted", [
    (1, 33003, 500, 1, "uniform", 40), (1, 45059, 64, 1, "early", 40),                 # sixteen wavefronts per unit, rows at odd addresses
    (1, 40001, 40, 1, "ties", 400), (1, 40001, 40, 5, "ties", 400),                    # more sponsored positions than slots
    (1, 36871, 700, 9, "early", 40), (1, 33000, 300, 3, "zeros", 40),
    (90, 32771, 200, 1, "uniform", 40), (90, 32771, 200, 7, "ties", 40),               # four wavefronts per unit
    (180, 5003, 30, 1, "ties", 60),                                                    # short rows of many units
])
def test_walk_without_margin(layers, n, K, pool_k, mode, planted):
    """The walk's segments between the mandatory ranges and at the rows' ends, in the instances that report no margin."""
    batch, hkv, ns, nr = 3, 2, 5, 9
    w, td, seqs = _inputs(n, batch, planted, (n - 1100, n), 3)
    A = _scores(mode, (layers, batch, hkv, n), np.random.default_rng(n + K))
    prm = ta.Params(n_sink=ns, n_recent=nr, pool_k=pool_k)
    seq = _dev(td.seq_len)
    anchor, spons, vouch = ta.ta_match_anchors(_dev(td.tok), td.tab_ids, td.tab_len, prm, seq_len=seq)
    idx, cnt = ta.ta_select(_dev(A), anchor, spons, vouch, K, prm, layers, hkv, seq_len=seq)
    idx, cnt = idx.cpu().numpy(), cnt.cpu().numpy()
    for l in (0, layers // 2, layers - 1):
        for b in range(batch):
            nb = int(td.seq_len[b])
            for h in range(hkv):
                row = A[l, b, h, :nb] if pool_k == 1 else ora.maxpool(A[l, b, h, :nb], pool_k)
                ref = ora.select(row, *seqs[b], K, ns, nr, alpha=1.0, beta=0.5, gamma=0.3)
                assert cnt[l, b, h] == len(ref)
                assert np.array_equal(idx[l, b, h, :len(ref)], ref), (l, b, h)

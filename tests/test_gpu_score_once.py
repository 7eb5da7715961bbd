"""Units of one chunk: both sweeps of the score step by the same workgroup, against the oracle.

A unit has one chunk where there are many units, or up to 192 keys (two chunks take four stages of 64).  The lengths lie around a stage, around
the window (the masked stages), and around the number of stages from which the main loop goes by whole turns (12 with 256 rows, 48 with up to 128).
"""
import numpy as np
import pytest
import torch

import paper_2604_11288_amd as ta
from oracle import ta_oracle as ora
from paper_2604_11288_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _close(got, ref):
    return np.all(np.abs(got - ref) <= 1e-3 * np.abs(ref) + 1e-7)


def _check(w, A, Q, K, lens, causal, units):
    G = w.hq // w.hkv
    for l, b, g in units:
        nb = int(lens[b])
        ref = ora.score(wl.bf16_bits(Q[l, b, g * G:(g + 1) * G]), wl.bf16_bits(K[l, b, g, :nb]), causal) if nb else np.zeros(0, np.float32)
        got = A[l, b, g].cpu().numpy()
        assert _close(got[:nb], ref), (l, b, g, nb)
        assert not got[nb:].any(), (l, b, g, nb)


@pytest.mark.parametrize("hq,window,n,lens", [
    (8, 16, 127, (127, 1, 64, 0)),            # 32 rows, fewer than 128 keys; an empty sequence
    (16, 32, 65, (65, 63, 33, 2)),            # 64 rows
    (32, 32, 100, (100, 32, 31, 99)),         # 128 rows; as many keys as window rows, one fewer
    (64, 32, 126, (126, 65, 5, 0)),           # 256 rows
    (32, 32, 128, (128, 127, 65, 64)),
    (8, 16, 192, (192, 191, 129, 128)),       # the longest of few units that have one chunk
    (32, 32, 192, (192, 191, 129, 128)),
    (64, 32, 192, (192, 191, 129, 128)),
    (32, 32, 193, (193, 192, 129, 0)),        # two chunks
])
def test_short_rows_match_the_oracle(hq, window, n, lens):
    w = wl.scaled(wl.CONFIGS["c1_single_layer"], layers=2, batch=4, n=n, hq=hq, hkv=8, window=window)
    Q, K, _ = wl.make_qkv(w, device=DEV, with_v=False)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    for causal in (True, False):
        A = torch.full((2, 4, 8, n), float("nan"), device=DEV)
        ta.ta_score(Q, K, ta.Params(causal=causal), seq_len=seq, A=A)
        _check(w, A, Q, K, lens, causal, [(l, b, g) for l in range(2) for b in range(4) for g in (0, 7)])


@pytest.mark.parametrize("hq,window,n,lens,paged", [
    (8, 32, 700, None, False),                # 32 rows, workgroups of two wavefronts
    (32, 32, 3008, (3008, 3007, 129, 0, 1500, 64, 2944, 31), False),      # 47 stages, ragged
    (32, 32, 3137, (3137, 3073, 3072, 128, 1, 700, 3136, 3000), False),   # 50 stages: whole turns
    (32, 32, 1500, (1500, 1499, 64, 63, 0, 800, 1472, 33), True),
    (64, 32, 704, None, False),               # 256 rows, 11 stages
    (64, 32, 833, (833, 768, 767, 40, 0, 64, 832, 500), True),            # 14 stages: whole turns
    # units longer than what the first sweep leaves to the cache (64 stages with 128 rows, 42 with 64), and units of just that length
    (32, 32, 4500, (4500, 4097, 4096, 4160, 4224, 100, 0, 4095), False),
    (32, 32, 4500, (4500, 4097, 4096, 4160, 4224, 100, 0, 4095), True),   # 71 pages: beyond 64 of a chunk the table is read
    (16, 32, 2900, (2900, 2753, 2752, 2689, 2688, 64, 0, 2687), False),   # 64 rows, workgroups of two wavefronts
    (8, 32, 4500, (4500, 4097, 4096, 2689, 2688, 64, 0, 4224), True),
])
def test_many_units_match_the_oracle(hq, window, n, lens, paged):
    w = wl.scaled(wl.CONFIGS["c1_single_layer"], layers=16, batch=8, n=n, hq=hq, hkv=8, window=window)
    Q, K, _ = wl.make_qkv(w, device=DEV, with_v=False)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV) if lens else None
    prm = ta.Params()
    if paged:
        ps = 64
        slots = (n + ps - 1) // ps
        table = torch.randperm(8 * slots, generator=torch.Generator().manual_seed(n)).to(torch.int32).view(8, slots)
        pool = torch.zeros((16, 8 * slots, ps, 8, 128), dtype=torch.bfloat16, device=DEV)
        rows = torch.zeros((16, 8, slots * ps, 8, 128), dtype=torch.bfloat16, device=DEV)
        rows[:, :, :n] = K.transpose(2, 3)
        pool[:, table.view(-1).long().to(DEV)] = rows.view(16, 8 * slots, ps, 8, 128)
        kv = ta.PagedKV(pool, pool, table.to(DEV), ps, 8 * slots, pool.stride()[:4], 16, 8, 8, n)
        A = ta.ta_score_paged(Q, kv, prm, seq_len=seq)
    else:
        A = ta.ta_score(Q, K, prm, seq_len=seq)
    _check(w, A, Q, K, lens or (n,) * 8, True, [(l, b, (3 * l + b) % 8) for l in (0, 9, 15) for b in range(8)])


@pytest.mark.parametrize("hq,layers,n,budget,form", [
    (32, 2, 190, 100, "dense"),               # keys for the cache, no hint: up to 128 MiB of keys, a third of them gathered
    (32, 2, 190, 64, "pages of 64"),          # 64 * 3 >= 190
    (32, 2, 190, 63, "pages of 64"),          # 63 * 3 < 190
    (32, 8, 1000, 400, "pages of 64"),        # 131 072 000 bytes of keys, just below the line
    (32, 8, 1048, 400, "pages of 64"),        # and 137 363 456, above it
    (32, 8, 3200, 64, "dense"),               # 50 stages: whole turns
    (32, 8, 3200, 64, "pages of 192"),        # a page size that is no power of two
    (32, 8, 700, 64, "layers"),
    (16, 8, 1100, 64, "pages of 64"),         # 64 rows: narrow workgroups, the match in front of them
    (16, 8, 4500, 64, "layers"),
    (64, 2, 190, 100, "pages of 64"),         # 256 rows, three stages
    (64, 4, 1000, 500, "dense"),              # 16 stages: whole turns
    (64, 4, 1000, 334, "pages of 64"),
    (64, 4, 1000, 333, "pages of 64"),
    (64, 8, 1100, 64, "layers"),
    (64, 16, 640, 64, "pages of 192"),        # ten stages
])
def test_whole_pass_over_units_of_one_chunk(hq, layers, n, budget, form):
    # the match rides along behind the units' workgroups
    w = wl.scaled(wl.CONFIGS["c2_full_model"], layers=layers, batch=8, n=n, hq=hq, hkv=8, window=32, planted=2)
    td = wl.make_tokens(w, clean=False)
    lens = (n, n - 1, 64, 129, 0, 31, n // 2, 128)
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    Q, K, V = wl.make_qkv(w, device=DEV)
    prm = ta.Params(n_sink=4, n_recent=4)
    tok = torch.from_numpy(td.tok).to(DEV)
    if form == "layers":
        plan = ta.LayerEvictPlan(tok, td.tab_ids, td.tab_len, list(Q), list(K), list(V), budget, prm, seq_len=seq)
    elif form != "dense":
        page_size = int(form.split()[-1])
        Kp, Vp, table, pages, strides = wl.make_paged(K, V, page_size)
        kv = ta.PagedKV(Kp, Vp, table, page_size, pages, strides, layers, 8, 8, n)
        plan = ta.EvictPlan(tok, td.tab_ids, td.tab_len, Q, None, None, budget, prm, seq_len=seq, paged=kv)
    else:
        plan = ta.EvictPlan(tok, td.tab_ids, td.tab_len, Q, K, V, budget, prm, seq_len=seq)
    plan.A.fill_(float("nan"))
    plan.run()
    units = [(l, b, (3 * l + b) % 8) for l in (0, layers - 1) for b in range(8)]
    _check(w, plan.A, Q, K, lens, True, units)
    for l, b, g in units:
        nb = lens[b]
        a, s, v = ora.evict_sequence(td.tok[b, :nb], td.tab_ids, td.tab_len) if nb else (np.zeros(0, np.uint8), np.zeros(0, np.uint8), np.zeros(0, np.float32))
        assert np.array_equal(plan.anchor[b, :nb].cpu().numpy(), a) and np.array_equal(plan.spons[b, :nb].cpu().numpy(), s), b
        assert np.array_equal(plan.vouch[b, :nb].cpu().numpy(), v), b
        sel = ora.select(plan.A[l, b, g, :nb].cpu().numpy(), a, s, v, budget, 4, 4) if nb else np.zeros(0, np.int32)
        c = int(plan.cnt[l, b, g])
        assert c == len(sel) and np.array_equal(plan.idx[l, b, g, :c].cpu().numpy(), sel), (l, b, g)
        rows = torch.from_numpy(sel).long().to(DEV)
        assert torch.equal(plan.Kout[l][b, g, :c], K[l, b, g][rows]) and torch.equal(plan.Vout[l][b, g, :c], V[l, b, g][rows]), (l, b, g)

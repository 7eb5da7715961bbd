"""A generation step as one launch: the state after every step equals the two-launch step's, bit for bit.

The two-launch step (no words to count in) is compared with the oracle in test_gpu_decode.py through the same binding where the
one-launch form does not run; here both run side by side, at the forms' limits: spans that one load of flags holds and one more,
positions at the start of a sequence, rankings that vouchers decide because no plain row is left, no mandatory rows or nothing else,
sequences that reach their capacity, group widths, pages, and steps that take turns.
"""
import copy

import numpy as np
import pytest
import torch

import paper_2604_11288_amd as ta
from paper_2604_11288_amd import binding as tb
from paper_2604_11288_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MARK = 32 * 8 + 1                  # the word with a bit per tile of positions; its highest belongs to none where there are fewer than 56: a step of one launch clears it
STATE = ("tok", "len", "anchor", "budget", "vouch", "spons", "pos", "A", "Kc", "Vc", "stepped")


def _state(layers, batch, hq, hkv, K, n, cap, prm, page_size, vocabulary, lens, seed):
    g = torch.Generator().manual_seed(seed)
    tok = torch.randint(0, vocabulary, (batch, n), generator=g, dtype=torch.int32).to(DEV)
    ids = np.full((16, 4), -1, np.int32)
    ids[:, 0] = np.arange(16)
    ids[8:, 1] = np.arange(8)
    tab_len = np.array([1] * 8 + [2] * 8, np.int32)
    seq_len = torch.tensor(lens, dtype=torch.int32, device=DEV)
    anchor, spons, vouch = ta.ta_match_anchors(tok, ids, tab_len, prm, seq_len=seq_len)
    A = torch.rand((layers, batch, hkv, n), generator=g).to(DEV)
    idx, cnt = ta.ta_select(A, anchor, spons, vouch, K, prm, layers, hkv, seq_len=seq_len)
    rows = [torch.randn((layers, batch, hkv, K, 128), generator=g).to(torch.bfloat16).to(DEV) for _ in range(2)]
    pages = None
    if page_size:
        Kp, Vp, table, num_pages, strides = wl.make_slot_pool(layers, batch, hkv, 128, K + 1, page_size, DEV)
        pages = ta.PagedKV(Kp, Vp, torch.from_numpy(table).to(DEV), page_size, num_pages, strides, layers, batch, hkv, K + 1)
    st = ta.DecodeState(layers, batch, hq, hkv, K, cap, DEV, pages=pages)
    ta.ta_decode_init(st, tok, anchor, idx, cnt, *rows, prm, seq_len=seq_len, A=A)
    return st, ids, tab_len


@pytest.mark.parametrize("shape,kw,vocabulary,page_size", [
    ((2, 1, 8, 2, 300, 900), {}, 400, 0), ((2, 2, 8, 2, 300, 900), {}, 400, 16), ((1, 1, 4, 1, 600, 1500), {}, 400, 0),
    ((1, 2, 4, 1, 1024, 1500), {}, 400, 0), ((1, 1, 4, 1, 1600, 2500), {}, 400, 64), ((16, 9, 8, 4, 150, 400), {}, 400, 0),
    ((32, 5, 16, 4, 111, 300), {}, 400, 0), ((32, 12, 8, 4, 40, 100), {}, 400, 16), ((32, 16, 8, 4, 40, 100), dict(launches=2), 400, 16),   # every spread of the slots
    ((1, 1, 7, 1, 200, 500), {}, 400, 0), ((1, 1, 12, 1, 200, 500), {}, 400, 0), ((1, 1, 16, 1, 200, 500), {}, 400, 16),       # heads of a group
    ((2, 3, 8, 2, 64, 300), dict(span_L=0), 400, 0), ((2, 3, 8, 2, 64, 300), dict(span_L=1), 100, 0),
    ((2, 3, 8, 2, 64, 300), dict(span_L=7), 100, 0), ((2, 3, 8, 2, 64, 300), dict(span_L=8, launches=2), 100, 0),
    ((2, 3, 8, 2, 64, 300), {}, 17, 0), ((2, 3, 8, 2, 300, 900), dict(rho=1.5), 20, 16),                                       # nearly all sponsored: vouchers decide
    ((8, 3, 8, 4, 900, 5000), dict(budget_decay=0.0), 17, 0), ((32, 3, 8, 8, 100, 3000), dict(budget_decay=0.5), 17, 0),       # and their tiles are overwritten meanwhile
    ((8, 5, 8, 4, 300, 2044), dict(budget_decay=0.5), 17, 64),
    ((2, 1, 8, 2, 8, 100), {}, 400, 0), ((2, 1, 8, 2, 40, 100), dict(n_sink=0, n_recent=0), 40, 0), ((2, 1, 8, 2, 1, 9), dict(n_sink=0, n_recent=1), 40, 0),
    ((3, 2, 8, 2, 64, 300), dict(gamma=2.0, budget_decay=1.25), 60, 0), ((3, 2, 8, 2, 64, 300), dict(last_query=1), 60, 0),
])
def test_one_launch_equals_two(shape, kw, vocabulary, page_size):
    layers, batch, hq, hkv, K, n = shape
    steps = 24
    kw = dict(kw)
    launches = kw.pop("launches", 1)
    prm = ta.Params(**{**dict(n_sink=4, n_recent=4), **kw})
    lens = [n] + [max(1, n // 3 - b) for b in range(batch - 1)]
    cap = n + 11                                                  # the first sequence reaches its capacity on the way
    args = (layers, batch, hq, hkv, K, n, cap, prm, page_size, vocabulary, lens, 3)
    (one, ids, tab_len), (two, _, _), (turns, _, _) = _state(*args), _state(*args), _state(*args)
    words, two.sync = turns.sync, None
    g = torch.Generator(device=DEV).manual_seed(5)
    for t in range(steps):
        tok = torch.randint(0, vocabulary, (batch,), generator=g, device=DEV, dtype=torch.int32)
        q, k, v = (torch.randn((layers, batch, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (hq, hkv, hkv))
        turns.sync = words if t % 3 else None
        one.sync[:, MARK] = -1 << 31
        got = []
        for st in (one, two, turns):
            evicted = torch.full((layers, batch, hkv), -7, dtype=torch.int32, device=DEV)
            ta.ta_decode_step(st, tok, q, k, v, ids, tab_len, prm, evicted=evicted)
            got.append(evicted)
        for st, e in ((one, got[0]), (turns, got[2])):
            assert torch.equal(e, got[1]), t
            for name in STATE:
                a, b = getattr(st, name), getattr(two, name)
                assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b), (t, name)
        assert one.sync[:, MARK].any().item() == (launches == 2)
        one.sync[:, MARK] = 0
        assert not one.sync.any() and not words.any()


@pytest.mark.parametrize("shape,kw,vocabulary,page_size", [
    ((2, 2, 8, 2, 255, 700), {}, 400, 0), ((2, 2, 8, 2, 256, 700), {}, 400, 16), ((1, 2, 4, 1, 511, 1500), {}, 400, 0), ((1, 1, 4, 1, 767, 1500), {}, 400, 0),
    ((1, 2, 4, 1, 1535, 2500), {}, 400, 64), ((1, 1, 4, 1, 2047, 2500), {}, 400, 0),                        # every spread of the slots, at its limit
    ((2, 3, 8, 2, 64, 300), dict(span_L=0), 400, 0), ((2, 3, 8, 2, 64, 300), dict(span_L=7), 100, 0), ((2, 3, 8, 2, 64, 300), dict(span_L=8, launches=2), 100, 0),
    ((2, 3, 8, 2, 64, 300), {}, 17, 0), ((2, 3, 8, 2, 300, 900), dict(rho=1.5), 20, 16), ((32, 3, 8, 8, 100, 3000), dict(budget_decay=0.0), 17, 0),  # vouchers decide
    ((2, 1, 8, 2, 1, 9), dict(n_sink=0, n_recent=1), 40, 0), ((40, 13, 8, 8, 8, 60), dict(beta=-1.0, launches=2), 40, 0),
])
def test_one_launch_equals_two_without_attention(shape, kw, vocabulary, page_size):
    test_one_launch_equals_two(shape, {**dict(alpha=0.0), **kw}, vocabulary, page_size)


def test_steps_of_two_states_overlap():
    """Two states on two streams, each with more workgroups of positions than an XCD can hold: nothing of one waits for the other, and
    both end as they do one after the other."""
    layers, batch, hq, hkv, K, n, cap, steps = 4, 32, 8, 2, 300, 700, 40000, 12
    prm = ta.Params()
    states = []
    for seed in (3, 4):
        lens = [n - 7 * b - seed for b in range(batch)]
        (st, ids, tab_len), (alone, _, _) = (_state(layers, batch, hq, hkv, K, n, cap, prm, 0, 400, lens, seed) for _ in range(2))
        alone.sync = None                                         # two launches
        states.append((st, alone))
    g = torch.Generator(device=DEV).manual_seed(6)
    inputs = [[(torch.randint(0, 400, (batch,), generator=g, device=DEV, dtype=torch.int32),
                *(torch.randn((layers, batch, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (hq, hkv, hkv)))
               for _ in states] for _ in range(steps)]
    for step in inputs:
        for (_, alone), x in zip(states, step):
            ta.ta_decode_step(alone, *x, ids, tab_len, prm)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in states]
    for step in inputs:
        for (st, _), x, stream in zip(states, step, streams):
            ta.ta_decode_step(st, *x, ids, tab_len, prm, stream=stream)
    torch.cuda.synchronize()
    for st, alone in states:
        for name in STATE:
            assert torch.equal(getattr(st, name), getattr(alone, name)), name
        assert not st.sync.any()


@pytest.mark.parametrize("n,K", [(n, 5) for n in (8, 505, 1018, 1023, 1024, 2041, 3066, 32760, 40900, 57335, 57336)] +
                         [(500, 6), (28663, 6), (28664, 6), (65528, 900), (114680, 900), (229367, 900), (229368, 900),
                          (57336, 7), (100000, 7), (229367, 7), (229368, 7), (40000, 8), (57335, 8), (57336, 8)])
def test_budgets_decay_once_in_every_tile(n, K):
    """Tiles of 512 to 4096 positions, lengths that end at and step over their edges, the longest rows of one launch and one position more."""
    prm = ta.Params(n_sink=0, n_recent=1, budget_decay=0.75)
    layers, B, waves, rounds = {5: (1, 3, 4, 1), 6: (171, 3, 2, 1), 7: (1, 4, 4, 4), 8: (129, 4, 2, 2), 900: (1, 3, 8, 2)}[K]
    lens = [n, max(1, n - 5), max(1, n // 2), max(1, n - 1000)][:B]
    st, ids, tab_len = _state(layers, B, 4, 1, K, n, n + 9, prm, 0, 40, lens, 7)
    g = torch.Generator(device=DEV).manual_seed(8)
    want = st.budget.clone()
    tiles = -(-(n + 9) // (256 * waves * rounds))                 # at most 56, else two launches
    for t in range(8):
        tok = torch.randint(0, 40, (B,), generator=g, device=DEV, dtype=torch.int32)
        st.sync[:, MARK] = -1 << 31 if tiles != 56 else 0
        ta.ta_decode_step(st, tok, *(torch.randn((layers, B, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (4, 1, 1)), ids, tab_len, prm)
        assert tiles == 56 or st.sync[:, MARK].any().item() == (tiles > 56)
        for b in range(B):
            want[b, lens[b] + t] = prm.sponsor_B if st.anchor[b, lens[b] + t] else 0.0
        want *= 0.75
    assert torch.equal(st.budget, want) and st.len.tolist() == [x + 8 for x in lens]


@pytest.mark.parametrize("layers,K,page_size", [(16, 279, 0), (16, 279, 16), (20, 220, 0), (20, 220, 16)])
def test_more_keys_than_the_cache_keeps(layers, K, page_size):
    """One launch and two over keys of more than 272 MB, which the last-level cache does not hold: each layer's units end as they do in a state of that
    layer alone, bit for bit."""
    batch, hq, hkv, n = 32, 16, 8, 400
    prm = ta.Params()
    lens = [n - 3 * b for b in range(batch)]
    big, ids, tab_len = _state(layers, batch, hq, hkv, K, n, n + 8, prm, page_size, 400, lens, 11)
    assert layers * batch * hkv * (K + 1) * 256 > 272 << 20
    of_layer = ("pos", "A", "Kc", "Vc")
    alone = {}
    for l in (0, 10, 11, layers - 1):                             # the first, those around the cache's size, the last
        pages = None
        if page_size:
            p = big.pages
            pages = ta.PagedKV(p.Kpool[l:l + 1].clone(), p.Vpool[l:l + 1].clone(), p.table, p.page_size, p.num_pages, p.strides, 1, batch, hkv, K + 1)
        alone[l] = ta.DecodeState(1, batch, hq, hkv, K, n + 8, DEV, pages=pages)
        for name in STATE:
            if not (page_size and name in ("Kc", "Vc")):
                getattr(alone[l], name).copy_(getattr(big, name)[l:l + 1] if name in of_layer else getattr(big, name))
    g = torch.Generator(device=DEV).manual_seed(12)
    for _ in range(3):
        tok = torch.randint(0, 400, (batch,), generator=g, device=DEV, dtype=torch.int32)
        q, k, v = (torch.randn((layers, batch, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (hq, hkv, hkv))
        ta.ta_decode_step(big, tok, q, k, v, ids, tab_len, prm)
        for l, st in alone.items():
            ta.ta_decode_step(st, tok, q[l:l + 1].contiguous(), k[l:l + 1].contiguous(), v[l:l + 1].contiguous(), ids, tab_len, prm)
    for l, st in alone.items():
        for name in of_layer:
            a, b = getattr(big, name)[l:l + 1], getattr(st, name)
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)) if a.dtype == torch.bfloat16 else torch.equal(a, b), (l, name)


def test_words_off_an_eight_byte_boundary():
    """Two of the words are one number of eight bytes: elsewhere the step is two launches and leaves them alone."""
    prm = ta.Params()
    (st, ids, tab_len), (two, _, _) = (_state(1, 2, 4, 1, 64, 200, 240, prm, 0, 100, [200, 150], 4) for _ in range(2))
    st.sync, two.sync = torch.zeros(2 * tb.TA_DECODE_SYNC_WORDS + 1, dtype=torch.int32, device=DEV)[1:], None
    g = torch.Generator(device=DEV).manual_seed(9)
    for _ in range(3):
        x = [torch.randint(0, 100, (2,), generator=g, device=DEV, dtype=torch.int32)]
        x += [torch.randn((1, 2, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (4, 1, 1)]
        for s in (st, two):
            ta.ta_decode_step(s, *x, ids, tab_len, prm)
    assert all(torch.equal(getattr(st, name), getattr(two, name)) for name in STATE) and not st.sync.any()


def test_copies_count_in_words_of_their_own():
    prm = ta.Params()
    st, ids, tab_len = _state(1, 1, 4, 1, 64, 200, 240, prm, 0, 100, [200], 4)
    g = torch.Generator(device=DEV).manual_seed(10)
    deep, shallow = copy.deepcopy(st), copy.copy(st)              # the shallow one goes on with the same tensors
    for other in (deep, shallow):
        assert other.sync.data_ptr() != st.sync.data_ptr() and not other.sync.any()
    for t in range(6):
        x = [torch.randint(0, 100, (1,), generator=g, device=DEV, dtype=torch.int32)]
        x += [torch.randn((1, 1, h, 128), generator=g, device=DEV).to(torch.bfloat16) for h in (4, 1, 1)]
        for s in (deep, (st, shallow)[t % 2]):
            s.sync[:, MARK] = -1 << 31
            ta.ta_decode_step(s, *x, ids, tab_len, prm)
            assert not s.sync.any()                               # one launch
        assert all(torch.equal(getattr(st, name), getattr(deep, name)) for name in STATE)

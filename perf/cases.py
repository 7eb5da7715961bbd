"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values; "kind" says which of the public paths it takes:

  evict     one eviction pass over a whole cache through a plan (anchor match, window scores,
            protected top-K, gather), over one stacked tensor ("dense"), a page pool ("paged"), one
            tensor per layer ("layers"), or with the prefill's log-sum-exps given ("lse");
            alpha = 0 is the attention-free policy
  generate  a prompt's retained rows are handed to the generation state, then `steps` tokens are
            generated, each with an eviction step of its own
  learned   learned anchor detection on the prompt's hidden states, vouchers, one selection per
            sequence, gather
  embed     anchors by similarity: once over the embedding table, then by token ID for a batch of
            prompts, and their vouchers

Sizes are those of the configurations in paper_2604_11288_amd/workloads.py, some with fewer sequences
so that several sets of inputs fit the card, and odd lengths as the tests have them.
"""
import math

import torch

import paper_2604_11288_amd as ta
from paper_2604_11288_amd import workloads as wl

ROW = 256                        # bytes of a key or value row (d = 128, bf16)
MAX_SCORED = 256 << 25           # layers * sequences * KV heads * positions * query rows per key of the largest case (17 GB of keys and values)
MAX_STEPPED = 16 * 32 * 64 * 8 * 257   # slots visited by the largest generation: steps * layers * sequences * KV heads * slots


def _evict(name, **kw):
    case = dict(name=name, kind="evict", form="dense", layers=32, batch=1, n=4096, min_len=0, hq=32, hkv=8, window=32,
                n_recent=4, K=1024, alpha=1.0, pool_k=1, k_protected=-1, table=16, planted=8, page_size=0, heads_first=False)
    case.update(kw)
    return case


def _generate(name, **kw):
    case = dict(name=name, kind="generate", layers=32, batch=1, n=4096, min_len=0, hq=32, hkv=8, K=1024, alpha=1.0, steps=32,
                table=16, planted=8, page_size=0)
    case.update(kw)
    return case


def _learned(name, **kw):
    case = dict(name=name, kind="learned", layers=32, batch=1, n=4096, hkv=8, K=256, d_model=4096, hidden=128)
    case.update(kw)
    return case


def _embed(name, **kw):
    case = dict(name=name, kind="embed", vocabulary=128256, d_model=4096, concepts=16, batch=16, n=4096)
    case.update(kw)
    return case


def listed():
    return [
        # one layer of one 4K prompt at the smallest budget (c1): what an engine calls layer by layer
        _evict("single_layer_4k", layers=1, K=16, planted=4),
        # one 4K prompt through a whole model at its largest budget (c2)
        _evict("full_model_4k"),
        # two prompts of odd, unequal lengths in a serving engine's page pool, small budget
        _evict("paged_ragged_3k", form="paged", batch=2, n=3001, min_len=1500, K=64, page_size=64),
        # one 16K prompt whose prefill attention kernel has left its log-sum-exps: keys are read once
        _evict("prefill_lse_16k", form="lse", n=16384, K=512),
        # max-pooled scores (the SnapKV setting) on a past_key_values list of per-layer tensors, wide query groups
        _evict("pooled_layers_8k", form="layers", layers=24, n=8192, hq=64, n_recent=32, pool_k=7),
        # the attention-free policy on long prompts (c3, four of its sixteen sequences)
        _evict("attention_free_32k", batch=4, n=32768, n_recent=64, K=512, alpha=0.0, window=0, table=64, planted=32),
        # one long document (c4, one of its four sequences)
        _evict("long_context_128k", n=131072, window=64, n_recent=128, table=64, planted=128),
        # a batch of agents' prompts of unequal lengths (c5, eight of its sixty-four sequences)
        _evict("agentic_ragged_16k", batch=8, n=16384, min_len=2048, K=256),
        # generation after c2: one user waits for every token
        _generate("generate_one_sequence"),
        # generation after c5: all sixty-four agents at once, short prompts
        _generate("generate_agentic_batch", batch=64, n=2048, min_len=1024, K=256, steps=16),
        # TA-LearnRank on one 4K prompt: detector, vouchers, selection, gather
        _learned("learned_detector_4k"),
        # anchors by embedding similarity for a 128K vocabulary, then flags and vouchers of sixteen prompts
        _embed("embedding_128k_vocabulary"),
    ]


def _log_int(rng, lo, hi):
    """A whole number between lo and hi, uniform over its logarithm."""
    return int(round(lo * math.exp(rng.uniform(0.0, math.log(max(hi, lo) / lo)))))


def draw(rng):
    """One more case of the same ranges: kinds in about the proportion of the list above, sizes over their logarithm."""
    kind = rng.choices(("evict", "generate", "learned", "embed"), (8, 2, 1, 1))[0]
    if kind == "evict":
        form = rng.choice(("dense", "dense", "dense", "dense", "lse", "paged", "layers"))
        alpha = 0.0 if form in ("dense", "paged") and rng.random() < 0.2 else 1.0
        layers = rng.choice((8, 16, 24)) if form == "layers" else rng.choice((1, 8, 32, 32))
        hq, hkv = rng.choice(((32, 8), (32, 8), (64, 8), (8, 2)))
        window = rng.choice((16, 32, 32, 64)) if alpha else 0
        per_key = max(hq // hkv * window, 256)             # rows scored per key, as the largest listed case counts them
        n = min(_log_int(rng, 700, 131072), MAX_SCORED // (layers * hkv * per_key))
        batch = min(_log_int(rng, 1, 16), MAX_SCORED // (layers * hkv * n * per_key))
        K = _log_int(rng, 16, min(1024, n // 2))
        ragged = batch > 1 and rng.random() < 0.6
        case = _evict("", form=form, layers=layers, batch=batch, n=n, min_len=n // rng.choice((2, 4, 8)) if ragged else 0,
                      hq=hq, hkv=hkv, window=window, n_recent=min(rng.choice((4, 4, 32, 64)), K // 2), K=K, alpha=alpha,
                      pool_k=rng.choice((3, 5, 7, 9)) if alpha and rng.random() < 0.15 else 1,
                      k_protected=K // 4 if rng.random() < 0.1 else -1, table=rng.choice((16, 64)),
                      planted=rng.choice((4, 8, 32)), page_size=rng.choice((64, 128)) if form == "paged" else 0,
                      heads_first=form == "paged" and rng.random() < 0.5)
    elif kind == "generate":
        K = _log_int(rng, 64, 1500)
        batch = max(1, min(_log_int(rng, 1, 64), 64 * 257 // (K + 1)))
        n = _log_int(rng, K + 8, 8 * K)
        hq, hkv = rng.choice(((32, 8), (32, 8), (64, 8), (8, 2)))
        layers, steps = rng.choice((8, 32, 32)), rng.choice((8, 16, 32))
        while steps * layers * batch * hkv * (K + 1) > MAX_STEPPED:
            steps //= 2
        case = _generate("", layers=layers, batch=batch, n=n, min_len=max(16, n // 2) if batch > 1 else 0,
                         hq=hq, hkv=hkv, K=K, alpha=0.0 if rng.random() < 0.15 else 1.0, steps=steps,
                         page_size=rng.choice((0, 0, 16, 64)))
    elif kind == "learned":
        n = _log_int(rng, 512, 65536)
        batch = min(_log_int(rng, 1, 8), 131072 // n)
        case = _learned("", layers=rng.choice((1, 8, 32)), batch=batch, n=n, K=_log_int(rng, 32, min(1024, n // 2)),
                        d_model=rng.choice((1024, 2048, 4096)), hidden=rng.choice((32, 64, 128, 256)))
    else:
        case = _embed("", vocabulary=_log_int(rng, 8000, 160000), d_model=rng.choice((1024, 2048, 4096)),
                      concepts=_log_int(rng, 4, 200), batch=_log_int(rng, 1, 16), n=_log_int(rng, 500, 32768))
    del case["name"]
    return case


# ---- inputs ---------------------------------------------------------------------------------------

def _workload(case, seed):
    get = case.get
    return wl.Workload("case", layers=get("layers", 1), batch=case["batch"], n=case["n"], hq=get("hq", get("hkv", 1)), hkv=get("hkv", 1),
                       window=get("window", 0), n_recent=get("n_recent", 4), table_entries=get("table", 16), gram_min=1,
                       gram_max=3 if get("table", 16) <= 16 else 4, planted=get("planted", 8), alpha=get("alpha", 1.0),
                       seed=wl.BASE_SEED + seed, ragged=(case["min_len"], case["n"]) if get("min_len", 0) else None)


def _normal(shape, seed, dev):
    out = torch.empty(shape, dtype=torch.bfloat16, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    flat = out.view(-1)
    for part in flat.split(1 << 27):
        part.copy_(torch.randn(part.numel(), generator=g, device=dev))
    return out


def _log_sum_exps(Q, K, lens, window):
    """What a prefill attention kernel leaves behind: log-sum-exp of the window rows' scaled, causal logits."""
    L, B, hq, W, d = Q.shape
    hkv, n = K.shape[2], K.shape[3]
    out = torch.empty((L, B, hq, W), dtype=torch.float32, device=Q.device)
    last = torch.arange(W, device=Q.device).repeat(hq // hkv)          # row of the group -> window row
    for b in range(B):
        m = lens[b]
        hidden = torch.arange(m, device=Q.device)[None, :] > (m - window + last)[:, None]
        for l in range(L):
            for g in range(hkv):
                q = Q[l, b, g * (hq // hkv):(g + 1) * (hq // hkv)].reshape(-1, d).float()
                s = (q @ K[l, b, g, :m].float().T) * d ** -0.5
                out[l, b, g * (hq // hkv):(g + 1) * (hq // hkv)] = s.masked_fill_(hidden, -math.inf).logsumexp(1).view(-1, W)
    return out


def _bits(t):
    """Rows are moved, not computed: they are compared as the bit patterns they are."""
    return t.view(torch.int16)


def _prepare_evict(case, seed, dev):
    w = _workload(case, seed)
    td = wl.make_tokens(w)
    tok = torch.from_numpy(td.tok).to(dev)
    lens = td.seq_len.tolist()
    seq_len = torch.from_numpy(td.seq_len).to(dev) if w.ragged else None
    prm = ta.Params(n_sink=w.n_sink, n_recent=w.n_recent, alpha=w.alpha, pool_k=case["pool_k"], k_protected=case["k_protected"])
    shape = (w.layers, w.batch, w.hkv, w.n, w.d)
    Q = _normal((w.layers, w.batch, w.hq, w.window, w.d), w.seed * 3, dev) if w.window else None
    form = case["form"]
    args = (tok, td.tab_ids, td.tab_len)
    if form == "paged":
        ps = case["page_size"]
        slots = (w.n + ps - 1) // ps
        pages = w.batch * slots + 3
        table = torch.randperm(pages, generator=torch.Generator().manual_seed(w.seed))[: w.batch * slots]
        table = table.to(torch.int32).view(w.batch, slots).to(dev)
        first = case["heads_first"]
        pool = (w.layers, pages, w.hkv, ps, w.d) if first else (w.layers, pages, ps, w.hkv, w.d)
        Kp, Vp = _normal(pool, w.seed * 3 + 1, dev), _normal(pool, w.seed * 3 + 2, dev)
        st = Kp.stride()
        paged = ta.PagedKV(Kp, Vp, table, ps, pages, (st[0], st[1], st[3], st[2]) if first else st[:4], w.layers, w.batch, w.hkv, w.n)
        plan = ta.EvictPlan(*args, Q, None, None, case["K"], prm, seq_len=seq_len, paged=paged)
    else:
        K, V = _normal(shape, w.seed * 3 + 1, dev), _normal(shape, w.seed * 3 + 2, dev)
        if form == "layers":
            plan = ta.LayerEvictPlan(*args, [x for x in Q], [x for x in K], [x for x in V], case["K"], prm, seq_len=seq_len)
        else:
            lse = _log_sum_exps(Q, K, lens, w.window) if form == "lse" else None
            plan = ta.EvictPlan(*args, Q, K, V, case["K"], prm, seq_len=seq_len, lse=lse)
    out = dict(anchor=plan.anchor, spons=plan.spons, vouch=plan.vouch, A=plan.A, idx=plan.idx, cnt=plan.cnt)
    if form == "layers":
        out.update(Kout=[_bits(t) for t in plan.Kout], Vout=[_bits(t) for t in plan.Vout])
    else:
        out.update(Kout=_bits(plan.Kout), Vout=_bits(plan.Vout))
    return dict(kind="evict", plan=plan, out=out)


def _prepare_generate(case, seed, dev):
    """The outputs of a prompt's eviction pass (scores spread as attention is: a few positions hold most of it),
    the state, and the rows that the model will produce for the next tokens."""
    w = _workload(case, seed)
    K, steps = case["K"], case["steps"]
    td = wl.make_tokens(w)
    tok = torch.from_numpy(td.tok).to(dev)
    seq_len = torch.from_numpy(td.seq_len).to(dev)
    prm = ta.Params(n_sink=w.n_sink, n_recent=w.n_recent, alpha=w.alpha)
    anchor, spons, vouch = ta.ta_match_anchors(tok, td.tab_ids, td.tab_len, prm, seq_len=seq_len)
    g = torch.Generator(device=dev)
    g.manual_seed(w.seed)
    A = torch.randn((w.layers, w.batch, w.hkv, w.n), generator=g, device=dev).exp_().mul_(128.0 / w.n)
    idx, cnt = ta.ta_select(A, anchor, spons, vouch, K, prm, w.layers, w.hkv, seq_len=seq_len)
    rows = (w.layers, w.batch, w.hkv, K, w.d)
    pages = None
    if case["page_size"]:
        Kp, Vp, table, num_pages, strides = wl.make_slot_pool(w.layers, w.batch, w.hkv, w.d, K + 1, case["page_size"], dev, seed=w.seed)
        pages = ta.PagedKV(Kp, Vp, torch.from_numpy(table).to(dev), case["page_size"], num_pages, strides, w.layers, w.batch, w.hkv, K + 1)
    state = ta.DecodeState(w.layers, w.batch, w.hq, w.hkv, K, w.n + steps, dev, pages=pages)
    new_tok = torch.from_numpy(wl.make_decode_stream(w, td, steps)).to(dev)
    new = [wl.make_decode_qkv(w, t, dev) for t in range(steps)]
    evicted = torch.full((steps, w.layers, w.batch, w.hkv), -2, dtype=torch.int32, device=dev)
    out = dict(tok=state.tok, len=state.len, anchor=state.anchor, budget=state.budget, pos=state.pos, A=state.A,
               K=_bits(state.Kc), V=_bits(state.Vc), evicted=evicted)
    return dict(kind="generate", state=state, prm=prm, tok=tok, seq_len=seq_len, anchor=anchor, A=A if w.alpha else None, idx=idx, cnt=cnt,
                Kout=_normal(rows, w.seed * 3 + 1, dev), Vout=_normal(rows, w.seed * 3 + 2, dev), tab_ids=td.tab_ids, tab_len=td.tab_len,
                steps=[(new_tok[t], new[t][0] if w.alpha else None, new[t][1], new[t][2], evicted[t]) for t in range(steps)], out=out)


def _prepare_learned(case, seed, dev):
    w = _workload(case, seed)
    B, n, K = w.batch, w.n, case["K"]
    h, W1, W2 = wl.make_detector_inputs(B, n, case["d_model"], case["hidden"], seed=w.seed, p_anchor=0.01, device=dev)
    Kin, Vin = _normal((w.layers, B, w.hkv, n, w.d), w.seed * 3 + 1, dev), _normal((w.layers, B, w.hkv, n, w.d), w.seed * 3 + 2, dev)
    f32, u8, i32 = (dict(dtype=t, device=dev) for t in (torch.float32, torch.uint8, torch.int32))
    found = [torch.empty((B, n), **f32), torch.empty((B, n), **u8), torch.empty((B, n), **f32)]
    vouched = [torch.empty((B, n), **u8), torch.empty((B, n), **f32)]
    chosen = [torch.zeros((1, B, 1, K), **i32), torch.zeros((1, B, 1), **i32)]
    rows = [torch.zeros((w.layers, B, w.hkv, K, w.d), dtype=torch.bfloat16, device=dev) for _ in range(2)]
    out = dict(found=found, vouched=vouched, chosen=chosen, rows=[_bits(t) for t in rows])
    return dict(kind="learned", h=h, W1=W1, W2=W2, Kin=Kin, Vin=Vin, K=K, prm=ta.Params(alpha=0.0), found=found, vouched=vouched,
                chosen=chosen, rows=rows, out=out)


def _prepare_embed(case, seed, dev):
    V, B, n = case["vocabulary"], case["batch"], case["n"]
    x, C = wl.make_embedding_inputs(V, case["d_model"], case["concepts"], seed=wl.BASE_SEED + seed, p_near=0.02, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(wl.BASE_SEED + seed)
    tok = torch.randint(0, V, (B, n), generator=g, device=dev, dtype=torch.int32)
    f32, u8 = (dict(dtype=t, device=dev) for t in (torch.float32, torch.uint8))
    out = dict(table=[torch.empty((1, V), **f32), torch.empty((1, V), **u8)], anchor=torch.empty((B, n), **u8),
               vouched=[torch.empty((B, n), **u8), torch.empty((B, n), **f32)])
    return dict(kind="embed", x=x.unsqueeze(0), C=C, tok=tok, prm=ta.Params(), out=out)


def prepare(case, seed):
    make = dict(evict=_prepare_evict, generate=_prepare_generate, learned=_prepare_learned, embed=_prepare_embed)
    return make[case["kind"]](case, seed, torch.device("cuda"))


# ---- one pass ----------------------------------------------------------------------------------------

def run(state):
    s = state
    if s["kind"] == "evict":
        s["plan"].run()
    elif s["kind"] == "generate":
        ta.ta_decode_init(s["state"], s["tok"], s["anchor"], s["idx"], s["cnt"], s["Kout"], s["Vout"], s["prm"],
                          seq_len=s["seq_len"], A=s["A"])
        for tok, q, k, v, evicted in s["steps"]:
            ta.ta_decode_step(s["state"], tok, q, k, v, s["tab_ids"], s["tab_len"], s["prm"], evicted=evicted)
    elif s["kind"] == "learned":
        conf, anchor, budget = ta.ta_detect_anchors(s["h"], s["W1"], s["W2"], s["prm"], 0.3, True, scale=15.0, out=s["found"])
        spons, vouch = ta.ta_expand_vouchers(anchor, s["prm"], anchor_B=budget, out=s["vouched"])
        idx, cnt = ta.ta_select(None, anchor, spons, vouch, s["K"], s["prm"], 1, 1, out=s["chosen"])
        ta.ta_compact(s["Kin"], s["Vin"], idx, cnt, s["K"], idx_shared=True, out=s["rows"])
    else:
        sim, flags = ta.ta_embed_anchors(s["x"], s["C"], 0.5, out=s["out"]["table"])
        anchor = ta.ta_lookup_anchors(s["tok"], flags[0], out=s["out"]["anchor"])
        ta.ta_expand_vouchers(anchor, s["prm"], out=s["out"]["vouched"])
    return s["out"]


# ---- what a pass cannot do without, and how exact it is -----------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "embed":
        V, dm, E, at = case["vocabulary"], case["d_model"], case["concepts"], case["batch"] * case["n"]
        return dict(bytes=(V + E) * dm * 2 + V * 5 + at * (4 + 1 + 5), flops=2.0 * V * E * dm)
    B, n, units = case["batch"], case["n"], case["layers"] * case["batch"] * case["hkv"]
    m = (case["min_len"] + n) / 2 if case.get("min_len") else n          # mean length
    kept = min(case["K"], m)
    if kind == "learned":
        dm, hid = case["d_model"], case["hidden"]
        return dict(bytes=B * n * (2 * dm + 14) + hid * dm * 2 + B * kept * 4 + units * kept * 4 * ROW, flops=2.0 * B * n * hid * dm)
    G = case["hq"] // case["hkv"]
    scored = case["alpha"] != 0.0
    if kind == "generate":
        slots = case["K"] + 1
        hand_over = units * (kept * (2 * ROW + 8) + slots * (2 * ROW + 8)) + B * m * 16
        step = units * (slots * (4 + (ROW + 8 if scored else 0)) + 4 * ROW + (G * ROW if scored else 0)) + B * m * 14
        return dict(bytes=hand_over + case["steps"] * step, flops=case["steps"] * 2.0 * 128 * G * slots * units if scored else 0.0)
    sequences = B * m * (4 + 6)
    gathered = units * kept * 4 * ROW
    if not scored:
        return dict(bytes=sequences + gathered + B * kept * 4, flops=0.0)
    rows = G * case["window"]
    gathered -= units * kept * ROW                                       # the keys have been read for the scores
    return dict(bytes=sequences + gathered + units * (m * (ROW + 4) + rows * ROW + kept * 4), flops=2.0 * 128 * rows * m * units)


def tolerance(case):
    if case["kind"] == "evict" and case["alpha"] == 0.0:
        return "exact"                                                   # vouchers and utilities are specified operation by operation
    if case["kind"] == "learned":
        return dict(rel=1e-4, max=1e-3, differ=1e-3)                     # a logit is a sum of `hidden` sums of d_model bf16 products
    if case["kind"] == "embed":
        return dict(rel=2e-5, max=5e-4, differ=1e-4)
    # scores are fp32 sums; another order of summation may turn over a near-tie of the selection, which moves the
    # rows behind it in its unit
    return dict(rel=1e-5, max=2e-4, differ=0.01 if case["kind"] == "evict" else 1e-3)

"""The binding hands the library the tensors' present addresses.

The calls are recorded in the library's place, so these run without a GPU: what is checked is which addresses reach the C ABI."""
import copy
import ctypes
import pickle
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2604_11288_amd import binding as tb

STREAM = SimpleNamespace(cuda_stream=0)
LAYERS, B, HQ, HKV, N, W, K, D = 2, 2, 4, 2, 96, 4, 16, tb.TA_HEAD_DIM
TABLE = (np.array([[5, 6, -1, -1], [7, -1, -1, -1]], np.int32), np.array([2, 1], np.int32))


class Recorder:
    """libta.so with the calls that would launch kernels replaced by one that keeps what they were given: the addresses among
    the arguments, those in the structs, those in the per-layer tables, and the host tables' words."""

    def __init__(self):
        self.real = tb.lib()

    def __getattr__(self, name):
        return self.record if name.startswith(("ta_evict", "ta_decode")) else getattr(self.real, name)

    def record(self, *args):
        self.addresses, self.words = set(), []
        for a in args:
            if isinstance(a, int):
                self.addresses.add(a)
            elif isinstance(a, bytes):
                self.words.append(np.frombuffer(a, np.int32).copy())
            elif a is not None:
                self.struct(a._obj)
        return tb.TA_OK

    def struct(self, s):
        named = [getattr(s, f) for f, t in s._fields_ if t is ctypes.c_void_p and getattr(s, f)]
        self.addresses.update(named)
        if isinstance(s, tb.CLayerPtrs):
            for address in named:
                self.addresses.update((ctypes.c_uint64 * LAYERS).from_address(address))
        if isinstance(s, tb.CDecodeState) and s.pages:
            self.struct(tb.CPaged.from_address(s.pages))


@pytest.fixture
def recorder(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(tb, "lib", lambda: r)
    return r


def _bf16(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


def _paged():
    pool = lambda: _bf16(LAYERS, 16, 16, HKV, D)
    Kp, Vp = pool(), pool()
    return tb.PagedKV(Kp, Vp, torch.arange(12, dtype=torch.int32).view(B, 6), 16, 16, Kp.stride()[:4], LAYERS, B, HKV, N)


def _plan(form, table=TABLE):
    """A plan and the tensors whose addresses it passes."""
    tok, seq_len = torch.zeros((B, N), dtype=torch.int32), torch.full((B,), N, dtype=torch.int32)
    anchor_B = torch.zeros((B, N))
    lse = torch.zeros((LAYERS, B, HQ, W))
    prm = tb.Params(layer_K=torch.full((LAYERS,), K, dtype=torch.int32), allow=torch.ones((B, N), dtype=torch.uint8),
                    margin=torch.zeros((LAYERS * B * HKV, 2)))
    Q, Kin, Vin = _bf16(LAYERS, B, HQ, W, D), _bf16(LAYERS, B, HKV, N, D), _bf16(LAYERS, B, HKV, N, D)
    args, kw = (tok, *table), dict(seq_len=seq_len, anchor_B=anchor_B)
    tensors = [tok, seq_len, anchor_B, prm.layer_K, prm.allow, prm.margin]
    if form in ("dense", "lse", "static"):
        plan = tb.EvictPlan(*args, Q, Kin, Vin, K, prm, lse=lse if form == "lse" else None, static_scratch=form == "static", **kw)
        tensors += [Q, Kin, Vin, plan.Kout, plan.Vout]
    elif form == "paged":
        paged = _paged()
        plan = tb.EvictPlan(*args, Q, None, None, K, prm, lse=lse, paged=paged, **kw)
        tensors += [Q, paged.Kpool, paged.Vpool, paged.table, plan.Kout, plan.Vout]
    else:
        paged = _paged() if form == "layers_paged" else None
        keys = [_bf16(*(paged.Kpool if paged else Kin).shape[1:]) for _ in range(2 * LAYERS)]
        Ql = [_bf16(B, HQ, W, D) for _ in range(LAYERS)]
        plan = tb.LayerEvictPlan(*args, Ql, keys[:LAYERS], keys[LAYERS:], K, prm, paged=paged, lse=lse if paged else None, **kw)
        tensors += Ql + keys + plan.Kout + plan.Vout + ([paged.table] if paged else [])
    tensors += [plan.anchor, plan.spons, plan.vouch, plan.A, plan.idx, plan.cnt]
    if plan.ws is not None and form != "lse":                    # one sweep needs no workspace
        tensors.append(plan.ws)
    if form in ("lse", "paged", "layers_paged"):
        tensors.append(lse)
    return plan, tensors


def _move(tensors):
    """Every tensor gets another storage in place; the old ones are returned, so that no address is used twice."""
    old = []
    for t in tensors:
        old.append(t.detach())
        t.data = t.clone()
    return old


FORMS = ("dense", "static", "lse", "paged", "layers", "layers_paged")


@pytest.mark.parametrize("form", FORMS)
def test_plan_passes_present_addresses(recorder, form):
    plan, tensors = _plan(form)
    plan.run(STREAM)
    assert {t.data_ptr() for t in tensors} <= recorder.addresses
    old = _move(tensors)
    plan.run(STREAM)
    assert {t.data_ptr() for t in tensors} <= recorder.addresses
    assert not recorder.addresses & {t.data_ptr() for t in old}


@pytest.mark.parametrize("paged", (False, True))
def test_decode_state_passes_present_addresses(recorder, paged):
    pages = _paged() if paged else None
    state = tb.DecodeState(LAYERS, B, HQ, HKV, K, N, "cpu", pages=pages)
    tensors = [t for t in vars(state).values() if isinstance(t, torch.Tensor)] + ([pages.table] if paged else [])
    new = [torch.zeros(8) for _ in range(4)]

    def step():
        tb.ta_decode_step(state, *new, *TABLE, tb.Params(), stream=STREAM)
        assert {t.data_ptr() for t in tensors} <= recorder.addresses

    step()
    old = _move(tensors)
    step()
    assert not recorder.addresses & {t.data_ptr() for t in old}


@pytest.mark.parametrize("form", ("dense", "layers"))
@pytest.mark.parametrize("as_list", (False, True))
def test_plan_keeps_its_own_anchor_table(recorder, form, as_list):
    """The caller's arrays are filled again for the next request: the plan built from them runs on with what it was given."""
    ids, lens = TABLE[0].copy(), TABLE[1].copy()
    plan, _ = _plan(form, table=(ids.tolist() if as_list else ids, lens))
    ids[:], lens[:] = 9, 1
    plan.run(STREAM)
    assert [w.tolist() for w in recorder.words] == [TABLE[0].ravel().tolist(), TABLE[1].tolist()]


@pytest.mark.parametrize("fork", (copy.deepcopy, lambda x: pickle.loads(pickle.dumps(x))))
def test_params_and_state_can_be_copied_after_use(recorder, fork):
    """A generation is forked by copying its state: the copy has tensors of its own and the same values."""
    prm, state = tb.Params(alpha=0.25), tb.DecodeState(LAYERS, B, HQ, HKV, K, N, "cpu")
    tb.ta_decode_step(state, *[torch.zeros(8) for _ in range(4)], *TABLE, prm, stream=STREAM)
    state.budget.fill_(3.0)
    prm2, state2 = fork(prm), fork(state)
    assert prm2 == prm and bytes(prm2.c()) == bytes(prm.c())
    for name, t in vars(state).items():
        if isinstance(t, torch.Tensor):
            other = getattr(state2, name)
            assert torch.equal(other, t) and other.data_ptr() != t.data_ptr()


def test_params_struct_is_the_callers_own():
    """What a caller changes in a returned struct stays in that struct."""
    prm = tb.Params()
    prm.c().alpha = 0.0
    assert prm.c().alpha == prm.alpha == 1.0

"""The binding's short argument tests accept exactly what its full checks accept
(CPU tensors: nothing is launched)."""

import itertools
import types

import numpy as np
import pytest
import torch

from paper_2606_02544_amd import binding


def attention_args(page=0):
    b, B, L, hq, hkv, d = 2, 4, 3, 4, 2, 64
    bf = torch.bfloat16
    cache = (5, 16, hkv, d) if page else (b, 24, hkv, d)
    a = {"q": torch.zeros(b, B + L, hq, d, dtype=bf), "k_new": torch.zeros(b, B + L, hkv, d, dtype=bf),
         "v_new": torch.zeros(b, B + L, hkv, d, dtype=bf), "k_cache": torch.zeros(cache, dtype=bf),
         "v_cache": torch.zeros(cache, dtype=bf),
         "block_table": torch.zeros(b, 2, dtype=torch.int32) if page else None,
         "prefix_lens": torch.zeros(b, dtype=torch.int32), "step_map": torch.zeros(b, B, dtype=torch.int32),
         "num_ref": torch.zeros(b, dtype=torch.int32), "out": None, "lse": None}
    return a, dict(block_size=B, max_ref=L, max_prefix_len=20, page_size=page)


def spoiled(t):
    """Tensors that differ from t in one respect each (and None, and no tensor)."""
    yield t
    yield None
    yield t.tolist()
    yield t.numpy() if t.dtype != torch.bfloat16 else t.float().numpy()
    yield t.to(torch.float32 if t.dtype == torch.bfloat16 else torch.int64)
    yield t.to("meta")
    yield t[..., :-1]
    yield t[..., :-1].contiguous()
    yield t[:-1]
    yield t.unsqueeze(0)
    yield t.reshape(-1)
    if t.dim() > 1:
        yield t.transpose(0, 1)
        yield t.transpose(-1, -2).contiguous().transpose(-1, -2)
    if t.dim() == 4:
        yield torch.zeros(t.shape[:3] + (2 * t.shape[3],), dtype=t.dtype)[..., : t.shape[3]]
        yield torch.zeros((t.shape[0], t.shape[1] + 3) + tuple(t.shape[2:]), dtype=t.dtype)[:, : t.shape[1]]
        yield t[:, :, :1]


def full_attention(a, kw):
    try:
        return binding.check_attention_tensors(*a.values(), **kw)
    except (ValueError, AttributeError, TypeError):
        return None


@pytest.mark.parametrize("page", [0, 16])
def test_attention(page):
    a, kw = attention_args(page)
    a["out"], a["lse"] = torch.empty_like(a["q"]), torch.empty(2, 4, 7)
    seen = set()
    for name in a:
        if a[name] is None:
            continue
        for t in spoiled(a[name]):
            c = dict(a, **{name: t})
            got = binding._attention_hkv(*c.values(), *kw.values())
            assert got == full_attention(c, kw), (name, t)
            seen.add(got)
    assert seen == {2, None}
    for change in ({"block_size": 5}, {"max_prefix_len": 0}, {"max_prefix_len": 33}, {"page_size": 8},
                   {"max_prefix_len": 25}):
        k = dict(kw, **change)
        assert binding._attention_hkv(*a.values(), *k.values()) == full_attention(a, k), change
    both = dict(a, k_cache=a["k_cache"][:, ::2], v_cache=a["v_cache"][:, ::2])   # strided, alike
    k = dict(kw, max_prefix_len=8, page_size=8 if page else 0)
    assert binding._attention_hkv(*both.values(), *k.values()) == full_attention(both, k) == 2


@pytest.mark.parametrize("kind", ["accept", "lmhead"])
def test_accept_and_lmhead(kind):
    b, B, L, V, H = 2, 4, 3, 10, 64
    ints = {"draft_ids": torch.zeros(b, L, dtype=torch.int32), "step_map": torch.zeros(b, B, dtype=torch.int32),
            "num_ref": torch.zeros(b, dtype=torch.int32)}
    if kind == "accept":
        a = {"logits": torch.zeros(b, B, V, dtype=torch.bfloat16), **ints}
        short, full = binding._accept_inputs, binding._check_accept_inputs
    else:
        a = {"hidden": torch.zeros(b, B, H, dtype=torch.bfloat16),
             "weight": torch.zeros(V, H, dtype=torch.bfloat16), **ints}
        short, full = binding._lmhead_inputs, binding._check_lmhead_inputs

    def outcome(fn, args):
        try:
            return fn(*args.values())
        except Exception as e:
            return type(e), str(e)

    for name, t in itertools.chain.from_iterable(((n, t) for t in spoiled(x)) for n, x in a.items()):
        c = dict(a, **{name: t})
        assert outcome(short, c) == outcome(full, c), name


@pytest.fixture
def calls(monkeypatch):
    """The descriptors that calls hand to the library, as (field, value) dicts."""
    seen = []

    def record(desc, *_):
        seen.append({n: getattr(desc._obj, n) for n, _ in desc._obj._fields_})
        return 0

    monkeypatch.setattr(binding, "lib", lambda: types.SimpleNamespace(
        simsd_verify_attention=record, simsd_verify_accept=record, simsd_verify_accept_sampled=record,
        simsd_verify_attention_workspace_size=lambda desc: 0))
    return seen


STREAM = types.SimpleNamespace(cuda_stream=0)


@pytest.mark.parametrize("name", ["scale", "rope_theta"])
def test_float_arguments_are_read_on_every_call(calls, name):
    a, kw = attention_args()
    del a["out"], a["lse"]
    for box in (torch.tensor(0.5), np.array(0.5)):
        for value in (0.5, 0.25, 2.0):
            box[...] = value
            binding.verify_attention(*a.values(), **kw, **{name: box}, stream=STREAM)
            assert calls[-1][name] == value
    for other in (1, np.float32(0.75), 0.3):
        binding.verify_attention(*a.values(), **kw, **{name: other}, stream=STREAM)
        assert calls[-1][name] == np.float32(other)
    for bad in ("0.5", None):
        with pytest.raises(TypeError):
            binding.verify_attention(*a.values(), **kw, **{name: bad}, stream=STREAM)


def test_integer_arguments_are_read_on_every_call(calls):
    a, kw = attention_args()
    del a["out"], a["lse"]
    for box in (torch.tensor(64), np.array(64)):
        for value in (64, 128, 0):
            box[...] = value
            binding.verify_attention(*a.values(), **kw, kv_chunk=box, stream=STREAM)
            assert calls[-1]["kv_chunk"] == value
    for name, value in dict(kw, kv_chunk=64).items():          # a float is refused, also once seen as an int
        with pytest.raises(TypeError):
            binding.verify_attention(*a.values(), **dict(kw, kv_chunk=64, **{name: float(value)}), stream=STREAM)


def test_chunks_per_row_is_read_on_every_call(calls):
    b, B, L, V = 2, 4, 3, 10
    logits, side = torch.zeros(b, B, V), torch.zeros(b, L, V)
    ints = (torch.zeros(b, L, dtype=torch.int32), torch.zeros(b, B, dtype=torch.int32),
            torch.zeros(b, dtype=torch.int32))

    def greedy(n):
        binding.verify_accept(logits, *ints, chunks_per_row=n, stream=STREAM)

    def sampled(n):
        binding.verify_accept_sampled(logits, side, *ints, torch.zeros(b, L + 1), chunks_per_row=n, stream=STREAM)

    for call in (greedy, sampled):
        box = torch.tensor(2)
        for value in (2, 5, 0):
            box.fill_(value)
            call(box)
            assert calls[-1]["chunks_per_row"] == value
        with pytest.raises(TypeError):
            call(2.0)

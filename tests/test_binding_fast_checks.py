"""The binding's short argument tests accept exactly what its full checks accept
(CPU tensors: nothing is launched)."""

import itertools

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

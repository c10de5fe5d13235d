"""Performance cases of the verification step, through the Python binding.

Each case is one call (or one whole step) that a serving program makes once per
target pass: verification attention, greedy acceptance, stochastic acceptance
and the LM head fused with the greedy scan.  Shapes are those of the synthetic
workloads in ``synth/configs.py`` (SDAR-1.7B layer, SDAR-8B layer, long context,
ragged paged batch) and generic ones between them; values follow
``synth/generate.py`` (logits N(0, 4) with planted drafts, drafter rows
correlated with the target's), except that queries and keys are N(0, 1), the
scale a normalised head has, so that the scores spread as they do in a model.

Kinds:
  step     attention of ``layers`` layers, then the greedy accept; ``graph``
           replays them from a HIP graph captured once, as a decode loop does
  attn     verification attention of one layer
  accept   greedy accept on stored logits
  sampled  stochastic accept (temperature, caller uniforms)
  lmhead   greedy accept with the LM head fused into the scan
"""

from __future__ import annotations

import math

import torch

from paper_2606_02544_amd import binding

DEV = "cuda"
SIGMA = 2.0                    # logits ~ N(0, 4), clipped to 6 sigma
PLANT = 6.25 * SIGMA           # a planted draft is its row's unique maximum
VOCAB = 151936
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # One decode step of a small model at batch 1, launched eagerly: the
        # smallest call, where host time, launches and round trips are all there is.
        {"name": "sdar-1.7b-step", "kind": "step", "dtype": "bf16", "layers": 1, "graph": False,
         "batch": 1, "hq": 16, "hkv": 8, "d": 128, "lo": 1024, "hi": 1024, "page": 0,
         "block": 4, "ref": 4, "committed": 0, "rope": 0.0, "vocab": VOCAB},
        # The same model's step as a latency-minded server runs it: several
        # layers' attention and the accept in one captured graph.
        {"name": "sdar-1.7b-graph", "kind": "step", "dtype": "bf16", "layers": 8, "graph": True,
         "batch": 1, "hq": 16, "hkv": 8, "d": 128, "lo": 1024, "hi": 1024, "page": 0,
         "block": 4, "ref": 4, "committed": 0, "rope": 0.0, "vocab": VOCAB},
        # A layer of the larger model at an ordinary batch, contiguous cache.
        {"name": "sdar-8b-attn", "kind": "attn", "dtype": "bf16",
         "batch": 8, "hq": 32, "hkv": 8, "d": 128, "lo": 4096, "hi": 4096, "page": 0,
         "block": 16, "ref": 16, "committed": 0, "rope": 0.0},
        # Long prompts with the longest blocks: 256 packed rows per KV head.
        {"name": "long-context-attn", "kind": "attn", "dtype": "bf16",
         "batch": 16, "hq": 32, "hkv": 8, "d": 128, "lo": 16384, "hi": 16384, "page": 0,
         "block": 32, "ref": 32, "committed": 0, "rope": 0.0},
        # A full serving batch of uneven requests on a paged cache.
        {"name": "ragged-paged-attn", "kind": "attn", "dtype": "bf16",
         "batch": 64, "hq": 32, "hkv": 8, "d": 128, "lo": 512, "hi": 32768, "page": 16,
         "block": 8, "ref": 8, "committed": 0, "rope": 0.0},
        # A later step inside a block (committed slots, fewer drafts than
        # slots), uneven prefixes, rotary embedding fused into the call.
        {"name": "rope-inside-block-attn", "kind": "attn", "dtype": "bf16",
         "batch": 24, "hq": 32, "hkv": 8, "d": 128, "lo": 101, "hi": 6007, "page": 64,
         "block": 16, "ref": 11, "committed": 4, "rope": 1000000.0},
        # The paper's own setting: FP32, batch 1, block of 8.
        {"name": "f32-attn", "kind": "attn", "dtype": "f32",
         "batch": 1, "hq": 32, "hkv": 8, "d": 128, "lo": 1024, "hi": 1024, "page": 0,
         "block": 8, "ref": 8, "committed": 0, "rope": 0.0},
        # Greedy accept of an ordinary batch.
        {"name": "sdar-8b-accept", "kind": "accept", "dtype": "bf16",
         "batch": 8, "block": 16, "ref": 16, "committed": 0, "vocab": VOCAB},
        # A tokenizer whose size is no multiple of a vector load, logits in FP32.
        {"name": "odd-vocab-accept-f32", "kind": "accept", "dtype": "f32",
         "batch": 32, "block": 8, "ref": 8, "committed": 0, "vocab": 50001},
        # Stochastic accept of the longest blocks.
        {"name": "long-context-sampled", "kind": "sampled", "dtype": "bf16", "temperature": 1.0,
         "batch": 16, "block": 32, "ref": 32, "committed": 0, "vocab": VOCAB},
        # LM head of a batch-1 step: four rows against the whole weight.
        {"name": "sdar-1.7b-lmhead", "kind": "lmhead", "dtype": "bf16", "hidden": 2048,
         "batch": 1, "block": 4, "ref": 4, "committed": 0, "vocab": VOCAB},
        # LM head of a large batch with the longest blocks: a matrix product.
        {"name": "long-context-lmhead", "kind": "lmhead", "dtype": "bf16", "hidden": 4096,
         "batch": 16, "block": 32, "ref": 32, "committed": 0, "vocab": VOCAB},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _block(rng, most):
    """(block, ref, committed): a fresh block, or a later step inside one."""
    block = _log_int(rng, 1, most)
    if rng.random() < 0.6:
        return block, block, 0
    ref = rng.randint(0, block)
    return block, ref, rng.randint(0, block - max(ref, 1))


def draw(rng):
    kind = rng.choices(["attn", "attn_f32", "accept", "sampled", "lmhead", "step"],
                       [8, 2, 3, 2, 4, 2])[0]
    while True:
        c = _draw(rng, kind)
        w = work(c)
        # No dearer than the largest listed cases of the same sort (the FP32
        # attention's products run at the vector rate, so they bound it sooner).
        if c["kind"] in ("attn", "step") and c["dtype"] == "f32":
            fits = w["bytes"] < 1e8 and w["flops"] < 3e9
        else:
            fits = w["bytes"] < 2.5e9 and w["flops"] < (6.4e11 if c["kind"] == "lmhead" else 3e11)
        if fits:
            return c


def _draw(rng, kind):
    if kind in ("attn", "attn_f32", "step"):
        block, ref, committed = _block(rng, 32)
        hkv = rng.choice([1, 2, 4, 8, 8, 8])
        hi = _log_int(rng, 16, 32768)
        c = {"kind": "attn", "dtype": "bf16", "batch": _log_int(rng, 1, 64),
             "hq": hkv * rng.choice([1, 2, 4, 4, 8]), "hkv": hkv, "d": rng.choice([64, 128, 128, 128]),
             "lo": hi if rng.random() < 0.4 else rng.randint(0, hi), "hi": hi,
             "page": rng.choice([0, 0, 16, 16, 32, 64]), "block": block, "ref": ref,
             "committed": committed, "rope": rng.choice([0.0, 0.0, 10000.0, 1000000.0])}
        if kind == "attn_f32":
            c["dtype"] = "f32"
            c["batch"] = _log_int(rng, 1, 8)
        if kind == "step":
            c.update(kind="step", dtype=rng.choice(["bf16", "bf16", "f32"]), layers=rng.randint(1, 4),
                     graph=rng.random() < 0.5, batch=_log_int(rng, 1, 8), vocab=_log_int(rng, 1000, VOCAB))
        return c
    block, ref, committed = _block(rng, 32)
    c = {"kind": kind, "dtype": "bf16" if kind == "lmhead" else rng.choice(["bf16", "bf16", "f32"]),
         "batch": _log_int(rng, 1, 32), "block": block, "ref": ref, "committed": committed,
         "vocab": VOCAB if rng.random() < 0.5 else _log_int(rng, 1000, VOCAB)}
    if kind == "lmhead":
        c["hidden"] = 64 * _log_int(rng, 8, 64)
        c["batch"] = _log_int(rng, 1, 16)
    if kind == "sampled":
        c["temperature"] = rng.choice([1.0, 1.0, 0.7, 1.3])
        c["batch"] = _log_int(rng, 1, 16)
        if not c["ref"]:                               # a stochastic step has drafts
            c["ref"], c["committed"] = block, 0
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
class _Draws:
    """Random numbers of one state: big tensors on the GPU, small ones on the host."""

    def __init__(self, seed):
        self.gpu = torch.Generator(device=DEV).manual_seed(seed)
        self.cpu = torch.Generator().manual_seed(seed)

    def normal(self, shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.gpu, device=DEV, dtype=dtype)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.cpu)

    def perm(self, n):
        return torch.randperm(n, generator=self.cpu)

    def ints(self, hi, *shape):
        return torch.randint(0, hi, shape, generator=self.cpu, dtype=torch.int32)


def _to_gpu(t):
    return t.to(torch.int32).to(DEV)


def _slots(c, r):
    """step_map [batch, B], num_ref [batch]: `ref` drafted slots in a random
    order, `committed` ones, the rest not drafted; and the verification row of
    each draft [batch, L]."""
    b, B, L = c["batch"], c["block"], c["ref"]
    step = torch.full((b, B), L + 1)
    rows = torch.zeros((b, L), dtype=torch.int64)
    for s in range(b):
        order = r.perm(B)
        step[s, order[:L]] = torch.arange(1, L + 1)
        step[s, order[L:L + c["committed"]]] = 0
        rows[s] = order[:L]
    return step, torch.full((b,), L), rows


def _lens(c, r):
    """Prefix lengths spread evenly over [lo, hi], in a random order."""
    b = c["batch"]
    u = (torch.arange(b) + r.uniform(b)) / b
    lens = c["lo"] + (u * (c["hi"] - c["lo"] + 1)).floor()
    return lens.clamp(c["lo"], c["hi"]).to(torch.int64)[r.perm(b)]


def _attn_inputs(c, r, slots):
    dt, d = DTYPES[c["dtype"]], c["d"]
    b, n_new = c["batch"], c["block"] + c["ref"]
    step, num_ref, _ = slots
    lens = _lens(c, r)
    s = {"q": r.normal((b, n_new, c["hq"], d), dt), "k_new": r.normal((b, n_new, c["hkv"], d), dt),
         "v_new": r.normal((b, n_new, c["hkv"], d), dt), "prefix_lens": _to_gpu(lens),
         "step_map": _to_gpu(step), "num_ref": _to_gpu(num_ref), "block_table": None}
    if c["page"]:
        per = (lens + c["page"] - 1) // c["page"]
        total = int(per.sum())
        table = torch.full((b, -(-c["hi"] // c["page"])), total)     # unused entries: a spare page
        order, at = r.perm(total), 0
        for i in range(b):
            n = int(per[i])
            table[i, :n] = order[at:at + n]
            at += n
        s["block_table"] = _to_gpu(table)
        shape = (total + 1, c["page"], c["hkv"], d)
    else:
        shape = (b, c["hi"], c["hkv"], d)
    s["k_cache"], s["v_cache"] = r.normal(shape, dt), r.normal(shape, dt)
    return s


def _plants(c, r):
    """Draft ids [batch, L] and which of them are planted as the argmax."""
    ids = r.ints(c["vocab"], c["batch"], c["ref"])
    return ids, r.uniform(c["batch"], c["ref"]) < 0.6


def _logits_inputs(c, r, slots):
    b, B, L, V = c["batch"], c["block"], c["ref"], c["vocab"]
    step, num_ref, rows = slots
    logits = r.normal((b, B, V)).mul_(SIGMA).clamp_(-6 * SIGMA, 6 * SIGMA).to(DTYPES[c["dtype"]])
    ids, planted = _plants(c, r)
    at = planted.nonzero(as_tuple=True)
    logits[at[0].to(DEV), rows[at].to(DEV), ids[at].long().to(DEV)] = PLANT
    return {"logits": logits, "draft_ids": _to_gpu(ids), "step_map": _to_gpu(step),
            "num_ref": _to_gpu(num_ref)}


def _sampled_inputs(c, r, slots):
    s = _logits_inputs(c, r, slots)
    b, L, V = c["batch"], c["ref"], c["vocab"]
    rows = slots[2].to(DEV)
    x = r.normal((b, L, V)).mul_(0.6 * SIGMA)
    x += 0.8 * s["logits"].gather(1, rows[:, :, None].expand(b, L, V)).float()
    x.clamp_(-6 * SIGMA, 6 * SIGMA).scatter_(2, s["draft_ids"].long()[:, :, None], PLANT)
    s["draft_logits"] = x.to(DTYPES[c["dtype"]])
    s["uniforms"] = r.uniform(b, L + 1).to(DEV)
    return s


def _lmhead_inputs(c, r, slots):
    b, B, H = c["batch"], c["block"], c["hidden"]
    step, num_ref, rows = slots
    weight = r.normal((c["vocab"], H), torch.bfloat16).mul_(SIGMA / math.sqrt(H))
    hidden = r.normal((b, B, H))
    ids, planted = _plants(c, r)
    at = planted.nonzero(as_tuple=True)
    if len(at[0]):
        w = weight[ids[at].long().to(DEV)].float()
        pull = w * (6.25 * SIGMA / w.square().sum(1, keepdim=True))
        i, k = at[0].to(DEV), rows[at].to(DEV)
        hidden[i, k] = 0.5 * hidden[i, k] + pull
    return {"hidden": hidden.to(torch.bfloat16), "weight": weight, "draft_ids": _to_gpu(ids),
            "step_map": _to_gpu(step), "num_ref": _to_gpu(num_ref)}


def prepare(case, seed):
    c, r = dict(case), _Draws(seed)
    slots = _slots(c, r)
    kind = c["kind"]
    if kind == "attn":
        return {"case": c, "attn": _attn_inputs(c, r, slots)}
    if kind == "accept":
        return {"case": c, "accept": _logits_inputs(c, r, slots)}
    if kind == "sampled":
        return {"case": c, "sampled": _sampled_inputs(c, r, slots)}
    if kind == "lmhead":
        return {"case": c, "lmhead": _lmhead_inputs(c, r, slots)}
    state = {"case": c, "layers": [_attn_inputs(c, r, slots) for _ in range(c["layers"])],
             "accept": _logits_inputs(c, r, slots)}
    if c["graph"]:
        _step(state)                                   # grows the binding's workspaces first
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            state["out"] = _step(state)
        state["graph"] = graph
    return state


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _attention(c, s):
    return binding.verify_attention(
        s["q"], s["k_new"], s["v_new"], s["k_cache"], s["v_cache"], s["block_table"],
        s["prefix_lens"], s["step_map"], s["num_ref"], block_size=c["block"], max_ref=c["ref"],
        max_prefix_len=c["hi"], page_size=c["page"], rope_theta=c["rope"])


def _step(state):
    c, a = state["case"], state["accept"]
    outs = [_attention(c, s) for s in state["layers"]]
    return outs + [binding.verify_accept(a["logits"], a["draft_ids"], a["step_map"], a["num_ref"])]


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "attn":
        return _attention(c, state["attn"])
    if kind == "accept":
        a = state["accept"]
        return binding.verify_accept(a["logits"], a["draft_ids"], a["step_map"], a["num_ref"])
    if kind == "sampled":
        a = state["sampled"]
        return binding.verify_accept_sampled(a["logits"], a["draft_logits"], a["draft_ids"],
                                             a["step_map"], a["num_ref"], a["uniforms"],
                                             temperature=c["temperature"])
    if kind == "lmhead":
        a = state["lmhead"]
        return binding.verify_accept_lmhead(a["hidden"], a["weight"], a["draft_ids"],
                                            a["step_map"], a["num_ref"])
    if c["graph"]:
        state["graph"].replay()
        return state["out"]
    return _step(state)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _attn_work(c):
    e = 4 if c["dtype"] == "f32" else 2
    b, n_new, d = c["batch"], c["block"] + c["ref"], c["d"]
    keys = b * (c["lo"] + c["hi"]) / 2
    moved = 2 * keys * c["hkv"] * d * e + b * n_new * (2 * c["hq"] + 2 * c["hkv"]) * d * e
    moved += b * n_new * c["hq"] * 4
    return moved, 4 * c["hq"] * d * n_new * (keys + b * n_new / 2)


def _accept_work(c, rows_per_seq):
    e = 4 if c["dtype"] == "f32" else 2
    rows = c["batch"] * rows_per_seq
    return rows * c["vocab"] * e, 4 * rows * c["vocab"]


def work(case):
    c = case
    kind = c["kind"]
    if kind == "attn":
        moved, ops = _attn_work(c)
    elif kind == "accept":
        moved, ops = _accept_work(c, c["block"] - c["committed"])
    elif kind == "sampled":
        moved, ops = _accept_work(c, 2 * c["ref"])
    elif kind == "lmhead":
        rows = c["batch"] * c["block"]
        moved = (c["vocab"] + rows) * c["hidden"] * 2
        ops = 2 * rows * c["vocab"] * c["hidden"]
    else:
        moved, ops = _accept_work(c, c["block"] - c["committed"])
        m, o = _attn_work(c)
        moved, ops = moved + c["layers"] * m, ops + c["layers"] * o
    # Step maps, draft ids and the small outputs of each sequence.
    return {"bytes": moved + c["batch"] * 16 * (c["block"] + c["ref"] + 1), "flops": ops}


def tolerance(case):
    # bf16 attention rounds its output (and each split's partial) once: 2^-9 of
    # a value.  FP32 attention, and the probabilities of every other kind, are
    # sums in FP32.  Whole values (ids, lengths) differ only where two logits,
    # or the draw's running sum and its target, are equal to rounding.
    if case["kind"] in ("attn", "step") and case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 4e-2}
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _rotate(x, pos, theta):
    """x [b, n, heads, d] turned by pos [b, n] (dims i and i + d/2 pair)."""
    half = x.shape[-1] // 2
    freq = theta ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / x.shape[-1])
    ang = pos.double()[:, :, None, None] * freq
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * ang.cos() - hi * ang.sin(), hi * ang.cos() + lo * ang.sin()], -1)


def _exact_attention(c, s):
    b, B, L, g, d = c["batch"], c["block"], c["ref"], c["hq"] // c["hkv"], c["d"]
    n = B + L
    step, lens = s["step_map"].long(), s["prefix_lens"].long()
    # Sections and step labels of the new slots, then the temporal mask.
    data = torch.arange(n, device=DEV) >= B
    tau = torch.cat([step, torch.arange(1, L + 1, device=DEV).expand(b, L)], 1)
    ti, tj = tau[:, :, None], tau[:, None, :]
    di, dj = data[None, :, None], data[None, None, :]
    sees = torch.where(di, torch.where(dj, tj <= ti, tj > ti), torch.where(dj, tj < ti, tj >= ti))
    sees |= ~dj & (tj == 0)
    q, k_new, v_new = s["q"].double(), s["k_new"].double(), s["v_new"].double()
    if c["rope"]:
        slot = torch.argsort(torch.where((step >= 1) & (step <= L), step, L + 1), dim=1, stable=True)[:, :L]
        pos = lens[:, None] + torch.cat([torch.arange(B, device=DEV).expand(b, B), slot], 1)
        q, k_new = _rotate(q, pos, c["rope"]), _rotate(k_new, pos, c["rope"])
    out = torch.empty((b, n, c["hq"], d), dtype=torch.float64, device=DEV)
    lse = torch.empty((b, c["hq"], n), dtype=torch.float64, device=DEV)
    for i in range(b):
        m = int(lens[i])
        if c["page"]:
            pages = s["block_table"][i, :-(-m // c["page"])].long()
            k, v = (s[t][pages].reshape(-1, c["hkv"], d)[:m] for t in ("k_cache", "v_cache"))
        else:
            k, v = s["k_cache"][i, :m], s["v_cache"][i, :m]
        k = torch.cat([k.double(), k_new[i]]).permute(1, 2, 0).contiguous()     # [hkv, d, m + n]
        v = torch.cat([v.double(), v_new[i]]).permute(1, 0, 2).contiguous()
        rows = q[i].view(n, c["hkv"], g, d).permute(1, 0, 2, 3).reshape(c["hkv"], n * g, d)
        x = torch.matmul(rows, k).div_(math.sqrt(d)).view(c["hkv"], n, g, m + n)
        x[..., m:].masked_fill_(~sees[i][None, :, None, :], -math.inf)
        z = torch.logsumexp(x, -1)
        p = (x - z[..., None]).exp_().view(c["hkv"], n * g, m + n)
        out[i] = torch.matmul(p, v).view(c["hkv"], n, g, d).permute(1, 0, 2, 3).reshape(n, c["hq"], d)
        lse[i] = z.permute(0, 2, 1).reshape(c["hq"], n)
    return out, lse


def _accepted(hit):
    """Leading true values of each row."""
    return hit.long().cumprod(1).sum(1).to(torch.int32)


def _draft_rows(c, a):
    """Verification row of each draft [batch, L]."""
    step = a["step_map"].long()
    key = torch.where((step >= 1) & (step <= c["ref"]), step, c["ref"] + 1)
    return torch.argsort(key, dim=1, stable=True)[:, :c["ref"]]


def _exact_greedy(c, a, top, ids, z, drafted):
    """Outputs from each row's largest logit, its index, its log-sum-exp and the
    drafted tokens' logits."""
    scanned = a["step_map"] >= 1
    rows = _draft_rows(c, a)
    target = torch.where(scanned, ids.to(torch.int32), -1)
    conf = torch.where(scanned, (top - z).exp(), 0.0)
    prob = (drafted - z.gather(1, rows)).exp()
    return target, conf, prob, _accepted(target.gather(1, rows) == a["draft_ids"])


def _exact_accept(c, a):
    x = a["logits"].double()
    top = x.amax(-1)
    index = torch.arange(c["vocab"], device=DEV)
    ids = torch.stack([torch.where(r == t[:, None], index, c["vocab"]).amin(-1)   # lowest on ties
                       for r, t in zip(x, top)])
    rows = _draft_rows(c, a)
    drafted = x[torch.arange(c["batch"], device=DEV)[:, None], rows, a["draft_ids"].long()]
    return _exact_greedy(c, a, top, ids, torch.logsumexp(x, -1), drafted)


def _exact_sampled(c, a):
    b, L = c["batch"], c["ref"]
    rows, at = _draft_rows(c, a), torch.arange(b, device=DEV)[:, None]
    ids, u = a["draft_ids"].long(), a["uniforms"].double()
    p = torch.softmax(a["logits"][at, rows].double() / c["temperature"], -1)     # [b, L, V]
    f = torch.softmax(a["draft_logits"].double() / c["temperature"], -1)
    pt, pf = (t.gather(2, ids[..., None])[..., 0] for t in (p, f))
    acc = _accepted(u[:, :L] * pf < pt)
    token = torch.full((b,), -1, dtype=torch.int32, device=DEV)
    for i in range(b):
        n = int(acc[i])
        if n < L:
            rest = (p[i, n] - f[i, n]).clamp_(min=0)
            run_sum = (rest if rest.sum() > 0 else p[i, n]).cumsum(0)
            token[i] = int((run_sum <= u[i, L] * run_sum[-1]).sum())
    return pt, pf, acc, token


def _exact_lmhead(c, a):
    b, B = c["batch"], c["block"]
    h = a["hidden"].double().view(b * B, -1)
    x = torch.empty((b * B, c["vocab"]), dtype=torch.float64, device=DEV)
    for v in range(0, c["vocab"], 16384):
        x[:, v:v + 16384] = h @ a["weight"][v:v + 16384].double().t()
    x = x.view(b, B, -1)
    top, ids = x.max(-1)
    drafted = x[torch.arange(b, device=DEV)[:, None], _draft_rows(c, a), a["draft_ids"].long()]
    return _exact_greedy(c, a, top, ids, torch.logsumexp(x, -1), drafted)


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "step":
        c["graph"] = False
    state = prepare(c, seed)
    if c["kind"] == "attn":
        return _exact_attention(c, state["attn"])
    if c["kind"] == "accept":
        return _exact_accept(c, state["accept"])
    if c["kind"] == "sampled":
        return _exact_sampled(c, state["sampled"])
    if c["kind"] == "lmhead":
        return _exact_lmhead(c, state["lmhead"])
    return [_exact_attention(c, s) for s in state["layers"]] + [_exact_accept(c, state["accept"])]

"""The calls that a serving worker makes of this package, as cases for timing.

Six kinds of case, each one pass of a step through the public entry points:

  decode   one projection, one token per request            lora_apply_decode
  layer    the seven projections of a dense decoder layer   lora_plan_apply_decode_multi, lora_apply_decode_planned, ..._multi
  catalog  tokens that name adapters by catalog id          lora_slot_lookup, lora_apply_decode
  moe      gate, up and down of a packed expert layer       moe_plan_route, moe_lora_apply_multi, moe_lora_apply_down
  prefill  prompts as contiguous runs of rows               lora_apply_segmented
  load     an adapter from host memory into a GPU slot      lora_slots_upload_experts

Sizes are those of the package's benchmark workloads (workloads/gen.py) and lie around them.  Activations
are N(0, 1), adapters N(0, 0.02), alpha is twice the rank, everything bf16; what a program keeps between
steps (slot tables, plans, workspaces) is made in prepare().
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2605_13779_amd as M

ZIPF = 1.1                                   # slot popularity of decode traffic
RANKS = (1, 2, 4, 6, 8, 12, 16, 24, 32, 48, 64)


def listed():
    return [
        # A single request in flight: nothing but latency.
        dict(name="decode, one token", kind="decode", tokens=1, d_in=2560, d_out=2560, rank=16, slots=64, map="zipf"),
        # A few dozen requests on the widest adapters a slot can hold (the tables of the rank-64 prefill, while decoding).
        dict(name="decode, rank 64", kind="decode", tokens=93, d_in=7168, d_out=7168, rank=64, slots=16, map="uniform"),
        # A full decode batch of a dense 4B-like model, all seven projections of one layer.
        dict(name="layer, 256 tokens", kind="layer", tokens=256, hidden=2560, kv=1024, inter=9728, rank=16, slots=64),
        # The same layer under a batch beyond the usual one, an odd number of rows.
        dict(name="layer, 1001 tokens", kind="layer", tokens=1001, hidden=2560, kv=1024, inter=9728, rank=16, slots=64),
        # A compact catalog: every token brings a rank-1 adapter of its own, named by catalog id.
        dict(name="catalog, rank 1", kind="catalog", tokens=512, d_in=4096, d_out=4096, rank=1, slots=1024),
        # Expert layer of a 30B-like mixture: a decode step of a few dozen requests ...
        dict(name="moe, 48 tokens", kind="moe", tokens=48, hidden=2048, inter=768, experts=128, top_k=8, slots=32, rank=8),
        # ... the benchmark's batch ...
        dict(name="moe, 2048 tokens", kind="moe", tokens=2048, hidden=2048, inter=768, experts=128, top_k=8, slots=32, rank=8),
        # ... and a prefill-sized one.
        dict(name="moe, 8000 tokens", kind="moe", tokens=8000, hidden=2048, inter=768, experts=128, top_k=8, slots=32, rank=8),
        # Prompts on adapters of the usual rank (the q projection of the dense layer above).
        dict(name="prefill, rank 16", kind="prefill", tokens=8192, segments=16, d_in=2560, d_out=2560, rank=16, slots=64),
        # Prompts on rank-64 adapters.
        dict(name="prefill, rank 64", kind="prefill", tokens=8192, segments=16, d_in=7168, d_out=7168, rank=64, slots=16),
        # The widest projection and a batch of long prompts, the largest call.
        dict(name="prefill, rank 64, wide", kind="prefill", tokens=14999, segments=11, d_in=7168, d_out=18432, rank=64, slots=16),
        # A cold adapter: 256 host tensors (128 experts) into a slot.
        dict(name="load, 128 experts", kind="load", d_in=2048, d_out=768, experts=128, table_rank=8, rank=8),
    ]


def _log(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def _draw(rng):
    kind = rng.choice(("decode", "layer", "catalog", "moe", "prefill", "prefill", "load"))
    if kind == "decode":
        return dict(kind=kind, tokens=_log(rng, 1, 2048), d_in=_log(rng, 256, 9728, 8), d_out=_log(rng, 256, 9728, 8),
                    rank=rng.choice(RANKS), slots=rng.randint(1, 64), map=rng.choice(("zipf", "uniform")))
    if kind == "layer":
        hidden = _log(rng, 1024, 4096, 64)
        return dict(kind=kind, tokens=_log(rng, 1, 1024), hidden=hidden, kv=_log(rng, 256, hidden, 64),
                    inter=_log(rng, hidden, 9728, 64), rank=rng.choice((8, 12, 16, 32)), slots=rng.randint(1, 64))
    if kind == "catalog":
        slots = _log(rng, 64, 1024)
        return dict(kind=kind, tokens=_log(rng, 1, slots), d_in=_log(rng, 1024, 7168, 8), d_out=_log(rng, 1024, 7168, 8),
                    rank=rng.choice((1, 1, 2, 4)), slots=slots)
    if kind == "moe":
        experts = rng.choice((8, 16, 64, 128))
        return dict(kind=kind, tokens=_log(rng, 1, 8000), hidden=_log(rng, 1024, 4096, 64), inter=_log(rng, 384, 2048, 64),
                    experts=experts, top_k=min(experts // 2, rng.choice((1, 2, 4, 6, 8))), slots=rng.randint(1, 32),
                    rank=rng.choice((2, 4, 8, 8, 16)))
    if kind == "prefill":
        tokens = _log(rng, 64, 16384)
        return dict(kind=kind, tokens=tokens, segments=min(tokens, _log(rng, 1, 64)), d_in=_log(rng, 512, 9728, 8),
                    d_out=_log(rng, 512, 18432, 8), rank=rng.choice(RANKS[3:]), slots=rng.randint(1, 64))
    table = rng.choice((8, 16, 32, 64))
    experts = rng.choice((1, 8, 32, 128))
    return dict(kind=kind, d_in=_log(rng, 512, 4096, 64), d_out=_log(rng, 512, 4096, 64), experts=experts,
                table_rank=table, rank=rng.choice((table, rng.randint(max(1, table // 4), table))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most and (c["kind"] != "load" or work(c)["bytes"] <= 64e6):
            return c


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


# ---- inputs ------------------------------------------------------------------------------------------

def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _site(g, d_in, d_out, rank, slots, experts=0, ids=None):
    site = M.Site(d_in, d_out, rank, slots, n_experts=experts)
    lead = (experts,) if experts else ()
    for s in range(slots):
        A, B = _normal(g, lead + (rank, d_in), 0.02), _normal(g, lead + (d_out, rank), 0.02)
        M.lora_slots_upload(site, s, s if ids is None else int(ids[s]), A, B, rank, 2.0 * rank)
    return site


def _zipf_p(slots):
    w = np.arange(1, slots + 1, dtype=np.float64) ** -ZIPF
    return w / w.sum()


def _token_slot(r, tokens, slots, how):
    if how == "zipf":                        # popular slots first
        ts = r.choice(slots, size=tokens, p=_zipf_p(slots))
    else:                                    # uniform, with requests on the base model (-1) among them
        ts = r.integers(-1, slots, size=tokens)
    return torch.from_numpy(ts.astype(np.int32)).cuda()


def _segments(r, tokens, n):
    """Prompt lengths: lognormal(6, 0.8) scaled to the batch, each at least one row."""
    ell = np.exp(6.0 + 0.8 * r.standard_normal(n))
    cuts = np.floor(np.cumsum(ell) / ell.sum() * (tokens - n)).astype(np.int64) + np.arange(1, n + 1)
    cuts[-1] = tokens
    return np.concatenate([[0], cuts]).astype(np.int32)


def prepare(case, seed):
    c = SimpleNamespace(**case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = np.random.default_rng(seed)
    s = SimpleNamespace(kind=c.kind)
    if c.kind == "decode":
        s.site = _site(g, c.d_in, c.d_out, c.rank, c.slots)
        s.x, s.y = _normal(g, (c.tokens, c.d_in)), _normal(g, (c.tokens, c.d_out))
        s.token_slot = _token_slot(r, c.tokens, c.slots, c.map)
    elif c.kind == "layer":
        h, kv, inter = c.hidden, c.kv, c.inter
        shapes = ((h, h), (h, kv), (h, kv), (h, h), (h, inter), (h, inter), (inter, h))      # q k v o gate up down
        s.sites = [_site(g, i, o, c.rank, c.slots) for i, o in shapes]
        s.ys = [_normal(g, (c.tokens, o)) for _, o in shapes]
        s.x_attn, s.x_o, s.x_mlp = (_normal(g, (c.tokens, h)) for _ in range(3))
        s.x_down = _normal(g, (c.tokens, inter))
        s.token_slot, s.slots = _token_slot(r, c.tokens, c.slots, "zipf"), c.slots
        s.plan = M.Plan(c.tokens, c.slots)
    elif c.kind == "catalog":
        ids = r.choice(10 ** 6, size=c.slots, replace=False)
        s.site = _site(g, c.d_in, c.d_out, c.rank, c.slots, ids=ids)
        s.x, s.y = _normal(g, (c.tokens, c.d_in)), _normal(g, (c.tokens, c.d_out))
        s.ids = torch.from_numpy(ids[r.permutation(c.slots)[:c.tokens]].astype(np.int64)).cuda()
        s.token_slot = torch.empty(c.tokens, dtype=torch.int32, device="cuda")
    elif c.kind == "moe":
        s.gate, s.up = (_site(g, c.hidden, c.inter, c.rank, c.slots, c.experts) for _ in range(2))
        s.down = _site(g, c.inter, c.hidden, c.rank, c.slots, c.experts)
        s.x, s.x_down = _normal(g, (c.tokens, c.hidden)), _normal(g, (c.tokens * c.top_k, c.inter))
        s.y_gate, s.y_up = (_normal(g, (c.tokens * c.top_k, c.inter)) for _ in range(2))
        s.y_down = _normal(g, (c.tokens, c.hidden))
        logits = torch.randn((c.tokens, c.experts), generator=g, device="cuda")
        top = torch.topk(logits, c.top_k, dim=1)
        s.topk, s.pair_w = top.indices.to(torch.int32).contiguous(), torch.softmax(top.values, dim=1).contiguous()
        s.token_slot = torch.from_numpy(r.integers(0, c.slots, size=c.tokens).astype(np.int32)).cuda()
        s.plan = M.Plan(c.tokens * c.top_k, c.slots * c.experts)
        s.workspace = torch.empty(M.moe_down_workspace_bytes(c.tokens, c.top_k, c.hidden), dtype=torch.uint8, device="cuda")
        s.slots, s.experts = c.slots, c.experts
    elif c.kind == "prefill":
        s.site = _site(g, c.d_in, c.d_out, c.rank, c.slots)
        s.x, s.y = _normal(g, (c.tokens, c.d_in)), _normal(g, (c.tokens, c.d_out))
        s.seg_off = _segments(r, c.tokens, c.segments)
        s.seg_slot = r.integers(0, c.slots, size=c.segments).astype(np.int32)
    else:
        s.site, s.rank = M.Site(c.d_in, c.d_out, c.table_rank, 4, n_experts=c.experts), c.rank
        cpu = torch.Generator().manual_seed(seed)
        A = (torch.randn((c.experts, c.rank, c.d_in), generator=cpu) * 0.02).to(torch.bfloat16)
        B = (torch.randn((c.experts, c.d_out, c.rank), generator=cpu) * 0.02).to(torch.bfloat16)
        s.tensors = M.ExpertTensors(list(A.view(torch.int16).numpy().view(np.uint16)), list(B.view(torch.int16).numpy().view(np.uint16)))
        s.tables = [b.view(4, -1)[2] for b in (s.site.bufs[0][:site_bytes(c)[0]], s.site.bufs[1][:site_bytes(c)[1]])]
    return s


def site_bytes(c):
    """Bytes of the A and B tables of a load case's site (four slots)."""
    r_pad = 1 << (c.table_rank - 1).bit_length()
    return 8 * c.experts * r_pad * c.d_in, 8 * c.experts * r_pad * c.d_out


def run(s):
    if s.kind == "decode":
        M.lora_apply_decode(s.site, s.x, s.y, s.token_slot)
        return s.y
    if s.kind == "layer":
        q, k, v, o, gate, up, down = s.sites
        yq, yk, yv, yo, yg, yu, yd = s.ys
        M.lora_plan_apply_decode_multi([q, k, v], s.plan, s.token_slot, s.slots, [s.x_attn] * 3, [yq, yk, yv])
        M.lora_apply_decode_planned(o, s.plan, s.x_o, yo)
        M.lora_apply_decode_multi([gate, up], s.plan, [s.x_mlp] * 2, [yg, yu])
        M.lora_apply_decode_planned(down, s.plan, s.x_down, yd)
        return s.ys
    if s.kind == "catalog":
        M.lora_slot_lookup(s.site, s.ids, s.token_slot)
        M.lora_apply_decode(s.site, s.x, s.y, s.token_slot)
        return s.token_slot, s.y
    if s.kind == "moe":
        M.moe_plan_route(s.plan, s.topk, s.token_slot, s.slots, s.experts)
        M.moe_lora_apply_multi([s.gate, s.up], s.plan, [s.x, s.x], [s.y_gate, s.y_up])
        M.moe_lora_apply_down(s.down, s.plan, s.x_down, s.pair_w, s.token_slot, s.workspace, s.y_down)
        return s.y_gate, s.y_up, s.y_down
    if s.kind == "prefill":
        M.lora_apply_segmented(s.site, s.x, s.y, s.seg_off, s.seg_slot)
        return s.y
    M.lora_slots_upload_experts(s.site, 2, 77, s.tensors, None, s.rank, 2.0 * s.rank)
    return s.tables


# ---- what a pass cannot do without ---------------------------------------------------------------------

def _touched(n, p):
    """Expected number of distinct picks in n draws with probabilities p."""
    return float(np.sum(1.0 - (1.0 - np.asarray(p)) ** n))


def work(case):
    c = SimpleNamespace(**case)
    if c.kind == "load":
        r_pad = 1 << (c.table_rank - 1).bit_length()
        return {"bytes": 2 * c.experts * (c.rank + r_pad) * (c.d_in + c.d_out), "flops": 0}
    if c.kind == "moe":
        pairs, keys = c.tokens * c.top_k, c.slots * c.experts
        per_key = c.top_k / (c.slots * c.experts)          # a token touches a given (slot, expert) with this probability
        touched = keys * (1.0 - (1.0 - per_key) ** c.tokens)
        rows = 2 * (c.tokens * c.hidden + 2 * 2 * pairs * c.inter) + 2 * (pairs * c.inter + 2 * c.tokens * c.hidden)
        return {"bytes": rows + 3 * touched * c.rank * (c.hidden + c.inter) * 2 + 4 * (2 * pairs + c.tokens),
                "flops": 3 * 2 * pairs * c.rank * (c.hidden + c.inter)}
    if c.kind == "layer":
        h, kv, inter = c.hidden, c.kv, c.inter
        ins, outs = 3 * h + inter, 3 * h + 2 * kv + 2 * inter            # one x for q, k, v and one for gate, up
        both = 6 * h + inter + outs
        touched = _touched(c.tokens, _zipf_p(c.slots))
        return {"bytes": 2 * c.tokens * (ins + 2 * outs) + touched * c.rank * both * 2 + 4 * c.tokens,
                "flops": 2 * c.tokens * c.rank * both}
    if c.kind == "prefill":
        rows, touched, extra = c.tokens, _touched(c.segments, np.full(c.slots, 1 / c.slots)), 8 * c.segments
    elif c.kind == "catalog":
        rows, touched, extra = c.tokens, c.tokens, 16 * c.tokens + 12 * c.slots
    elif c.map == "zipf":
        rows, touched, extra = c.tokens, _touched(c.tokens, _zipf_p(c.slots)), 4 * c.tokens
    else:
        rows = c.tokens * c.slots / (c.slots + 1)
        touched, extra = _touched(c.tokens, np.full(c.slots, 1 / (c.slots + 1))), 4 * c.tokens
    return {"bytes": 2 * rows * (c.d_in + 2 * c.d_out) + touched * c.rank * (c.d_in + c.d_out) * 2 + extra,
            "flops": 2 * rows * c.rank * (c.d_in + c.d_out)}


def tolerance(case):
    """bf16 results of fp32 sums: two correct roundings of one sum are at most one bf16 step (2^-8) apart.  A
    load moves bytes."""
    return "exact" if case["kind"] == "load" else {"rel": 4e-3, "max": 1.6e-2}

"""The work that is measured: passes of the KV-cache eviction path through its public entry points.

Four kinds of pass, as the program around a language model makes them:

  evict       the prefill step of one layer: scores -> selection -> compaction;
  accumulate  the scores with every row as an accumulator (window = sequence: plain accumulation);
  attend      the same step beside the attention of the observed rows, which hands over the rows'
              normalisers: attention -> scores -> selection -> compaction;
  decode      one generation step on the compact cache, one of a loop of such steps.

Inputs are Gaussian queries, keys and values with what the method looks for: a direction that the
query heads of a KV head share, an attention sink at token 0, and heavy-hitter keys along the mean
query.  The heavy hitters are as many as the selected budget and stand out clearly, so that the
retained set is decided by the data and not by the last bits of two nearly equal scores.
"""
import math

import torch

from paper_2506_03762_amd import binding as B

QUERY_BIAS = 4.0     # of the queries' mean, along a random direction per KV head
HITTER_KEY = 2.0     # a heavy hitter's part along the mean query, over the length of a Gaussian key
SINK_KEY = 4.0       # token 0's key is this much longer
TOKENS_AHEAD = 8     # generated tokens a decode state holds; a loop's steps take them in turn


def _evict(name, batch, hq, hkv, d, n, window, budget, recent, **more):
    case = dict(kind="evict", batch=batch, hq=hq, hkv=hkv, d=d, n=n, window=window, budget=budget,
                recent=recent, sink=0, dtype="bf16", layout="bhnd", fixed_scale=False,
                value_prior=True)
    if name:
        case["name"] = name
    case.update(more)
    return case


def _decode(name, batch, hq, hkv, d, n, budget, recent, **more):
    case = dict(kind="decode", batch=batch, hq=hq, hkv=hkv, d=d, n=n, budget=budget, recent=recent,
                sink=0, dtype="bf16", value_prior=False, static=False)
    if name:
        case["name"] = name
    case.update(more)
    return case


def listed():
    return [
        # the smallest problem: a short prompt of a small fp32 model, where latency is everything
        _evict("evict_tiny_f32", 1, 2, 2, 64, 512, 32, 128, 32, dtype="f32"),
        # one layer of a 7B multi-head model after a prompt of 4096 tokens
        _evict("evict_4k", 1, 32, 32, 128, 4096, 64, 512, 64),
        # one layer of a grouped-query model after a long prompt: the headline workload
        _evict("evict_32k", 1, 32, 8, 128, 32768, 64, 2048, 64),
        # one layer of a batch of long prompts, a fifth of the cache kept: the most memory traffic
        _evict("evict_16k_batch4", 4, 32, 32, 128, 16384, 64, 3276, 64),
        # sizes that divide nothing: three prompts in token-major layout, head dimension 64, sinks
        _evict("evict_ragged_d64", 3, 12, 4, 64, 5003, 40, 701, 33, sink=4, layout="bnhd"),
        # eight query heads per KV head: more observed rows than one tile of the kernels holds
        _evict("evict_wide_group", 1, 64, 8, 128, 16384, 64, 1638, 64),
        # plain accumulated attention scores (every row observed), the baseline policy the method
        # is compared with: at 4096 tokens, and at 32768, the most arithmetic
        _evict("accumulate_4k", 1, 32, 32, 128, 4096, 4096, 512, 64, kind="accumulate",
               fixed_scale=True, value_prior=False),
        _evict("accumulate_32k", 1, 32, 8, 128, 32768, 32768, 2048, 64, kind="accumulate",
               fixed_scale=True, value_prior=False),
        # eviction beside the attention of the observed rows, long grouped-query prompt
        _evict("attend_32k", 1, 32, 8, 128, 32768, 64, 2048, 64, kind="attend", fixed_scale=True),
        # generation with running eviction: a batch of eight with 32 heads
        _decode("decode_batch8", 8, 32, 32, 128, 4096, 1024, 64),
        # generation for one sequence of a grouped-query model: few heads, bound by latency
        _decode("decode_gqa_single", 1, 32, 8, 128, 32768, 2048, 64),
        # generation for a batch with eight query heads per KV head
        _decode("decode_wide_group", 16, 64, 8, 128, 16384, 1536, 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the ranges that the listed ones stand for, odd ones among them."""
    kind = rng.choice(["evict", "evict", "evict", "attend", "accumulate", "decode", "decode"])
    d = rng.choice([64, 128, 128])
    hkv = rng.choice([2, 4, 8, 8, 16, 32])
    group = rng.choice([1, 1, 2, 3, 4, 4, 7, 8])
    if kind == "decode":
        f32 = rng.random() < 0.15
        batch = rng.randint(1, 16)
        # a head's dots have to fit the chip's local memory
        budget = min(_log_int(rng, 100, 4096), 16000 // group)
        recent = rng.randint(8, 64)
        return _decode(None, batch, hkv * group, hkv, d, _log_int(rng, 2 * budget, 40 * budget),
                       budget, recent, sink=rng.choice([0, 0, 4]), dtype="f32" if f32 else "bf16",
                       value_prior=rng.random() < 0.15, static=batch * hkv <= 16 and budget < 2048)
    fixed = kind == "attend" or rng.random() < 0.3
    if kind == "accumulate":
        n = _log_int(rng, 700, 32768)
        while hkv * group > 32 or hkv * group * n * n > 32 * 32768 ** 2:
            hkv, group = max(1, hkv // 2), max(1, group // 2)
        budget, recent = max(64, n // rng.randint(4, 30)), rng.randint(8, 48)
        return _evict(None, 1, hkv * group, hkv, d, n, n, budget, recent, kind=kind,
                      fixed_scale=fixed, value_prior=rng.random() < 0.3,
                      layout=rng.choice(["bhnd", "bhnd", "bnhd"]))
    f32 = rng.random() < 0.15
    n = _log_int(rng, 256, 3000 if f32 else 65536)
    batch = rng.choice([1, 1, 1, 2, 3, 4, 8])
    while batch * hkv * n > 4 * 32 * 16384:   # no more tokens and heads than the largest layer
        batch, hkv = max(1, batch // 2), hkv // 2 if batch == 1 else hkv
    sink = rng.choice([0, 0, 4])
    recent = rng.randint(8, 64)
    budget = max(recent + sink + 16, int(n * rng.uniform(0.03, 0.3)))
    window = min(rng.choice([8, 16, 32, 32, 64, 64, 100, 128]), n // 3)
    return _evict(None, batch, hkv * group, hkv, d, n, window, budget, recent, kind=kind, sink=sink,
                  dtype="f32" if f32 else "bf16", layout=rng.choice(["bhnd", "bhnd", "bnhd"]),
                  fixed_scale=fixed, value_prior=rng.random() < 0.85)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _params(case, **more):
    scale = dict(scale_mode=B.AHA_SCALE_FIXED, fixed_scale=B.default_fixed_scale(case["d"])) \
        if case.get("fixed_scale") else {}
    return B.Params(batch=case["batch"], n_q_heads=case["hq"], n_kv_heads=case["hkv"],
                    head_dim=case["d"], budget=case["budget"], recent=case["recent"],
                    sink=case["sink"], dtype=B.AHA_F32 if case["dtype"] == "f32" else B.AHA_BF16,
                    **scale, **more)


def _heads(case, heads, gen):
    """A Gaussian [b, heads, n, d] tensor in the layout of the case."""
    b, n, d = case["batch"], case["n"], case["d"]
    if case["layout"] == "bnhd":
        return torch.randn((b, n, heads, d), generator=gen, device="cuda",
                           dtype=_dtype(case)).transpose(1, 2)
    return torch.randn((b, heads, n, d), generator=gen, device="cuda", dtype=_dtype(case))


def _prepare_prefill(case, gen):
    b, hq, hkv, n, d = case["batch"], case["hq"], case["hkv"], case["n"], case["d"]
    group, dt = hq // hkv, _dtype(case)
    q, k, v = (_heads(case, h, gen) for h in (hq, hkv, hkv))
    bias = torch.randn((b, hkv, 1, d), generator=gen, device="cuda").repeat_interleave(group, dim=1)
    q += (QUERY_BIAS * bias / bias.norm(dim=-1, keepdim=True)).to(dt)
    k[:, :, 0] *= SINK_KEY
    # heavy hitters: as many as are selected by score, anywhere that every observed row sees
    rows = min(case["window"], 256)
    mean = q[:, :, n - rows:].float().reshape(b, hkv, group * rows, d).mean(dim=2, keepdim=True)
    mean = HITTER_KEY * math.sqrt(d) * mean / mean.norm(dim=-1, keepdim=True)
    lo, hi = 1 + case["sink"], n - max(case["recent"], rows)
    count = min(case["budget"] - case["recent"] - case["sink"], hi - lo)
    where = lo + torch.rand((b, hkv, hi - lo), generator=gen, device="cuda").topk(count).indices
    where = where.unsqueeze(-1).expand(b, hkv, count, d)
    k.scatter_(2, where, (k.gather(2, where).float() + mean).to(dt))

    p = _params(case, seq_len=n, window=case["window"],
                value_prior=int(case["value_prior"])).with_strides(q, k, v)
    s = dict(kind=case["kind"], p=p, q=q, k=k, v=v, ws=B.alloc_workspace(p),
             scores=torch.empty((b, hkv, n), dtype=torch.float32, device="cuda"))
    if case["kind"] != "accumulate":
        s["idx"] = torch.empty((b, hkv, case["budget"]), dtype=torch.int32, device="cuda")
        s["cache"] = B.CompactCache.empty(p)
    if case["kind"] == "attend":
        s["out"] = torch.empty((b, hq, case["window"], d), dtype=dt, device="cuda")
        s["lse"] = torch.empty((b, hq, case["window"]), dtype=torch.float32, device="cuda")
        s["ws_attn"] = torch.empty(max(256, B.window_attention_workspace_bytes(p)),
                                   dtype=torch.uint8, device="cuda")
    return s


def _prepare_decode(case, gen):
    b, hq, hkv, n, d = case["batch"], case["hq"], case["hkv"], case["n"], case["d"]
    budget, recent, dt = case["budget"], case["recent"], _dtype(case)
    p = _params(case, seq_len=0, window=0, decode_value_prior=int(case["value_prior"]))
    c = B.CompactCache.empty(p)
    for t in (c.k, c.v):
        t.normal_(generator=gen)
    # what compaction leaves: ascending positions, the recent ones last, one free slot
    pos = torch.cat([torch.arange(budget - recent, device="cuda") * (n - recent) // (budget - recent),
                     torch.arange(n - recent, n, device="cuda"),
                     torch.full((1,), -1, device="cuda")])
    c.pos.copy_(pos.to(torch.int32).expand_as(c.pos))
    c.scores.normal_(generator=gen).mul_(0.5).exp_().mul_(0.05 * hq / hkv)
    c.scores[:, :, budget] = 0.0
    c.free_slot.fill_(budget)
    new = [torch.randn((TOKENS_AHEAD, b, h, d), generator=gen, device="cuda", dtype=dt)
           for h in (hq, hkv, hkv)]
    return dict(kind="decode", p=p, cache=c, new=list(zip(*(t.unbind(0) for t in new))), seen=n,
                out=torch.empty((b, hq, d), dtype=dt, device="cuda"),
                ws=None if case["static"] else
                torch.empty(max(256, B.workspace_bytes(p)), dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return _prepare_decode(case, gen) if case["kind"] == "decode" else _prepare_prefill(case, gen)


def run(state):
    p = state["p"]
    if state["kind"] == "decode":
        c, out = state["cache"], state["out"]
        state["seen"] += 1   # a generation loop: every step sees one token more
        q, k, v = state["new"][state["seen"] % TOKENS_AHEAD]
        if state["ws"] is None:
            B.aha_decode_step_static(p, q, k, v, c.k, c.v, c.scores, c.pos, c.free_slot,
                                     state["seen"], out)
        else:
            B.aha_decode_step(p, q, k, v, c.k, c.v, c.scores, c.pos, c.free_slot, state["seen"],
                              out, state["ws"])
        return dict(out=out, k=c.k, v=c.v, scores=c.scores, pos=c.pos, free_slot=c.free_slot)

    q, k, v, scores, ws = state["q"], state["k"], state["v"], state["scores"], state["ws"]
    if state["kind"] == "accumulate":
        B.aha_prefill_scores(p, q, k, v, scores, ws)
        return dict(scores=scores)
    results = dict(scores=scores, idx=state["idx"])
    if state["kind"] == "attend":
        B.aha_prefill_window_attention(p, q, k, v, state["out"], state["lse"], state["ws_attn"])
        B.aha_prefill_scores_lse(p, q, k, v, state["lse"], scores, ws)
        results.update(out=state["out"], lse=state["lse"])
    else:
        B.aha_prefill_scores(p, q, k, v, scores, ws)
    c, idx = state["cache"], state["idx"]
    B.aha_select_topk(p, scores, idx, ws)
    B.aha_compact_kv(p, k, v, scores, idx, c.k, c.v, c.scores, c.pos, c.free_slot)
    results.update(k_cache=c.k, v_cache=c.v, scores_c=c.scores, pos_c=c.pos, free_slot=c.free_slot)
    return results


def work(case):
    """Every input read once and every output written once; each product formed once."""
    b, hq, hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    e, slots = 4 if case["dtype"] == "f32" else 2, case["budget"] + 1
    if case["kind"] == "decode":
        heads = 2 * slots * d * e + 8 * slots + 8 * slots + 2 * d * e  # K, V; scores and positions in and out
        return {"bytes": b * hkv * heads + 2 * b * hq * d * e, "flops": 4.0 * b * hq * slots * d}
    n, r = case["n"], case["window"]
    pairs = r * n - r * (r - 1) // 2        # query rows times the keys they see
    values = case["value_prior"] or case["kind"] == "attend"
    nbytes = b * hkv * n * d * e * (2 if values else 1) + b * hq * r * d * e + b * hkv * n * 4
    flops = 2.0 * b * hq * d * pairs
    if case["kind"] == "attend":
        nbytes += b * hq * r * (d * e + 4)
        flops *= 2
    if case["kind"] != "accumulate":        # the compact cache, its scores, positions and indices
        nbytes += b * hkv * slots * (2 * d * e + 12)
        if not values:                      # retained value rows are read for the gather alone
            nbytes += b * hkv * slots * d * e
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the results differ by from the same path in 64 bits: scores, sums of fp32
    terms, by up to 2e-6 of their norm; attention outputs in bf16, rounded and weighted with
    rounded probabilities, by up to 2.3e-3 and 9e-3 at most."""
    if case["dtype"] == "bf16" and case["kind"] in ("attend", "decode"):
        return {"rel": 1e-2, "max": 0.05}
    return {"rel": 1e-5}

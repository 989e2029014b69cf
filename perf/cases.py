"""The calls a user of this library makes, as cases to time and to compare.

A case is a dict of plain values.  `stage` names what a pass does:

  encode   stage 1 over a whole pool (dbsa_preencode_attn)
  append   one new group joins an encoded pool: its keys and queries are rotated at their ids
           (dbsa_rope_apply) and its rows encoded (dbsa_preencode_attn on an append layout)
  prefill  stage 2, the prompts of a batch of questions (dbsa_query_attn or its _rope form)
  decode   stage 2, one generated token per question (dbsa_decode_attn, its _rope form or the fp8 pool)
  request  prefill and the decode step behind it
  whole    encode, prefill and one decode step, on a pool so small that launches are what it costs

Layouts, workspaces, output tensors and rotary tables are made in prepare(): a program keeps them for the 32
layers and all the generated tokens of a batch.  Tile heights follow the rule the benchmark uses: 64 tokens, 128
where every query head has its own KV head (encoding), 32 for questions shorter than 64 tokens.
Values: N(0, 1), keys scaled per channel by exp(0.5 z), demonstrations of random length, groups closed at the
demonstration boundary next to equal shares: the same distributions as the synthetic inputs of the benchmark.
"""
import json
import math
import random

import numpy as np
import torch

from paper_2503_08640_amd import binding as B

ROPE_BASE = 500000.0


def listed():
    gqa = {"heads": 32, "kv_heads": 8, "dim": 128, "dtype": "bf16", "sink": 64, "window": 0}
    mha = dict(gqa, kv_heads=32)
    pool90 = {"pool": 90112, "groups": 22, "demo_lo": 32, "demo_hi": 256}
    pool30 = {"pool": 32768, "groups": 8, "demo_lo": 32, "demo_hi": 128}
    ask = {"rope": False, "fp8": False, "ragged": False}
    return [
        # set-up of a 90k-token pool for a grouped-query model: the largest call
        dict(gqa, name="encode_gqa_90k", stage="encode", **pool90),
        # set-up of a 30k-token pool for a multi-head model
        dict(mha, name="encode_mha_30k", stage="encode", **pool30),
        # a block of 50 demonstrations joins a pool kept the way the paper keeps it: first block = sink, two
        # preceding blocks visible, keys rotated at their encoding ids
        dict(gqa, name="append_block", stage="append", sink=1923, window=2, pool=88000, groups=47, demo_lo=28, demo_hi=47),
        # 16 questions of 64 tokens, 30 % of the pool each: the ordinary batch
        dict(gqa, name="prefill_b16", stage="prefill", queries=16, q_len=64, ratio=0.3, **pool90, **ask),
        # one question at a time, as the paper times its pipeline, over re-positioned caches
        dict(gqa, name="prefill_b1_rope", stage="prefill", queries=1, q_len=64, ratio=0.3, **pool90, **dict(ask, rope=True)),
        # the ordinary batch on the multi-head model
        dict(mha, name="prefill_mha_b16", stage="prefill", queries=16, q_len=64, ratio=0.3, **pool30, **ask),
        # one generated token for each of the 16 questions
        dict(gqa, name="decode_b16", stage="decode", queries=16, q_len=64, ratio=0.3, **pool90, **ask),
        # one generated token for a single question over re-positioned caches
        dict(gqa, name="decode_b1_rope", stage="decode", queries=1, q_len=64, ratio=0.3, **pool90, **dict(ask, rope=True)),
        # a large batch of short questions generates
        dict(gqa, name="decode_b128", stage="decode", queries=128, q_len=32, ratio=0.3, **pool90, **ask),
        # the ordinary batch generates over a pool stored as 8-bit floats
        dict(gqa, name="decode_fp8_b16", stage="decode", queries=16, q_len=64, ratio=0.3, **pool90, **dict(ask, fp8=True)),
        # a small model (head_dim 64) answers a few questions of different lengths: prompts, then a token
        dict(gqa, name="request_d64", stage="request", dim=64, queries=5, q_len=150, ratio=0.3, **pool30, **dict(ask, ragged=True)),
        # everything in fp32 on a pool of 8 demonstrations: what calls and launches cost
        dict(name="whole_fp32_tiny", stage="whole", heads=2, kv_heads=2, dim=64, dtype="f32", sink=4, window=0, pool=256,
             groups=2, demo_lo=32, demo_hi=32, queries=1, q_len=16, ratio=0.5, **ask),
    ]


def draw(rng):
    while True:  # none larger than the largest listed one
        c = _draw(rng)
        if work(c)["flops"] < 3e12:
            return c


def _draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    stage = rng.choice(["encode", "encode", "append", "prefill", "prefill", "prefill", "decode", "decode", "decode", "request",
                        "whole"])
    if stage == "whole":
        pool = log_int(256, 2048)
        return {"stage": stage, "heads": 4, "kv_heads": rng.choice([1, 2, 4]), "dim": rng.choice([64, 128]), "dtype": "f32",
                "sink": rng.randint(1, 64), "window": rng.choice([0, 1]), "pool": pool, "groups": max(2, pool // 256),
                "demo_lo": 16, "demo_hi": 48, "queries": rng.randint(1, 4), "q_len": rng.randint(2, 40), "ratio": 0.5,
                "rope": False, "fp8": False, "ragged": rng.random() < 0.5}
    heads, kv_heads, dim = rng.choice([(32, 8, 128)] * 5 + [(32, 32, 128)] * 2 +
                                      [(32, 4, 128), (24, 8, 128), (40, 8, 128), (32, 8, 64), (16, 16, 64)])
    # the shapes of the two large pools, and smaller ones; multi-head and off-size models keep to the smaller
    top = 90112 if (heads, kv_heads, dim) == (32, 8, 128) else 32768
    pool = log_int(4096, top)
    group = log_int(700, 4800)
    c = {"stage": stage, "heads": heads, "kv_heads": kv_heads, "dim": dim, "dtype": "bf16", "sink": rng.choice([4, 64, 64, 333, 1000]),
         "window": rng.choice([0, 0, 2]) if stage in ("encode", "append") else 0, "pool": pool,
         "groups": max(2, pool // group), "demo_lo": rng.choice([28, 32]), "demo_hi": rng.choice([47, 128, 256])}
    if stage in ("encode", "append"):
        return c
    q = log_int(1, 128)
    rope = dim == 128 and 32 % (heads // kv_heads) == 0 and rng.random() < 0.3
    c.update(queries=q, q_len=log_int(8, 512 if q <= 16 else 64), ratio=rng.choice([0.1, 0.3, 0.3, 0.5, 1.0]), rope=rope,
             fp8=stage == "decode" and dim == 128 and 32 % (heads // kv_heads) == 0 and rng.random() < 0.25,
             ragged=rng.random() < 0.5)
    return c


# ---------------------------------------------------------------------------------------------------------------
# pool structure and selections
# ---------------------------------------------------------------------------------------------------------------


def _structure(case, seed):
    """Token offsets of the demonstrations, demonstration index of each group's start; with questions, their packed
    offsets, their own keys so far (prompt and generated tokens) and the groups each one selected.  Lengths belong
    to the case, selections and generated tokens to the seed."""
    rnd = random.Random(json.dumps({x: case[x] for x in sorted(case) if x != "name"}))
    lens, total, lo, hi = [], 0, case["demo_lo"], case["demo_hi"]
    while total < case["pool"]:
        lens.append(rnd.randint(lo, hi))
        total += lens[-1]
    lens[-1] -= total - case["pool"]
    if lens[-1] < lo and len(lens) > 1:
        tail = lens.pop()
        lens[-1] += tail
    demos = case["sink"] + np.concatenate([[0], np.cumsum(lens)])
    starts = [0]
    for g in range(1, case["groups"]):
        want = case["sink"] + g * case["pool"] / case["groups"]
        starts.append(max(starts[-1] + 1, int(np.argmin(np.abs(demos - want)))))
    starts.append(len(lens))
    s = {"demos": demos.astype(np.int32), "starts": np.asarray(starts, np.int32), "n": int(demos[-1])}
    s["bounds"] = [int(x) for x in s["demos"][s["starts"]]]
    if "queries" in case:
        top = case["q_len"]
        q_lens = [rnd.randint(max(1, top // 2), top) if case["ragged"] else top for _ in range(case["queries"])]
        m = max(1, int(math.floor(case["ratio"] * case["groups"] + 0.5)))
        s["cu"] = np.concatenate([[0], np.cumsum(q_lens)]).astype(np.int32)
        rnd = random.Random(1000003 * seed + 17)
        s["own"] = [t + (1 if case["stage"] != "decode" else rnd.randint(1, 32)) for t in q_lens]
        s["sel"] = [sorted(rnd.sample(range(case["groups"]), m)) for _ in q_lens]
    return s


def _freqs(dim):
    return ROPE_BASE ** (-np.arange(0, dim, 2, dtype=np.float64) / dim)


def _inputs(case, seed):
    """Structure and device tensors, from the seed alone."""
    s = _structure(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed + 7)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    hq, hkv, d, n = case["heads"], case["kv_heads"], case["dim"], s["n"]

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)

    spread = torch.exp(0.5 * torch.randn((1, hkv, d), generator=gen, device="cuda"))

    def keys(rows):
        return (torch.randn((rows, hkv, d), generator=gen, device="cuda") * spread).to(dtype)

    t = {"k": keys(n), "v": normal(n, hkv, d)}
    if case["stage"] in ("encode", "whole"):
        t["q"] = normal(n, hq, d)
    if case["stage"] == "append":
        first = s["bounds"][-2]
        t.update(q_new=normal(n - first, hq, d), k_new=keys(n - first))
    if "queries" in case:
        b, tot, room = case["queries"], int(s["cu"][-1]), case["q_len"] + 33
        if case["stage"] != "decode":
            t.update(q_self=normal(tot, hq, d), k_self=keys(tot), v_self=normal(tot, hkv, d))
        if case["stage"] != "prefill":
            t.update(q_step=normal(b, hq, d), k_cache=keys(b * room).view(b, room, hkv, d),
                     v_cache=normal(b * room, hkv, d).view(b, room, hkv, d))
    if case.get("fp8"):  # one scale per KV head, largest value to the top of the format
        for name in ("k", "v"):
            x = t.pop(name).float()
            scale = (x.abs().amax(dim=(0, 2)) / 448.0).clamp_min(1e-12)
            t[name + "8"] = (x / scale[None, :, None]).to(torch.float8_e4m3fn)
            t[name + "_scale"] = scale.contiguous()
    return s, t


def prepare(case, seed):
    s, t = _inputs(case, seed)
    state = dict(t, case=case, scale=1.0 / math.sqrt(case["dim"]))
    pool = (case["sink"], s["demos"], s["starts"])
    tile = 128 if case["heads"] == case["kv_heads"] else B.BENCH_BLOCK_M_PREENCODE
    if case["stage"] in ("encode", "whole"):
        state["layout"] = B.dbsa_layout_build(*pool, case["window"], block_m=tile, block_n=64)
        state["o"] = torch.empty_like(t["q"])
    if case["stage"] == "append":
        first = s["bounds"][-2]
        state["layout"] = B.dbsa_layout_build_append(*pool, case["window"], case["groups"] - 1, block_m=tile, block_n=64)
        state["q"] = torch.zeros((s["n"], case["heads"], case["dim"]), device="cuda", dtype=t["q_new"].dtype)
        state["o"] = torch.empty_like(state["q"])
        state["table"] = B.dbsa_rope_table(_freqs(case["dim"]), s["n"])
        state["first"] = first
    if "queries" in case:
        short = case["q_len"] < 64
        state["asked"] = B.dbsa_layout_build(
            *pool, 0, cu_qlens=s["cu"], sel_ptr=np.cumsum([0] + [len(x) for x in s["sel"]]),
            sel_idx=[g for x in s["sel"] for g in x], n_split=0, block_n=64,
            block_m=B.BENCH_BLOCK_M_SHORT_QUERY if short else B.BENCH_BLOCK_M_QUERY)
        need = state["asked"].workspace_bytes(case["heads"], case["dim"])
        state["workspace"] = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
        state["self_len"] = torch.tensor(s["own"], dtype=torch.int32, device="cuda")
        if case["rope"]:
            state["table"] = B.dbsa_rope_table(_freqs(case["dim"]), 2 * s["n"] + case["q_len"] + 40)
        for name in ("q_self", "q_step"):
            if name in t:
                state["o" + name[1:]] = torch.empty_like(t[name])
    return state


def _prefill(s):
    if s["case"]["rope"]:
        return B.dbsa_query_attn_rope(s["asked"], s["q_self"], s["k_self"], s["v_self"], s["k"], s["v"], s["table"],
                                      s["scale"], out=s["o_self"], workspace=s["workspace"])
    return B.dbsa_query_attn(s["asked"], s["q_self"], s["k_self"], s["v_self"], s["k"], s["v"], s["scale"], out=s["o_self"],
                             workspace=s["workspace"])


def _decode(s):
    own = (s["asked"], s["q_step"], s["k_cache"], s["v_cache"], s["self_len"])
    if s["case"]["fp8"]:
        return B.dbsa_decode_attn_kv8(*own, s["k8"], s["v8"], s["k_scale"], s["v_scale"], s["scale"], out=s["o_step"],
                                      workspace=s["workspace"], rope_table=s.get("table"))
    if s["case"]["rope"]:
        return B.dbsa_decode_attn_rope(*own, s["k"], s["v"], s["table"], s["scale"], out=s["o_step"], workspace=s["workspace"])
    return B.dbsa_decode_attn(*own, s["k"], s["v"], s["scale"], out=s["o_step"], workspace=s["workspace"])


def run(state):
    s, stage = state, state["case"]["stage"]
    if stage == "encode":
        return {"o": B.dbsa_preencode_attn(s["layout"], s["q"], s["k"], s["v"], s["scale"], out=s["o"])}
    if stage == "append":
        new = slice(s["first"], None)
        k = B.dbsa_rope_apply(s["k_new"], s["table"], first_id=s["first"], out=s["k"][new])
        q = B.dbsa_rope_apply(s["q_new"], s["table"], first_id=s["first"], out=s["q"][new])
        o = B.dbsa_preencode_attn(s["layout"], s["q"], s["k"], s["v"], s["scale"], out=s["o"])
        return {"k": k, "q": q, "o": o[new]}
    if stage == "prefill":
        return {"o": _prefill(s)}
    if stage == "decode":
        return {"o": _decode(s)}
    if stage == "request":
        return {"o": _prefill(s), "step": _decode(s)}
    o = B.dbsa_preencode_attn(s["layout"], s["q"], s["k"], s["v"], s["scale"], out=s["o"])
    return {"pool": o, "o": _prefill(s), "step": _decode(s)}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------


def work(case):
    s = _structure(case, 1)
    hq, hkv, d, es, stage = case["heads"], case["kv_heads"], case["dim"], 4 if case["dtype"] == "f32" else 2, case["stage"]
    row_q, row_kv = hq * d * es, hkv * d * es
    pairs = moved = 0.0
    b, sink = s["bounds"], case["sink"]
    spans = list(zip(b[:-1], b[1:]))
    if stage in ("encode", "append", "whole"):
        todo = range(len(spans)) if stage != "append" else [len(spans) - 1]
        for g in todo:
            n = spans[g][1] - spans[g][0]
            before = sum(y - x for x, y in spans[max(0, g - case["window"]):g])
            pairs += n * (sink + before) + n * (n + 1) // 2
        if stage == "append":  # new rows: q, k read and written rotated; o written; the window, the sink and v read
            g = len(spans) - 1
            n = spans[g][1] - spans[g][0]
            seen = sink + sum(y - x for x, y in spans[max(0, g - case["window"]):g])
            moved += 3 * n * row_q + 3 * n * row_kv + 2 * seen * row_kv + n * d * 4
        else:
            pairs += sink * (sink + 1) // 2
            moved += 2 * s["n"] * row_q + 2 * s["n"] * row_kv
    if "queries" in case:
        lens = [spans[g][1] - spans[g][0] for g in range(len(spans))]
        union = sink + sum(lens[g] for g in set(g for x in s["sel"] for g in x))
        row_pool = hkv * d * (1 if case["fp8"] else es)
        prompts = [int(y - x) for x, y in zip(s["cu"][:-1], s["cu"][1:])]
        if stage != "whole":
            moved += 2 * union * row_pool
        for t, own, sel in zip(prompts, s["own"], s["sel"]):
            seen = sink + sum(lens[g] for g in sel)
            if stage != "decode":
                pairs += t * seen + t * (t + 1) // 2
                moved += 2 * t * row_q + 2 * t * row_kv
            if stage != "prefill":
                pairs += seen + own
                moved += 2 * row_q + 2 * own * row_kv
    return {"bytes": float(moved), "flops": 4.0 * d * hq * pairs}


def tolerance(case):
    # bf16: inputs and outputs rounded to 8 bits, probabilities rounded once before they weigh the values, the
    # scaled query once more.  fp32: sums of up to a few thousand terms in another order.
    return {"rel": 5e-6} if case["dtype"] == "f32" else {"rel": 1.2e-2}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits, from the definition
# ---------------------------------------------------------------------------------------------------------------


def _rotate(x, ids):
    """x [T, H, D] at position ids (a number or [T]); channel i pairs with channel i + D/2."""
    d = x.shape[2]
    ids = torch.as_tensor(ids, dtype=torch.float64, device=x.device).reshape(-1, 1, 1)
    angle = ids * torch.as_tensor(_freqs(d), device=x.device)[None, None, :]
    c, s = torch.cos(angle), torch.sin(angle)
    lo, hi = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)


def _attend(q, k, v, scale, mask=None):
    """q [T, Hq, D] over k, v [N, Hkv, D]; mask [T, N] of visible pairs."""
    t, hq, d = q.shape
    r = hq // k.shape[1]
    out = torch.empty_like(q)
    for h in range(k.shape[1]):
        rows = q[:, h * r:(h + 1) * r].permute(1, 0, 2).reshape(r * t, d)
        w = scale * (rows @ k[:, h].t().contiguous())
        if mask is not None:
            w = w.view(r, t, -1).masked_fill(~mask, -math.inf).view(r * t, -1)
        out[:, h * r:(h + 1) * r] = (torch.softmax(w, 1) @ v[:, h].contiguous()).view(r, t, d).permute(1, 0, 2)
    return out


def _encode(case, s, q, k, v, groups):
    """{group: rows} of the groups asked for, and the sink's rows under -1."""
    sink, b, scale, got = case["sink"], s["bounds"], 1.0 / math.sqrt(case["dim"]), {}
    for g in groups:
        lo, hi = (b[g], b[g + 1]) if g >= 0 else (0, sink)
        back = b[max(0, g - case["window"])] if g >= 0 else 0
        seen = torch.cat([torch.arange(sink if g >= 0 else 0), torch.arange(back, hi)]).cuda()
        mask = seen[None, :] <= torch.arange(lo, hi, device="cuda")[:, None]
        got[g] = _attend(q[lo:hi].double(), k[seen].double(), v[seen].double(), scale, mask)
    return got


def exact(case, seed):
    s, t = _inputs(case, seed)
    stage, b, scale = case["stage"], s["bounds"], 1.0 / math.sqrt(case["dim"])
    out = {}
    if stage in ("encode", "whole"):
        rows = _encode(case, s, t["q"], t["k"], t["v"], range(-1, case["groups"]))
        out["o" if stage == "encode" else "pool"] = torch.cat([rows[g] for g in range(-1, case["groups"])])
    if stage == "append":
        g = case["groups"] - 1
        ids = torch.arange(b[g], b[g + 1], device="cuda")
        q_new, k_new = _rotate(t["q_new"].double(), ids), _rotate(t["k_new"].double(), ids)
        sink, back = case["sink"], b[max(0, g - case["window"])]
        seen = torch.cat([torch.arange(sink), torch.arange(back, b[g])]).cuda()
        mask = torch.cat([torch.ones((len(ids), len(seen)), dtype=torch.bool, device="cuda"), ids[None, :] <= ids[:, None]], 1)
        o = _attend(q_new, torch.cat([t["k"][seen].double(), k_new]),
                    torch.cat([t["v"][seen].double(), t["v"][b[g]:].double()]), scale, mask)
        out = {"k": k_new, "q": q_new, "o": o}
    if "queries" in case:
        if case["fp8"]:
            k, v = (t[x + "8"].float().double() * t[x + "_scale"].double()[None, :, None] for x in ("k", "v"))
        else:
            k, v = t["k"], t["v"]
        prompts, steps = [], []
        for u, sel in enumerate(s["sel"]):
            lo, hi, own = int(s["cu"][u]), int(s["cu"][u + 1]), s["own"][u]
            ids = torch.cat([torch.arange(case["sink"])] + [torch.arange(b[g], b[g + 1]) for g in sel]).cuda()
            ku, vu, n = k[ids].double(), v[ids].double(), len(ids)
            if case["rope"]:  # kept with the rotation of its token id, wanted at its place in the concatenation
                ku = _rotate(ku, torch.arange(n, device="cuda") - ids)

            def at(x, first, on=case["rope"]):
                return _rotate(x, first) if on else x

            if stage != "decode":
                a = torch.arange(hi - lo, device="cuda")
                mask = torch.cat([torch.ones((hi - lo, n), dtype=torch.bool, device="cuda"), a[None, :] <= a[:, None]], 1)
                prompts.append(_attend(at(t["q_self"][lo:hi].double(), n + a), torch.cat([ku, at(t["k_self"][lo:hi].double(), n)]),
                                       torch.cat([vu, t["v_self"][lo:hi].double()]), scale, mask))
            if stage != "prefill":
                steps.append(_attend(at(t["q_step"][u:u + 1].double(), n + own - 1),
                                     torch.cat([ku, at(t["k_cache"][u, :own].double(), n)]),
                                     torch.cat([vu, t["v_cache"][u, :own].double()]), scale))
        if prompts:
            out["o"] = torch.cat(prompts)
        if steps:
            out["o" if stage == "decode" else "step"] = torch.cat(steps)
    return out

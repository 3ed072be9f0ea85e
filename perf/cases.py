"""Performance cases of the multi-token paged attention library.

A case is one call sequence of a serving program on one batch:

* ``step``     one transformer layer over a batch whose plan is in hand: KV append (or rotary
               embedding fused with the append), then multi-token paged attention;
* ``one_shot`` the same layer through the forms that take the length arrays and build the plan
               inside the call;
* ``swap``     pages copied out to a staging buffer and pages copied back in (tier swapping).

The lengths of a batch come from the case alone (``lens_seed``), the values and the placement of the
pages from the seed that is handed to ``prepare``.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2312_05516_amd import binding as pv
from paper_2312_05516_amd import workloads as wl

PAGE = wl.PAGE_SIZE


def _batch(name, heads, dtype, requests, ctx, new, *, turns, ctx_kind="uniform", rope="",
           kind="step", lens_seed=1):
    """One case.  heads = (query heads, KV heads, head size); ctx = (lowest, highest) cached tokens of
    a request (kind "lognormal": median 1000, clipped to that range); `turns` = share of the requests
    that bring a new prompt of new = (lowest, highest) tokens, the others generate one token."""
    return {"name": name, "kind": kind, "dtype": dtype, "q_heads": heads[0], "kv_heads": heads[1],
            "head_dim": heads[2], "requests": requests, "ctx_lo": ctx[0], "ctx_hi": ctx[1],
            "ctx_kind": ctx_kind, "new_lo": new[0], "new_hi": new[1], "turns": turns, "rope": rope,
            "lens_seed": lens_seed}


def _swap(name, heads, dtype, pages, lens_seed=1):
    return {"name": name, "kind": "swap", "dtype": dtype, "kv_heads": heads[1],
            "head_dim": heads[2], "pages": pages, "lens_seed": lens_seed}


MHA = (40, 40, 128)    # 13B-shaped layer
GQA = (64, 8, 128)     # 70B-shaped layer
GQA_D64 = (32, 8, 64)  # the other head size the library has
SMALL = (4, 4, 64)     # the tiny configuration


def listed():
    return [
        # two short chats answered together, the smallest call there is: launches and host time
        _batch("tiny_turns", SMALL, "f16", 2, (37, 100), (5, 12), turns=1.0),
        # a few interactive users, each generating a token over a chat of some length
        _batch("decode_few", GQA, "bf16", 4, (700, 9000), (1, 1), turns=0.0, rope="half"),
        # one of them sends a follow-up question through the calls that need no plan
        _batch("one_shot_turn", GQA, "bf16", 3, (300, 3000), (24, 150), turns=0.4, kind="one_shot"),
        # an ordinary generation batch of a grouped-query model
        _batch("decode_gqa", GQA, "bf16", 96, (16, 8192), (1, 1), turns=0.0,
               ctx_kind="lognormal"),
        # the largest generation batch: 256 requests, 40 heads each (12 GB of K/V read)
        _batch("decode_heavy", MHA, "f16", 256, (512, 4096), (1, 1), turns=0.0),
        # 8 query tokens a request over 2048 cached ones (the shape of the paper's kernel figure)
        _batch("few_tokens", MHA, "f16", 32, (2048, 2048), (8, 8), turns=1.0),
        # new turns and generation steps in one batch, every query head with its own KV head
        _batch("mixed_mha", MHA, "f16", 32, (200, 1800), (20, 300), turns=0.5),
        # the same with grouped-query heads, skewed history lengths
        _batch("mixed_gqa", GQA, "bf16", 64, (16, 4096), (16, 512), turns=0.3,
               ctx_kind="lognormal"),
        # the same with head size 64
        _batch("mixed_d64", GQA_D64, "bf16", 48, (100, 3000), (16, 400), turns=0.4),
        # first turns: prompts without any history, rotary embedding in front
        _batch("first_turns", MHA, "f16", 8, (0, 0), (150, 1500), turns=1.0, rope="interleaved"),
        # prompts over long histories, bound by the matrix cores: the largest amount of arithmetic
        _batch("long_history", GQA, "bf16", 8, (16384, 32768), (512, 512), turns=1.0),
        # 16 K tokens swapped out and as many swapped in, in chunks of two pages
        _swap("swap_pages", MHA, "f16", 1024),
    ]


# A drawn case stays below these (what the largest listed cases read and compute)
_MOST_BYTES = 11e9
_MOST_FLOPS = 2.8e12


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    lens_seed = rng.randrange(1 << 20)
    dtype = rng.choice(["f16", "bf16"])
    # whole layers, and the head groups that are left of them when a layer is cut over several GPUs
    heads = rng.choice([MHA, MHA, GQA, GQA, (40, 10, 128), (16, 2, 128), (10, 10, 128), GQA_D64,
                        (12, 12, 64)])
    kind = rng.choice(["decode", "decode", "few_tokens", "mixed", "mixed", "mixed", "first",
                       "long", "one_shot", "swap"])
    if kind == "swap":
        case = _swap("", heads, dtype, 2 * log_int(16, 1024), lens_seed)
        del case["name"]
        return case
    rope = rng.choice(["", "", "half", "interleaved"]) if kind != "one_shot" else ""
    while True:
        ctx_kind = "uniform"
        turns = 1.0
        requests = log_int(1, 256)
        if kind == "decode":
            new, turns = (1, 1), 0.0
            lo = log_int(16, 4000)
            ctx = (lo, lo + log_int(16, 8000))
            ctx_kind = rng.choice(["uniform", "lognormal"])
        elif kind == "few_tokens":
            n = rng.randint(2, 16)
            new = (n, n)
            lo = log_int(64, 8000)
            ctx = (lo, lo + rng.randint(0, 500))
        elif kind in ("mixed", "one_shot"):
            if kind == "one_shot":
                requests = log_int(1, 32)
            turns = rng.uniform(0.1, 1.0)
            lo = log_int(16, 200)
            new = (lo, lo + log_int(16, 600))
            ctx = (log_int(16, 1000), 0)
            ctx = (ctx[0], ctx[0] + log_int(100, 4000))
            ctx_kind = rng.choice(["uniform", "lognormal"])
        elif kind == "first":
            requests = log_int(1, 32)
            lo = log_int(16, 500)
            new = (lo, lo + log_int(16, 1500))
            ctx = (0, 0)
        else:  # long
            requests = log_int(1, 16)
            n = log_int(16, 700)
            new = (n, n + rng.randint(0, 60))
            lo = log_int(4000, 24000)
            ctx = (lo, lo + rng.randint(0, 8000))
        case = _batch("", heads, dtype, requests, ctx, new, turns=round(turns, 3),
                      ctx_kind=ctx_kind, rope=rope, lens_seed=lens_seed,
                      kind="one_shot" if kind == "one_shot" else "step")
        del case["name"]
        w = work(case)
        if w["bytes"] <= _MOST_BYTES and w["flops"] <= _MOST_FLOPS and (
                w["bytes"] / _MOST_BYTES + w["flops"] / _MOST_FLOPS <= 1.0):
            return case


def _lengths(case):
    """(cached tokens, new tokens) of every request."""
    rng = np.random.default_rng(case["lens_seed"])
    n = case["requests"]
    if case["ctx_kind"] == "lognormal":
        ctx = np.clip(np.rint(np.exp(rng.normal(np.log(1000.0), 1.0, size=n))), case["ctx_lo"],
                      case["ctx_hi"]).astype(np.int64)
    else:
        ctx = rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=n)
    turn = np.zeros(n, dtype=bool)
    if case["turns"] > 0:
        turn[rng.permutation(n)[:max(1, round(case["turns"] * n))]] = True
    new = np.where(turn, rng.integers(case["new_lo"], case["new_hi"] + 1, size=n), 1)
    return ctx, new


def _values(shape, dtype, gen):
    """N(0, 1) in the 16-bit type, as in the configurations."""
    td = torch.float16 if dtype == "f16" else torch.bfloat16
    return torch.empty(shape, dtype=td, device="cuda").normal_(generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype, hkv, d = case["dtype"], case["kv_heads"], case["head_dim"]
    if case["kind"] == "swap":
        n = case["pages"]
        num_pages = 3 * n
        rng = np.random.default_rng(seed)
        chunks = rng.permutation(num_pages // 2)[:n]  # chunks of two pages, out then in
        ids = np.stack([2 * chunks, 2 * chunks + 1], axis=1).ravel().astype(np.int32)
        pool = (num_pages, hkv * PAGE * d)
        return {"kind": "swap", "desc": pv.pool_desc(num_pages, hkv, d, dtype), "n": n,
                "k": _values(pool, dtype, gen), "v": _values(pool, dtype, gen),
                "out_ids": torch.from_numpy(ids[:n]).cuda(),
                "in_ids": torch.from_numpy(ids[n:]).cuda(),
                "out_stage": torch.empty((n, 2, hkv * PAGE * d), device="cuda",
                                         dtype=torch.float16 if dtype == "f16" else torch.bfloat16),
                "in_stage": _values((n, 2, hkv * PAGE * d), dtype, gen)}
    ctx, new = _lengths(case)
    b = wl.custom(ctx, new, num_q_heads=case["q_heads"], num_kv_heads=hkv, head_dim=d,
                  dtype=dtype, seed=seed)
    pool = (b.num_pages, hkv * PAGE * d)
    st = {"kind": case["kind"], "b": b, "desc": pv.pool_desc(b.num_pages, hkv, d, dtype),
          "k": _values(pool, dtype, gen), "v": _values(pool, dtype, gen),
          "q": _values((b.total_q, b.num_q_heads, d), dtype, gen),
          "k_new": _values((b.total_q, hkv, d), dtype, gen),
          "v_new": _values((b.total_q, hkv, d), dtype, gen),
          "table": torch.from_numpy(b.page_table).cuda()}
    st["out"] = torch.empty_like(st["q"])
    if case["kind"] == "one_shot":
        ws = pv.attn_workspace_bytes(st["desc"], b.num_q_heads, b.num_reqs, b.total_q,
                                     int(b.kv_lens.max()))
    else:
        st["plan"] = pv.plan_create(st["desc"], b.num_q_heads, b.ctx_lens, b.q_lens,
                                    b.max_pages_per_req)
        pv.plan_upload(st["plan"])
        ws = pv.plan_workspace_bytes(st["plan"])
        if case["rope"]:
            st["rope"] = case["rope"]
            st["cos_sin"] = torch.from_numpy(
                pv.rope_table(10000.0, d, int(b.kv_lens.max()))).cuda()
            st["q_rot"] = torch.empty_like(st["q"])
    st["ws"] = torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    k, v = st["k"], st["v"]
    if st["kind"] == "swap":
        pv.pages_gather(st["desc"], k, v, st["out_ids"], st["n"], st["out_stage"])
        pv.pages_scatter(st["desc"], st["in_stage"], st["in_ids"], st["n"], k, v)
        return {"stage": st["out_stage"], "k": k, "v": v}
    b = st["b"]
    if st["kind"] == "one_shot":
        pv.kv_append(st["desc"], st["k_new"], st["v_new"], st["table"], b.max_pages_per_req,
                     b.ctx_lens, b.q_lens, b.q_start, k, v)
        pv.multi_token_paged_attn(st["desc"], b.num_q_heads, st["q"], k, v, st["table"],
                                  b.max_pages_per_req, b.ctx_lens, b.q_lens, b.q_start, b.scale,
                                  st["out"], st["ws"])
        return {"out": st["out"], "k": k, "v": v}
    q = st["q"]
    if "rope" in st:
        q = st["q_rot"]
        pv.rope_kv_append_planned(st["plan"], st["q"], q, st["k_new"], st["v_new"],
                                  st["cos_sin"], st["rope"], st["table"], k, v)
    else:
        pv.kv_append_planned(st["plan"], st["k_new"], st["v_new"], st["table"], k, v)
    pv.multi_token_paged_attn_planned(st["plan"], q, k, v, st["table"], b.scale, st["out"],
                                      st["ws"])
    return {"out": st["out"], "k": k, "v": v}


def work(case):
    hkv, d = case["kv_heads"], case["head_dim"]
    if case["kind"] == "swap":  # out and in: each page read once and written once
        return {"bytes": 4 * case["pages"] * 2 * hkv * PAGE * d * 2, "flops": 0}
    ctx, new = (x.astype(np.int64) for x in _lengths(case))
    hq, total = case["q_heads"], int(new.sum())
    kv = ctx + new
    nbytes = 2 * int(ctx.sum()) * hkv * d * 2       # cached K and V, read once
    nbytes += 2 * 2 * total * hkv * d * 2           # new K and V: read, and stored in the pool
    nbytes += 2 * total * hq * d * 2                # queries in, result out
    nbytes += 4 * int(((kv + PAGE - 1) // PAGE).sum())
    if case["rope"]:
        nbytes += 2 * total * d                     # the angles of these positions
    pairs = int((new * ctx + new * (new + 1) // 2).sum())
    return {"bytes": nbytes, "flops": 4 * d * hq * pairs}


def tolerance(case):
    # Probabilities and results are rounded to the 16-bit type once each, and scaled queries may be.
    # Against the same attention in 64 bits the results are off by 2.5e-4 to 2.9e-4 (f16) and 2.0e-3
    # to 2.9e-3 (bf16) on the listed cases.
    if case["kind"] == "swap":
        return "exact"
    return {"rel": 1.2e-3 if case["dtype"] == "f16" else 1e-2}

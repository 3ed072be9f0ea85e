"""Distance of the attention results from attention in 64 bits, over lists that the plan cuts in
different ways."""
import math

import numpy as np
import pytest

from paper_2312_05516_amd import workloads as wl

pytestmark = pytest.mark.gpu

MHA, GQA, GQA_D64, PART = (40, 40, 128), (64, 8, 128), (32, 8, 64), (12, 12, 64)


def _state(ctx, new, heads, dtype, seed):
    """Batch with N(0, 1) values in the pool and the queries (the new rows are in the pool too)."""
    import torch
    b = wl.custom(ctx, new, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2],
                  dtype=dtype, seed=seed)
    td = torch.float16 if dtype == "f16" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def draw(*shape):
        return torch.empty(shape, dtype=td, device="cuda").normal_(generator=gen)
    pool = (b.num_pages, b.num_kv_heads * 16 * b.head_dim)
    return b, draw(b.total_q, b.num_q_heads, b.head_dim), draw(*pool), draw(*pool)


def _run(b, q, k, v, scale=None):
    import torch
    from paper_2312_05516_amd import binding as pv
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    ws = torch.empty(max(pv.plan_workspace_bytes(plan), 256), dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    pv.multi_token_paged_attn_planned(plan, q, k, v, torch.from_numpy(b.page_table).cuda(),
                                      b.scale if scale is None else scale, out, ws)
    torch.cuda.synchronize()
    items = [pv.plan_num_work_items(plan, kind) for kind in (0, 1)]
    plan.destroy()
    return out, items


def _in_64_bits(b, q, k, v, scale=None):
    import torch
    hkv, d, g = b.num_kv_heads, b.head_dim, b.num_q_heads // b.num_kv_heads
    kv_, vv = k.view(b.num_pages, hkv, d // 8, 16, 8), v.view(b.num_pages, hkv, 2, d, 8)
    want = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for r in range(b.num_reqs):
        c, n, s0 = int(b.ctx_lens[r]), int(b.q_lens[r]), int(b.q_start[r])
        kv = c + n
        pages = torch.from_numpy(b.page_table[r, :(kv + 15) // 16].astype(np.int64)).cuda()
        kk = kv_[pages].permute(1, 0, 3, 2, 4).reshape(hkv, -1, d)[:, :kv].double()
        vd = vv[pages].permute(1, 0, 2, 4, 3).reshape(hkv, -1, d)[:, :kv].double()
        qq = q[s0:s0 + n].double().view(n, hkv, g, d).permute(1, 2, 0, 3).reshape(hkv, g * n, d)
        hidden = (torch.arange(kv, device="cuda")[None, :] >
                  (c + torch.arange(n, device="cuda"))[:, None]).repeat(g, 1)
        s = torch.bmm(qq.contiguous(), kk.transpose(1, 2).contiguous())
        s *= b.scale if scale is None else scale
        o = torch.bmm(torch.softmax(s.masked_fill_(hidden[None], -math.inf), -1), vd.contiguous())
        want[s0:s0 + n] = o.view(hkv, g, n, d).permute(2, 0, 1, 3).reshape(n, hkv * g, d)
    return want


def _error(out, want):
    return float((out.double() - want).norm() / want.norm())


@pytest.mark.parametrize("ctx,new,heads,dtype", [
    ([700, 3000, 9000, 5000], [1] * 4, GQA, "bf16"),       # parts that run at once
    ([1999] * 56, [1] * 56, GQA, "bf16"),                  # whole
    ([100 + 150 * i for i in range(20)], [1] * 20, GQA, "f16"),
    ([600, 1999, 2600, 4000] * 20, [1] * 80, GQA, "bf16"),  # only the longest are cut
    ([150 * i for i in range(24)], [1] * 24, GQA_D64, "f16"),
    ([1000] * 10, [128] * 10, MHA, "bf16"),                # matrix-core kernel, whole
    ([1500] * 18, [50] * 18, MHA, "f16"),
    ([400, 900, 1700, 3000] * 2, [200] * 8, GQA, "bf16"),
    ([900] * 6, [100] * 6, GQA_D64, "bf16"),
    ([300 * i for i in range(10)], [60] * 10, PART, "f16"),
])
def test_lists_cut_into_fewer_parts_are_no_further_from_64_bits(monkeypatch, ctx, new, heads, dtype):
    """The probabilities are rounded to 16 bits, except that of each part's reference, so fewer parts
    alone mean a larger error.  Against the cut into about 1024 parts, on the same values: the bound
    is that cut's own error, but for 0.1 % (lists of the 128-row kernel round nearly alike, the lists
    of the other one are 20 % closer)."""
    b, q, k, v = _state(ctx, new, heads, dtype, 61)
    want = _in_64_bits(b, q, k, v)
    out, items = _run(b, q, k, v)
    monkeypatch.setenv("PV_SPLIT_TARGET", "1024")
    even, even_items = _run(b, q, k, v)
    err, even_err = _error(out, want), _error(even, want)
    print(f"{items} {err:.4e}, {even_items} {even_err:.4e}", flush=True)
    assert err <= even_err * 1.001


@pytest.mark.parametrize("ctx,new,heads", [
    ([16000], [365], (10, 10, 128)), ([14000], [70], GQA), ([20000, 9000], [188, 200], GQA),
    ([28000], [128], (16, 2, 128))])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_few_long_prompts_are_no_further_from_64_bits(monkeypatch, ctx, new, heads, dtype):
    """Too few 256-row tiles for a kernel of their own: the 128-row kernel takes them.  Against the
    256-row kernel on the same values, whose queries are rounded once more: no further from 64 bits."""
    from paper_2312_05516_amd import binding as pv
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)

    def tiles():
        plan = pv.plan_create(pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype),
                              b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
        n = pv.plan_num_work_items(plan, 3)
        plan.destroy()
        return n
    b, q, k, v = _state(ctx, new, heads, dtype, 91)
    want = _in_64_bits(b, q, k, v)
    assert tiles() == 0
    err = _error(_run(b, q, k, v)[0], want)
    monkeypatch.setenv("PV_TILE_MIN_KEYS", "8192")
    assert tiles() > 0
    other = _error(_run(b, q, k, v)[0], want)
    print(f"{err:.4e}, with the 256-row kernel {other:.4e}", flush=True)
    assert err <= other
    assert err <= (1.2e-3 if dtype == "f16" else 1e-2)


@pytest.mark.parametrize("ctx,new,heads", [([22000], [640], GQA), ([48000], [2048], (10, 10, 128)),
                                           ([150000, 120000], [560, 300], (16, 2, 128))])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_few_tiles_over_many_keys_are_no_further_from_64_bits(monkeypatch, ctx, new, heads, dtype):
    """Few 256-row tiles over so many keys that they go to the 256-row kernel all the same: with scores
    scaled in fp32, no further from 64 bits than in the 128-row kernel, which rounds nothing that this
    one does not (0.1 % for the parts, which begin at other keys).  Negative, small and zero scales."""
    from paper_2312_05516_amd import binding as pv
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    b, q, k, v = _state(ctx, new, heads, dtype, 93)
    want = _in_64_bits(b, q, k, v)

    def run(scale=None):
        plan = pv.plan_create(pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype),
                              b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
        variants, items = pv.plan_kernel_variants(plan), pv.plan_num_work_items(plan, 3)
        plan.destroy()
        return _run(b, q, k, v, scale)[0], variants & 16, items
    out, scaled, items = run()
    assert scaled and items > 0
    err = _error(out, want)
    for scale in (-b.scale, 1e-30, -1e-30, 0.0):
        exact = _in_64_bits(b, q, k, v, scale)
        # nearly equal weights: an average of 20 K values or more, small against their rounding
        d = float((run(scale)[0].double() - exact).abs().max() / exact.abs().max())
        print(f"scale {scale:.2g}: {d:.2e} of the largest result", flush=True)
        assert d <= (2e-3 if dtype == "f16" else 1.6e-2)
    monkeypatch.setenv("PV_TILE_MIN_KEYS", "0")
    out, _, items = run()
    assert items == 0
    other = _error(out, want)
    print(f"{err:.4e}, with the 128-row kernel {other:.4e}", flush=True)
    assert err <= other * 1.001


@pytest.mark.parametrize("bits", [-300.0, -30.0, -3.0, 3.0, 30.0, 300.0])
@pytest.mark.parametrize("heads,dtype,reqs", [(MHA, "f16", 10), ((20, 20, 64), "bf16", 24)])
def test_reference_is_renewed_under_falling_and_rising_scores(heads, dtype, reqs, bits):
    """Prompts over 1000 cached tokens that are left whole, so that the reference maximum of a row is
    renewed on the way: scores that fall or rise by so many powers of two over the KV range, up to
    where all but a few probabilities vanish.  Tolerance: probabilities and results rounded to 16 bits
    once each (N(0, 1) values: 2.9e-4 and 2.3e-3), times four."""
    import torch
    b, q, k, v = _state([1000] * reqs, [100] * reqs, heads, dtype, 71)
    hkv, d = b.num_kv_heads, b.head_dim
    # one direction of the head carries the slope: score += 4 * slope(position) * scale
    kk = k.view(b.num_pages, hkv, d // 8, 16, 8)
    q[..., 0] = 4.0
    span = bits * math.log(2.0) / (4.0 * b.scale)
    for r in range(b.num_reqs):
        kv = int(b.kv_lens[r])
        n = (kv + 15) // 16
        pages = torch.from_numpy(b.page_table[r, :n].astype(np.int64)).cuda()
        slope = (torch.arange(16 * n, device="cuda", dtype=torch.float32) / kv - 0.5) * span
        rows = kk[pages]
        rows[:, :, 0, :, 0] = slope.view(n, 1, 16).to(k.dtype)
        kk[pages] = rows
    out, items = _run(b, q, k, v)
    assert items == [0, hkv * reqs]
    err = _error(out, _in_64_bits(b, q, k, v))
    assert err <= (1.2e-3 if dtype == "f16" else 1e-2), err


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_infinite_values_stay_infinite(dtype):
    """Generation steps over enough requests that the list is left whole (two-term probabilities): a
    V of plus or minus infinity at a visible key gives that infinity in its dimension, and no NaN."""
    import torch
    b, q, k, v = _state([1999] * 56, [1] * 56, GQA, dtype, 67)
    clean, _ = _run(b, q, k, v)
    vv = v.view(b.num_pages, 8, 2, 128, 8)
    for r, d, sign in ((0, 3, 1.0), (17, 100, -1.0), (55, 127, 1.0)):
        page = int(b.page_table[r, 5])  # keys 80-95
        vv[page, :, 1, d, 2] = sign * math.inf
        out, items = _run(b, q, k, v)
        got = out[int(b.q_start[r])]
        assert bool((got[:, d] == sign * math.inf).all()), (items, got[:, d])
        vv[page, :, 1, d, 2] = 0.0
        keep = torch.ones(128, dtype=torch.bool, device="cuda")
        keep[d] = False
        assert torch.equal(got[:, keep], clean[int(b.q_start[r])][:, keep])

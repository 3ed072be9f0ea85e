"""Matrix-core kernel, on a real MI355X: calls at the limits of its arithmetic."""
import numpy as np
import pytest

import helpers as H
from paper_2312_05516_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,hkv", [(128, 1 << 20), (64, 1 << 21)])
def test_pages_of_4_gib(monkeypatch, head_dim, hkv):
    """2^20 KV heads of size 128 (2^21 of size 64) make one page of the pool 4 GiB: the place of page 1
    does not fit 32 bits.  Page 0 holds other values than page 1, which the request's tokens lie in.
    Results of a few heads against float64; the tolerance is that of the other comparisons."""
    import torch
    from paper_2312_05516_amd import binding as pv
    monkeypatch.setenv("PV_WIDE_MIN_ROWS", "1")  # one row a unit: the matrix-core kernel takes it
    tokens = 7
    desc = pv.pool_desc(2, hkv, head_dim, "f16")
    plan = pv.plan_create(desc, hkv, [tokens - 1], [1], 1)
    assert pv.plan_num_work_items(plan, 1) == hkv and pv.plan_num_work_items(plan, 0) == 0
    pv.plan_upload(plan)
    page = (hkv, 16 * head_dim)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    k = torch.zeros((2,) + page, dtype=torch.float16, device="cuda")
    v = torch.zeros_like(k)
    heads = [0, 1, 31, hkv // 2, hkv - 1]
    for pool in (k, v):
        for hd in heads:
            pool[1, hd].normal_(generator=gen)
    q = torch.zeros((1, hkv, head_dim), dtype=torch.float16, device="cuda")
    for hd in heads:
        q[0, hd].normal_(generator=gen)
    out = torch.full_like(q, float("nan"))
    table = torch.tensor([[1]], dtype=torch.int32, device="cuda")
    pv.multi_token_paged_attn_planned(plan, q, k, v, table, 0.3, out, None)
    torch.cuda.synchronize()
    plan.destroy()
    for hd in heads:
        kk = k[1, hd].view(head_dim // 8, 16, 8).permute(1, 0, 2).reshape(16, head_dim)[:tokens]
        vv = v[1, hd].view(2, head_dim, 8).permute(0, 2, 1).reshape(16, head_dim)[:tokens]
        w = torch.softmax(0.3 * (kk.double() @ q[0, hd].double()), 0)
        err = float((w @ vv.double() - out[0, hd].double()).abs().max())
        print(f"head {hd} of {hkv}: {err:.2e}", flush=True)
        assert err <= H.TOL["f16"], hd


@pytest.mark.parametrize("head_dim,dtype", [(64, "f16"), (128, "f16"), (128, "bf16")])
@pytest.mark.parametrize("scale", [0.0, -0.0])
def test_zero_scale_does_not_hide_infinite_queries(head_dim, dtype, scale):
    """A scale of zero weighs all visible keys alike.  An infinity or a NaN in a query is still NaN
    (0 * inf), in its own row and no other; the same in the keys, for the rows that see them."""
    b = wl.custom([50, 0], [60, 40], num_q_heads=2, num_kv_heads=2, head_dim=head_dim, dtype=dtype,
                  seed=5)
    case = H.make_case(b, fill="nan")
    inf, nan = (0x7C00, 0x7E00) if dtype == "f16" else (0x7F80, 0x7FC0)
    case.q[3, 0, 7] = inf
    case.q[17, 1, head_dim - 1] = 0x8000 | inf
    case.q[59, 0, 0] = nan
    case.q[99, 1, 1] = 0x8000 | nan
    hidden = [(3, 0), (17, 1), (59, 0), (99, 1)]
    got, _, _ = H.gpu_run(case, scale=scale)
    got = H.bits_to_f64(got, dtype)
    case.q[:] = 0
    want = H.dense_causal_attention(case, scale=0.0)
    for row, head in hidden:
        assert np.isnan(got[row, head]).all(), (row, head)
        got[row, head] = want[row, head]
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= H.TOL[dtype]
    # an infinite key at position 80 of the first request: token 30 of the new ones and later see it
    case.k_new[30, 0, 5] = inf
    got, _, _ = H.gpu_run(case, scale=scale)
    got = H.bits_to_f64(got, dtype)
    assert np.isnan(got[30:60, 0]).all()
    got[30:60, 0] = want[30:60, 0]
    assert np.abs(got - want).max() <= H.TOL[dtype]

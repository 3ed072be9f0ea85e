"""Matrix-core kernel, on a real MI355X: which token and head a row is, for groups that do not divide a
tile of rows; the last block of an item, whose V slots past the end are zeroed in LDS; items that read
their K/V with the streaming hint, and items of the narrow kernel that share theirs."""
import numpy as np
import pytest

import helpers as H
from test_gpu_parity import _full_size_parity
from test_gpu_precision import _error, _in_64_bits, _run, _state
from paper_2312_05516_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,new", [(3, 97), (5, 60), (7, 37), (12, 23), (33, 9), (127, 3),
                                       (129, 2), (300, 2), (1000, 1)])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_rows_of_any_group(oracle, group, new, head_dim):
    """Rows in more than one 128-row item, the second of which starts inside a token."""
    b = wl.custom([37, 0], [new, new + 1], num_q_heads=group, num_kv_heads=1, head_dim=head_dim,
                  dtype="f16", seed=group)
    case = H.make_case(b, fill="nan")
    got, _, _ = H.gpu_run(case)
    want, _ = oracle.attn(H.pool_tuple(b), b.num_q_heads, case.q, case.k_pool1, case.v_pool1,
                          b.page_table, b.ctx_lens, b.q_lens, b.q_start, b.scale)
    err = np.abs(H.bits_to_f64(got, b.dtype) - want).max()
    print(f"group {group}, {new} tokens, head size {head_dim}: {err:.3e}", flush=True)
    assert err <= H.TOL[b.dtype], err


@pytest.mark.parametrize("scale", [-0.3, 0.0, 1e-30, 0.3])
@pytest.mark.parametrize("last", [1, 2, 7, 8, 9, 15, 16, 17, 25, 31, 32, 33, 47, 63])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_last_block(oracle, head_dim, last, scale):
    """`last` keys in the last block behind one or two whole ones, the slots behind them NaN; the
    second request's rows end in different blocks."""
    b = wl.custom([64 + last - 40, last], [40, 64], num_q_heads=2, num_kv_heads=2,
                  head_dim=head_dim, dtype="bf16", seed=last)
    case = H.make_case(b, fill="nan")
    got, _, _ = H.gpu_run(case, scale=scale)
    want, _ = oracle.attn(H.pool_tuple(b), b.num_q_heads, case.q, case.k_pool1, case.v_pool1,
                          b.page_table, b.ctx_lens, b.q_lens, b.q_start, scale)
    err = np.abs(H.bits_to_f64(got, b.dtype) - want).max()
    assert err <= H.TOL[b.dtype], err


@pytest.mark.parametrize("heads,new,reqs", [((8, 1, 128), 4, 5), ((8, 1, 128), 3, 600),
                                            ((2, 2, 128), 24, 300), ((4, 1, 64), 8, 5),
                                            ((1, 1, 64), 32, 600), ((16, 1, 64), 2, 300)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_units_of_two_narrow_items(oracle, heads, new, reqs, dtype):
    """17 to 32 rows a unit, so that two items read the same K/V, beside units of one; short lists
    are cut and merged, long ones are not.  (Probabilities in two terms: the next test.)"""
    rng = np.random.default_rng(new)
    ctx = rng.integers(0, 1500 if reqs == 5 else 90, size=reqs)
    b = wl.custom(ctx, np.where(np.arange(reqs) % 3 == 1, 1, new), num_q_heads=heads[0],
                  num_kv_heads=heads[1], head_dim=heads[2], dtype=dtype, seed=reqs)
    case = H.make_case(b, fill="nan")
    got, _, _ = H.gpu_run(case)
    want, _ = oracle.attn(H.pool_tuple(b), b.num_q_heads, case.q, case.k_pool1, case.v_pool1,
                          b.page_table, b.ctx_lens, b.q_lens, b.q_start, b.scale)
    err = np.abs(H.bits_to_f64(got, b.dtype) - want).max()
    print(f"{heads}, {reqs} x {new} tokens {dtype}: {err:.3e}", flush=True)
    assert err <= H.TOL[b.dtype], err


@pytest.mark.parametrize("heads,ctx,new,variants", [
    # bandwidth-oriented kernel: 1 = probabilities in two terms, 2 = streaming hint
    ((4, 1, 64), [341, 170, 90], [6, 6, 6], 0), ((8, 1, 128), [341, 170, 90], [3, 3, 3], 0),
    ((20, 10, 64), [550, 420, 700, 880, 610], [13] * 5, 1), ((16, 8, 128), [520, 480], [13, 13], 1),
    ((4, 1, 64), [341, 170, 90], [2, 2, 2], 2), ((8, 1, 128), [341, 170, 90], [1, 1, 1], 2),
    ((4, 1, 64), [520, 600], [3, 3], 3), ((16, 2, 128), [603], [1], 3),
    # 128-row kernel: 4 = renewed references, 8 = streaming hint
    ((8, 8, 64), [100, 0, 33], [140, 50, 90], 0), ((8, 8, 128), [100, 0, 33], [140, 50, 90], 0),
    ((12, 12, 64), [900] * 20, [100] * 20, 4), ((10, 10, 128), [800] * 16, [100] * 16, 4),
    ((40, 40, 64), [600] * 40, [60] * 40, 8), ((40, 40, 128), [300] * 28, [60] * 28, 8),
    ((20, 20, 64), [1000] * 24, [100] * 24, 12), ((20, 20, 128), [1500] * 20, [100] * 20, 12)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_every_variant_of_the_kernels(heads, ctx, new, variants, dtype):
    """Every instantiation that the launches choose from, with the plan held to it.  Tolerance against
    64 bits: probabilities and results rounded to 16 bits once each (3e-4 and 2.5e-3; two terms are
    closer), times four."""
    import torch
    from paper_2312_05516_amd import binding as pv
    b, q, k, v = _state(ctx, new, heads, dtype, 83)
    plan = pv.plan_create(pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype),
                          b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    assert pv.plan_kernel_variants(plan) == variants
    plan.destroy()
    # slots past the end of a request may hold anything
    kv_ = k.view(b.num_pages, b.num_kv_heads, b.head_dim // 8, 16, 8)
    vv = v.view(b.num_pages, b.num_kv_heads, 2, b.head_dim, 8)
    for r in range(b.num_reqs):
        end = int(b.kv_lens[r]) % 16
        page = int(b.page_table[r, (int(b.kv_lens[r]) - 1) // 16])
        for slot in range(end or 16, 16):
            kv_[page, :, :, slot, :] = float("nan")
            vv[page, :, slot // 8, :, slot % 8] = float("nan")
    out, items = _run(b, q, k, v)
    assert (items[0] == 0) == (variants >= 4 or min(new) * heads[0] // heads[1] > 32)
    err = _error(out, _in_64_bits(b, q, k, v))
    print(f"{items} {err:.2e}", flush=True)
    assert err <= (1.2e-3 if dtype == "f16" else 1e-2), err


@pytest.mark.parametrize("heads,dtype,ctx,reqs", [
    ((10, 10, 128), "f16", 1100, 24), ((40, 10, 128), "bf16", 1100, 24),
    ((32, 8, 64), "bf16", 1100, 60), ((12, 12, 64), "f16", 1100, 40),
    ((10, 10, 128), "bf16", 7000, 6),    # KV ranges in parts
    ((20, 20, 128), "f16", 1200, 20)])   # renewed references
def test_units_of_one_tile_in_a_large_batch(oracle, heads, dtype, ctx, reqs):
    """More K/V than the limit from which units of one 128-row tile read theirs with the streaming
    hint, beside units of several tiles and generation steps, which end anywhere in a block."""
    rng = np.random.default_rng(reqs)
    g = heads[0] // heads[1]
    new = np.array([(1, 128 // g, 40 // g, 150 // g)[i % 4] for i in range(reqs)])
    b = wl.custom(rng.integers(ctx - 100, ctx + 100, size=reqs), new, num_q_heads=heads[0],
                  num_kv_heads=heads[1], head_dim=heads[2], dtype=dtype, seed=reqs)
    assert 4 * int(b.kv_lens.sum()) * heads[1] * heads[2] > 96 << 20
    _full_size_parity(oracle, b, [0, 1, 2, 3], [0, heads[1] - 1])

"""Matrix-core kernel, on a real MI355X: which token and head a row is, for groups that do not divide a
tile of rows; the last block of an item, whose V slots past the end are zeroed in LDS; items that read
their K/V with the streaming hint, and items of the narrow kernel that share theirs."""
import numpy as np
import pytest

import helpers as H
from test_gpu_parity import _full_size_parity
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
    are cut (with probabilities in two terms) and merged, long ones are not."""
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

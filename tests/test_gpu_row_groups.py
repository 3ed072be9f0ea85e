"""Matrix-core kernel, on a real MI355X: which token and head a row is, for groups that do not divide
a tile of rows, and the last block of an item, whose V slots past the end are zeroed in LDS."""
import numpy as np
import pytest

import helpers as H
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

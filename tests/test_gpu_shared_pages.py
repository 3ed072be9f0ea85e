"""Requests of one batch that read the same pages (a common prefix; the sub-requests of a request that is
partly recomputed), on a real MI355X: where the 128-row kernel reads K/V with the streaming hint it
looks at the page table for such pages."""
import numpy as np
import pytest

from paper_2312_05516_amd import workloads as wl
from test_gpu_precision import _error, _in_64_bits, _run

pytestmark = pytest.mark.gpu

STREAMS = 8


def _variants(b):
    from paper_2312_05516_amd import binding as pv
    plan = pv.plan_create(pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype),
                          b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    v = pv.plan_kernel_variants(plan)
    plan.destroy()
    return v


@pytest.mark.parametrize("heads,dtype,reqs,prefix,prefixes", [
    ((40, 40, 128), "f16", 24, 640, 1), ((40, 10, 128), "bf16", 70, 512, 2),  # more than 64 requests
    ((64, 8, 128), "f16", 64, 640, 3), ((32, 8, 64), "bf16", 130, 400, 2),
    ((20, 20, 128), "bf16", 9, 2000, 9),     # everyone by himself, KV ranges in parts
    ((20, 20, 128), "bf16", 9, 2000, 2)])
def test_common_prefixes(heads, dtype, reqs, prefix, prefixes):
    """`prefixes` prefixes that the requests read in turn: the result is that of the same K/V in pages
    of every request's own, bit for bit.  Tolerance against 64 bits: probabilities and results rounded
    to 16 bits once each (2.9e-4 and 2.9e-3), times four."""
    import torch
    rng = np.random.default_rng(reqs)
    g = heads[0] // heads[1]
    new = [int(x) for x in rng.integers(1, 128 // g + 1, size=reqs)]
    ctx = [prefix + int(x) for x in rng.integers(0, 90, size=reqs)]
    b = wl.custom(ctx, new, num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=heads[2],
                  dtype=dtype, seed=reqs)
    assert _variants(b) & STREAMS
    td = torch.float16 if dtype == "f16" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)

    def draw(*shape):
        return torch.empty(shape, dtype=td, device="cuda").normal_(generator=gen)
    pool = (b.num_pages, b.num_kv_heads * 16 * b.head_dim)
    q, k, v = draw(b.total_q, b.num_q_heads, b.head_dim), draw(*pool), draw(*pool)
    n = prefix // 16
    own = b.page_table.copy()
    shared = own.copy()
    for r in range(reqs):
        shared[r, :n] = own[r % prefixes, :n]
        to, of = (torch.from_numpy(t[:n].astype(np.int64)).cuda() for t in (own[r], shared[r]))
        k[to], v[to] = k[of], v[of]
    want, _ = _run(b, q, k, v)
    exact = _in_64_bits(b, q, k, v)
    b.page_table = shared
    got, items = _run(b, q, k, v)
    err = _error(got, exact)
    print(f"{items} {err:.2e}", flush=True)
    assert items[1] > 0 and torch.equal(got, want)
    assert err <= (1.2e-3 if dtype == "f16" else 1.2e-2)


def test_sub_requests():
    """The first part of a conversation recomputed next to its new prompt, which reads those pages too:
    two rows of the table that begin with the same pages, the shorter row's remaining entries invalid."""
    import torch
    new, ctx = [], []
    for i in range(8):
        new += [100 - i, 80 + i]
        ctx += [0, 2000 + 17 * i]
    b = wl.custom(ctx, new, num_q_heads=40, num_kv_heads=40, head_dim=128, dtype="bf16", seed=3)
    assert _variants(b) & STREAMS
    table = b.page_table.copy()
    for r in range(0, 16, 2):
        n = (new[r] + 15) // 16
        table[r] = -1
        table[r, :n] = table[r + 1, :n]
    b.page_table = table
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)

    def draw(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    pool = (b.num_pages, b.num_kv_heads * 16 * b.head_dim)
    q, k, v = draw(b.total_q, b.num_q_heads, b.head_dim), draw(*pool), draw(*pool)
    got, items = _run(b, q, k, v)
    err = _error(got, _in_64_bits(b, q, k, v))
    print(f"{items} {err:.2e}", flush=True)
    assert items[1] > 0 and err <= 1.2e-2

"""Parity of the HIP library (through its C ABI) with the CPU oracle, on a real MI355X.

Bars (stated by the benchmark spec): KV append and everything that depends only on page-table indexing is
bit-exact; attention output is within max-abs-error 5e-3 (fp16) / 2e-2 (bf16) of the oracle.
"""
import numpy as np
import pytest

import helpers as H
from paper_2312_05516_amd import workloads as wl

pytestmark = pytest.mark.gpu


def oracle_out(oracle, case, pools=None, page_table=None, scale=None, **kw):
    b = case.batch
    kp, vp = pools if pools is not None else (case.k_pool1, case.v_pool1)
    out, _ = oracle.attn(H.pool_tuple(b), b.num_q_heads, case.q, kp, vp,
                         b.page_table if page_table is None else page_table, b.ctx_lens, b.q_lens,
                         b.q_start, b.scale if scale is None else scale, **kw)
    return out


def check_case(oracle, case, **kw):
    b = case.batch
    print(f"case {b.name}: ctx={b.ctx_lens.tolist()[:8]} q={b.q_lens.tolist()[:8]} "
          f"Hq={b.num_q_heads} Hkv={b.num_kv_heads} D={b.head_dim} {b.dtype}", flush=True)
    got_bits, kp, vp = H.gpu_run(case, **kw)
    # append: bit-exact pool image (also proves untouched slots kept their NaN fill)
    assert np.array_equal(kp, case.k_pool1), "K pool differs after append"
    assert np.array_equal(vp, case.v_pool1), "V pool differs after append"
    want = oracle_out(oracle, case)
    got = H.bits_to_f64(got_bits, b.dtype)
    assert np.isfinite(got).all(), "non-finite output"
    err = np.abs(got - want).max() if got.size else 0.0
    print(f"  max abs err {err:.3e}", flush=True)
    assert err <= H.TOL[b.dtype], err
    return got_bits


SHAPES = [
    # ctx_lens, q_lens, Hq, Hkv, D, dtype
    ([37, 100], [5, 12], 4, 4, 64, "f16"),
    ([0, 16, 31, 32, 33], [7, 1, 33, 1, 31], 4, 2, 64, "bf16"),
    ([5, 0, 48, 15, 1], [1, 1, 16, 17, 1], 8, 2, 128, "f16"),
    ([63, 64, 65, 0], [2, 1, 1, 1], 2, 1, 128, "bf16"),
    ([200, 0, 77], [40, 130, 1], 8, 1, 128, "bf16"),  # 8 query heads on one KV head
    ([300, 513], [70, 1], 5, 5, 128, "f16"),  # odd head count
    ([129], [64], 16, 1, 64, "f16"),  # 16 query heads share one KV head: one token fills a tile
    ([10, 10], [0, 3], 2, 2, 64, "f16"),  # a request without new tokens
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_small_shapes(oracle, shape):
    ctx, qn, hq, hkv, d, dt = shape
    b = wl.custom(ctx, qn, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, dtype=dt, seed=41)
    check_case(oracle, H.make_case(b, fill="nan"))


def test_tiny_config(oracle):
    check_case(oracle, H.make_case(wl.tiny(), fill="nan"))


def test_one_shot_entry_points_match_planned(oracle):
    b = wl.custom([45, 3, 260], [9, 1, 20], num_q_heads=8, num_kv_heads=2, head_dim=128,
                  dtype="f16", seed=43)
    case = H.make_case(b)
    planned = check_case(oracle, case)
    one = check_case(oracle, case, one_shot=True)
    assert np.array_equal(planned, one)


@pytest.mark.parametrize("reqs,head_dim", [(1, 128), (95, 64), (96, 128), (97, 64), (193, 128)])
def test_one_shot_append_of_any_number_of_requests(oracle, reqs, head_dim):
    """The one-shot append takes 96 requests a launch as kernel arguments: counts on both sides of
    that, requests without new tokens among them, runs that start and end anywhere in a page."""
    rng = np.random.default_rng(reqs)
    new = np.where(rng.random(reqs) < 0.2, 0, rng.integers(1, 41, size=reqs))
    new[-1] = 17
    b = wl.custom(rng.integers(0, 60, size=reqs), new, num_q_heads=2, num_kv_heads=2,
                  head_dim=head_dim, dtype="bf16", seed=900 + reqs)
    case = H.make_case(b, fill="nan")
    out, kp, vp = H.gpu_run(case, one_shot=True)
    assert np.array_equal(kp, case.k_pool1.ravel()) and np.array_equal(vp, case.v_pool1.ravel())
    assert np.abs(H.bits_to_f64(out, b.dtype) - oracle_out(oracle, case)).max() <= H.TOL[b.dtype]


def test_one_shot_calls_back_to_back_and_without_room_for_the_lists(oracle, monkeypatch):
    """Several one-shot attention calls in a row behind a kernel that keeps the stream busy, without a
    wait in between: the temporary plan of each is gone when its kernels start, and the next call's,
    of a batch with other lengths, may lie in the same host memory.  Then once more with no workspace
    at all (the lists then go to temporary device memory and the call waits).  All give their
    batch's planned result."""
    import torch
    from paper_2312_05516_amd import binding as pv
    monkeypatch.setenv("PV_SPLIT_TARGET", "1")  # no split KV ranges: no partial results to hold
    calls = []
    for i, (ctx, new) in enumerate([([300, 17, 900, 0], [33, 1, 140, 64]),
                                    ([17, 900, 0, 300], [1, 64, 140, 33]),
                                    ([0, 301, 33, 860], [140, 33, 64, 1]),
                                    ([900, 0, 300, 16], [64, 140, 33, 2])]):
        b = wl.custom(ctx, new, num_q_heads=8, num_kv_heads=2, head_dim=128, dtype="bf16",
                      seed=47 + i)
        case = H.make_case(b)
        planned, kpool, vpool = H.gpu_run(case)
        desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
        q = H.to_dev_bits(case.q, b.dtype)
        nbytes = pv.attn_workspace_bytes(desc, b.num_q_heads, b.num_reqs, b.total_q,
                                         int(b.kv_lens.max()))
        calls.append((b, planned, desc, q, H.to_dev_bits(kpool.reshape(case.k_pool0.shape), b.dtype),
                      H.to_dev_bits(vpool.reshape(case.v_pool0.shape), b.dtype),
                      torch.from_numpy(b.page_table).cuda(), torch.full_like(q, float("nan")),
                      torch.empty(nbytes, dtype=torch.uint8, device="cuda")))

    def call(i, out, space):
        b, _, desc, q, kp, vp, table, _, _ = calls[i]
        pv.multi_token_paged_attn(desc, b.num_q_heads, q, kp, vp, table, b.max_pages_per_req,
                                  b.ctx_lens, b.q_lens, b.q_start, b.scale, out, space)

    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(8):
        busy = busy @ busy * 1e-2
    for i in range(4):
        call(i, calls[i][7], calls[i][8])
    torch.cuda.synchronize()
    for c in calls:
        assert np.array_equal(H.from_dev_bits(c[7]), c[1])
    last = torch.full_like(calls[0][3], float("nan"))
    call(0, last, None)
    torch.cuda.synchronize()
    assert np.array_equal(H.from_dev_bits(last), calls[0][1])


def test_empty_batch_is_a_no_op():
    import torch
    from paper_2312_05516_amd import binding as pv
    desc = pv.pool_desc(8, 2, 64, "f16")
    plan = pv.plan_create(desc, 2, [], [], 4)
    pv.plan_upload(plan)
    dummy = torch.zeros(16, dtype=torch.float16, device="cuda")
    table = torch.zeros(4, dtype=torch.int32, device="cuda")
    pv.kv_append_planned(plan, dummy, dummy, table, dummy, dummy)
    pv.multi_token_paged_attn_planned(plan, dummy, dummy, dummy, table, 1.0, dummy, None)
    torch.cuda.synchronize()
    plan.destroy()


def test_split_kv_and_combine(oracle, monkeypatch):
    """Few long requests: the plan cuts their KV range into parts that are merged afterwards."""
    from paper_2312_05516_amd import binding as pv
    b = wl.custom([3000, 1500, 700], [1, 3, 40], num_q_heads=8, num_kv_heads=2, head_dim=128,
                  dtype="bf16", seed=47)
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    assert pv.plan_num_work_items(plan, 2) > 0 and pv.plan_workspace_bytes(plan) > 0
    plan.destroy()
    check_case(oracle, H.make_case(b, fill="nan"))
    b2 = wl.custom([5000], [1], num_q_heads=4, num_kv_heads=4, head_dim=64, dtype="f16", seed=48)
    check_case(oracle, H.make_case(b2, fill="nan"))


@pytest.mark.parametrize("parts", [2, 3, 4, 7, 8, 15, 16, 17, 32, 33, 70])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_merge_of_any_number_of_parts(oracle, monkeypatch, parts, head_dim):
    """The merge spreads the parts of a row over one to eight thread groups: counts on both sides of
    each step, more parts than a group has threads, rows that do not fill a workgroup."""
    from paper_2312_05516_amd import binding as pv
    monkeypatch.setenv("PV_MIN_SPLIT_KEYS", "32")
    monkeypatch.setenv("PV_SPLIT_TARGET", str(parts))
    b = wl.custom([32 * parts - 3], [3], num_q_heads=3, num_kv_heads=1, head_dim=head_dim,
                  dtype="bf16" if parts % 2 else "f16", seed=480 + parts)
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    assert pv.plan_num_work_items(plan, 0) == parts and pv.plan_num_work_items(plan, 2) == 1
    plan.destroy()
    check_case(oracle, H.make_case(b, fill="nan"))


@pytest.mark.parametrize("hkv,head_dim,dtype", [(33, 64, "f16"), (33, 64, "bf16"), (17, 128, "f16")])
def test_append_of_more_rows_than_the_streaming_limit(hkv, head_dim, dtype):
    """New rows of just over 32 MiB are read with the streaming hint: K and V bit for bit, partial
    8-slot groups at both ends of the long request."""
    n = (32 << 20) // (hkv * head_dim * 4) + 3
    b = wl.custom([5, 0], [n, 3], num_q_heads=hkv, num_kv_heads=hkv, head_dim=head_dim, dtype=dtype,
                  seed=540 + head_dim)
    assert b.total_q * hkv * head_dim * 4 > 32 << 20
    case = H.make_case(b, fill="nan")
    _, kp, vp = H.gpu_run(case)
    assert np.array_equal(kp, case.k_pool1.ravel()) and np.array_equal(vp, case.v_pool1.ravel())


@pytest.mark.parametrize("new,hkv,parts", [(128, 4, 16), (64, 16, 17), (128, 33, 9), (128, 33, 17)])
def test_merge_of_many_rows(oracle, monkeypatch, new, hkv, parts):
    """Merges of 512 to 4224 rows: eight, four and two thread groups a row become four, two and one
    where the rows fill the GPU by themselves, on both sides of the limit of 4096 rows times groups."""
    from paper_2312_05516_amd import binding as pv
    monkeypatch.setenv("PV_MIN_SPLIT_KEYS", "32")
    monkeypatch.setenv("PV_SPLIT_TARGET", str(parts * hkv))
    b = wl.custom([32 * parts - new], [new], num_q_heads=hkv, num_kv_heads=hkv, head_dim=64,
                  dtype="f16", seed=520 + parts)
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    assert pv.plan_num_work_items(plan, 1) == parts * hkv and pv.plan_num_work_items(plan, 2) == hkv
    plan.destroy()
    check_case(oracle, H.make_case(b, fill="nan"))


@pytest.mark.parametrize("kv_len", [1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 193])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_matrix_core_kernel_block_edges(oracle, monkeypatch, kv_len, head_dim):
    """KV lengths around the 32- and 64-key blocks of the 128-row kernel, whole and cut into parts of
    32 keys (a part then ends in the middle of a 64-key block: keys behind it are not the part's)."""
    new = min(kv_len, 41)
    b = wl.custom([kv_len - new, 70], [new, 40], num_q_heads=2, num_kv_heads=1, head_dim=head_dim,
                  dtype="bf16" if kv_len % 2 else "f16", seed=700 + kv_len)
    check_case(oracle, H.make_case(b, fill="nan"))
    monkeypatch.setenv("PV_MIN_SPLIT_KEYS", "32")
    monkeypatch.setenv("PV_SPLIT_TARGET", "64")
    check_case(oracle, H.make_case(b, fill="nan"))


@pytest.mark.parametrize("reqs,longest", [(512, 15), (513, 15), (513, 40), (700, 1100)])
def test_lists_longer_than_the_slots_of_the_narrow_kernel(oracle, reqs, longest):
    """With more items than run at once an item also touches the page ids of a later one: lists just
    up to and beyond that, page tables of one column and of more columns than a wavefront has lanes."""
    rng = np.random.default_rng(reqs + longest)
    ctx = rng.integers(0, 15, size=reqs)
    ctx[reqs // 2] = ctx[-1] = longest - 1
    b = wl.custom(ctx, np.ones(reqs, dtype=np.int64), num_q_heads=1, num_kv_heads=1, head_dim=128,
                  dtype="f16", seed=1100 + reqs)
    check_case(oracle, H.make_case(b, fill="nan"))


def test_workspace_is_checked():
    import torch
    from paper_2312_05516_amd import binding as pv
    b = wl.custom([4000], [1], num_q_heads=2, num_kv_heads=2, head_dim=64, seed=1)
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, 2, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    need = pv.plan_workspace_bytes(plan)
    assert need > 0
    dummy = torch.zeros(1 << 20, dtype=torch.float16, device="cuda")
    table = torch.zeros(b.max_pages_per_req, dtype=torch.int32, device="cuda")
    small = torch.empty(need - 1, dtype=torch.uint8, device="cuda")
    for ws in (None, small):
        with pytest.raises(pv.PvError) as e:
            pv.multi_token_paged_attn_planned(plan, dummy, dummy, dummy, table, 1.0, dummy, ws)
        assert e.value.status == 4
    with pytest.raises(pv.PvError) as e:
        pv.multi_token_paged_attn_planned(plan, None, dummy, dummy, table, 1.0, dummy, small)
    assert e.value.status == 1
    plan.destroy()


def test_page_permutation_gives_identical_bits(oracle):
    """Moving pages around (and rewriting the table) must not change a single output bit."""
    b = wl.custom([37, 100, 3, 700], [5, 12, 1, 20], num_q_heads=4, num_kv_heads=2, head_dim=128,
                  dtype="f16", seed=51)
    case = H.make_case(b, fill="random")
    base, _, _ = H.gpu_run(case)
    rng = np.random.default_rng(5)
    page_elems = b.num_kv_heads * b.page_size * b.head_dim
    for _ in range(2):
        perm = rng.permutation(b.num_pages)
        kp = np.empty_like(case.k_pool0).reshape(b.num_pages, page_elems)
        vp = np.empty_like(case.v_pool0).reshape(b.num_pages, page_elems)
        kp[perm] = case.k_pool0.reshape(b.num_pages, page_elems)
        vp[perm] = case.v_pool0.reshape(b.num_pages, page_elems)
        table = np.where(b.page_table >= 0, perm[np.maximum(b.page_table, 0)], -1).astype(np.int32)
        got, _, _ = H.gpu_run(case, page_table=table, pools=(kp.ravel(), vp.ravel()))
        assert np.array_equal(got, base)


def test_sub_requests_share_pages(oracle):
    """Two batch entries on the same pages (paper Section 4.3.4) against one full prefill."""
    L, n_drop, n_new = 150, 40, 21
    full = wl.custom([0], [L], num_q_heads=4, num_kv_heads=2, head_dim=64, seed=53)
    cf = H.make_case(full)
    ref = oracle_out(oracle, cf)
    sub = wl.custom([0, L - n_new], [n_drop, n_new], num_q_heads=4, num_kv_heads=2, head_dim=64,
                    seed=53, pool_pages=full.num_pages)
    sub.page_table = np.full((2, full.page_table.shape[1]), -1, dtype=np.int32)
    sub.page_table[0, :(n_drop + 15) // 16] = full.page_table[0, :(n_drop + 15) // 16]
    sub.page_table[1] = full.page_table[0]
    cs = H.make_case(sub)  # only used as a container below
    cs.q = np.concatenate([cf.q[:n_drop], cf.q[L - n_new:]])
    got_bits, _, _ = H.gpu_run(cs, pools=(cf.k_pool1, cf.v_pool1), do_append=False)
    got = H.bits_to_f64(got_bits, sub.dtype)
    want = np.concatenate([ref[:n_drop], ref[L - n_new:]])
    assert np.abs(got - want).max() <= H.TOL[sub.dtype]


def test_append_unique_patterns_both_dtypes(oracle):
    for dt, d in (("f16", 128), ("bf16", 64)):
        b = wl.custom([37, 0, 16, 15, 255], [5, 40, 1, 2, 1], num_q_heads=4, num_kv_heads=2,
                      head_dim=d, seed=57, dtype=dt)
        case = H.make_case(b, fill="nan")
        N, Hkv = b.total_q, b.num_kv_heads
        k_new = (np.arange(N * Hkv * d, dtype=np.uint32) % 30000 + 1).astype(np.uint16)
        v_new = (np.arange(N * Hkv * d, dtype=np.uint32) % 30000 + 30001).astype(np.uint16)
        k_new, v_new = k_new.reshape(N, Hkv, d), v_new.reshape(N, Hkv, d)
        kp, vp = case.k_pool0.copy(), case.v_pool0.copy()
        oracle.kv_append(H.pool_tuple(b), k_new, v_new, b.page_table, b.ctx_lens, b.q_lens,
                         b.q_start, kp, vp)
        _, gk, gv = H.gpu_run(case, k_new=k_new, v_new=v_new)
        assert np.array_equal(gk, kp) and np.array_equal(gv, vp)


def test_extreme_scores_stay_finite(oracle):
    """Large scale: softmax becomes (nearly) one-hot; V[t,0] = t/64 makes the output name the
    position while staying in the value range the 5e-3 bar is meant for."""
    D, ctx, n = 64, 45, 20
    b = wl.custom([ctx], [n], num_q_heads=1, num_kv_heads=1, head_dim=D, seed=8)
    L = ctx + n
    rng = np.random.default_rng(0)
    K = np.where(rng.random((L, 1, D)) < 0.5, -1.0, 1.0)
    V = np.zeros((L, 1, D))
    V[:, 0, 0] = np.arange(L) / 64.0
    case2 = H.make_case(b, fill="nan", k_full=[H.f64_to_bits(K, "f16")],
                        v_full=[H.f64_to_bits(V, "f16")])
    for target in [0, 15, 16, ctx - 1, ctx, ctx + 1, 47, 48, L - 1]:
        case2.q = np.repeat(H.f64_to_bits(K[target], "f16")[None], n, axis=0)
        got_bits, _, _ = H.gpu_run(case2, scale=1.0)
        got = H.bits_to_f64(got_bits, "f16")
        want = oracle_out(oracle, case2, scale=1.0)
        assert np.isfinite(got).all()
        assert np.abs(got - want).max() <= 5e-3, target


# ---------------------------------------------------------------------------------------------
# full-size configurations: parity on sampled (request, KV head) units
# ---------------------------------------------------------------------------------------------
def _full_size_parity(oracle, b, sample_reqs, sample_heads, value_seed=0):
    import torch
    from paper_2312_05516_amd import binding as pv
    dev = "cuda"
    tdt = torch.float16 if b.dtype == "f16" else torch.bfloat16
    Hq, Hkv, D = b.num_q_heads, b.num_kv_heads, b.head_dim
    print(f"full-size {b.name}: R={b.num_reqs} N={b.total_q} pages={b.num_pages} "
          f"sample reqs={list(sample_reqs)} heads={list(sample_heads)}", flush=True)
    kp = wl.random_values((b.num_pages, Hkv * b.page_size * D), b.dtype, b.seed * 11 + 1, 1.0, dev)
    vp = wl.random_values((b.num_pages, Hkv * b.page_size * D), b.dtype, b.seed * 11 + 2, 1.0, dev)
    q = wl.random_values((b.total_q, Hq, D), b.dtype, b.seed * 11 + 3, 1.0, dev)
    kn = wl.random_values((b.total_q, Hkv, D), b.dtype, b.seed * 11 + 4, 1.0, dev)
    vn = wl.random_values((b.total_q, Hkv, D), b.dtype, b.seed * 11 + 5, 1.0, dev)
    table = torch.from_numpy(b.page_table).to(dev)
    desc = pv.pool_desc(b.num_pages, Hkv, D, b.dtype)
    # sub-pool of the sampled requests BEFORE the append (for the oracle's own append)
    pages, remap = [], {}
    sub_table = np.full((len(sample_reqs), b.max_pages_per_req), -1, dtype=np.int32)
    for i, r in enumerate(sample_reqs):
        npg = int((b.kv_lens[r] + b.page_size - 1) // b.page_size)
        for lp in range(npg):
            p = int(b.page_table[r, lp])
            if p not in remap:
                remap[p] = len(pages)
                pages.append(p)
            sub_table[i, lp] = remap[p]
    idx = torch.tensor(pages, dtype=torch.long, device=dev)
    sub_k = H.from_dev_bits(kp.index_select(0, idx)).ravel().copy()
    sub_v = H.from_dev_bits(vp.index_select(0, idx)).ravel().copy()

    plan = pv.plan_create(desc, Hq, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    ws = torch.empty(max(pv.plan_workspace_bytes(plan), 256), dtype=torch.uint8, device=dev)
    out = torch.full((b.total_q, Hq, D), float("nan"), dtype=tdt, device=dev)
    pv.kv_append_planned(plan, kn, vn, table, kp, vp)
    pv.multi_token_paged_attn_planned(plan, q, kp, vp, table, b.scale, out, ws)
    torch.cuda.synchronize()
    plan.destroy()
    assert torch.isfinite(out.float()).all()

    # oracle on the sampled requests only (own append into the sub-pool, own attention)
    sel_rows = np.concatenate([np.arange(b.q_start[r], b.q_start[r] + b.q_lens[r])
                               for r in sample_reqs]).astype(np.int64)
    rows_t = torch.from_numpy(sel_rows).to(dev)
    q_s = H.from_dev_bits(q.index_select(0, rows_t))
    kn_s = H.from_dev_bits(kn.index_select(0, rows_t))
    vn_s = H.from_dev_bits(vn.index_select(0, rows_t))
    ctx_s = b.ctx_lens[list(sample_reqs)]
    ql_s = b.q_lens[list(sample_reqs)]
    qs_s = np.concatenate([[0], np.cumsum(ql_s)[:-1]]).astype(np.int32)
    pool_s = (len(pages), b.page_size, Hkv, D, b.dtype)
    oracle.kv_append(pool_s, kn_s, vn_s, sub_table, ctx_s, ql_s, qs_s, sub_k, sub_v)
    # append parity on the sampled pages: bit-exact
    got_k = H.from_dev_bits(kp.index_select(0, idx)).ravel()
    got_v = H.from_dev_bits(vp.index_select(0, idx)).ravel()
    assert np.array_equal(got_k, sub_k) and np.array_equal(got_v, sub_v)
    mask = np.zeros((len(sample_reqs), Hkv), dtype=np.uint8)
    mask[:, list(sample_heads)] = 1
    want, info = oracle.attn(pool_s, Hq, q_s, sub_k, sub_v, sub_table, ctx_s, ql_s, qs_s, b.scale,
                             unit_mask=mask)
    got = H.bits_to_f64(H.from_dev_bits(out.index_select(0, rows_t)), b.dtype)
    sel = ~np.isnan(want)
    assert sel.any()
    err = np.abs(got[sel] - want[sel]).max()
    print(f"  sampled elements {int(sel.sum())}, max abs err {err:.3e}", flush=True)
    assert err <= H.TOL[b.dtype], err


def _pick_reqs(b, k=4):
    order = np.argsort(b.kv_lens)
    qorder = np.argsort(b.q_lens)
    picks = [int(order[0]), int(order[-1]), int(qorder[-1]), int(qorder[0])]
    rng = np.random.default_rng(b.seed)
    picks += [int(x) for x in rng.choice(b.num_reqs, size=k, replace=False)]
    return sorted(set(picks))


def test_full_size_mha13b(oracle):
    b = wl.mha13b()
    _full_size_parity(oracle, b, _pick_reqs(b, 3), [0, 17, 39])


def test_full_size_gqa70b(oracle):
    b = wl.gqa70b()
    _full_size_parity(oracle, b, _pick_reqs(b, 3), [0, 5])


def test_full_size_decode_heavy(oracle):
    b = wl.decode_heavy()
    _full_size_parity(oracle, b, _pick_reqs(b, 6), [0, 13, 39])


def test_full_size_long_history(oracle):
    b = wl.long_history()
    order = np.argsort(b.kv_lens)
    # the oracle is O(n * L * D) per head: two requests x one KV head (8 query heads) stays ~20 s
    _full_size_parity(oracle, b, [int(order[0]), int(order[-1])], [3])


@pytest.mark.parametrize("kernels", ["one_attention_kernel", "two_attention_kernels",
                                     "with_256_row_kernel"])
def test_graph_replay_matches_eager(oracle, kernels, monkeypatch):
    """The planned calls of a mixed batch (append, attention, the merge) captured into one HIP
    graph: every replay must reproduce the eager result bit for bit, with eager work and
    synchronisations between the replays.  Once as the plan routes it (generation steps go to the
    matrix-core kernel too) and once with the limit for that lowered so that they keep their own
    kernel (the limit is read when the plan is created)."""
    import torch
    from paper_2312_05516_amd import binding as pv
    b = wl.custom([700, 40, 2200, 5], [1, 70, 3, 150], num_q_heads=8, num_kv_heads=2,
                  head_dim=128, dtype="bf16", seed=61)
    if kernels == "two_attention_kernels":
        monkeypatch.setenv("PV_UNIFY_MAX_STEPS", "10")
    if kernels == "with_256_row_kernel":  # the 150-token request: 600 rows = two 256-row tiles + rest
        monkeypatch.setenv("PV_TILE_MIN_KEYS", "128")
    case = H.make_case(b, fill="nan")
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    plan = pv.plan_create(desc, b.num_q_heads, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    if kernels == "one_attention_kernel":
        assert pv.plan_num_work_items(plan, 0) == 0 and pv.plan_num_work_items(plan, 1) > 0
    elif kernels == "with_256_row_kernel":
        assert pv.plan_num_work_items(plan, 3) >= 4 and pv.plan_num_work_items(plan, 1) > 0
    else:
        assert pv.plan_num_work_items(plan, 0) > 0 and pv.plan_num_work_items(plan, 1) > 0
    assert pv.plan_num_work_items(plan, 2) > 0
    table = torch.from_numpy(b.page_table).cuda()
    q = H.to_dev_bits(case.q, b.dtype)
    kn, vn = H.to_dev_bits(case.k_new, b.dtype), H.to_dev_bits(case.v_new, b.dtype)
    kp, vp = H.to_dev_bits(case.k_pool0, b.dtype), H.to_dev_bits(case.v_pool0, b.dtype)
    ws = torch.empty(max(pv.plan_workspace_bytes(plan), 256), dtype=torch.uint8, device="cuda")
    out = torch.zeros((b.total_q, b.num_q_heads, b.head_dim), dtype=q.dtype, device="cuda")

    def step():
        pv.kv_append_planned(plan, kn, vn, table, kp, vp)
        pv.multi_token_paged_attn_planned(plan, q, kp, vp, table, b.scale, out, ws)

    step()
    torch.cuda.synchronize()
    eager = H.from_dev_bits(out).copy()
    want = oracle_out(oracle, case)
    assert np.abs(H.bits_to_f64(eager, b.dtype) - want).max() <= H.TOL[b.dtype]
    g = torch.cuda.CUDAGraph()
    cap = torch.cuda.Stream()
    with torch.cuda.graph(g, stream=cap):
        step()
    for rep in range(4):
        out.zero_()
        ws.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(H.from_dev_bits(out), eager), rep
        step()  # eager work between replays
        torch.cuda.synchronize()
        assert np.array_equal(H.from_dev_bits(out), eager), rep
    plan.destroy()


@pytest.mark.parametrize("requests", [3, 300])
def test_one_shot_attention_captured_into_a_graph(oracle, requests):
    """The one-shot attention call under capture: its temporary plan is gone when the graph runs, so
    every replay has to bring its own lists.  One piece of them and several (300 requests); replays
    with the workspace overwritten and other one-shot calls (their plans reuse the freed host memory)
    in between.  Without room for the lists the call is refused and the capture stays usable."""
    import torch
    from paper_2312_05516_amd import binding as pv
    rng = np.random.default_rng(requests)
    b = wl.custom(rng.integers(0, 900 if requests == 3 else 30, size=requests),
                  rng.integers(1, 60 if requests == 3 else 5, size=requests), num_q_heads=4,
                  num_kv_heads=2, head_dim=128, dtype="f16", seed=63)
    case = H.make_case(b, fill="nan")
    planned, kpool, vpool = H.gpu_run(case)
    other = wl.custom(rng.integers(0, 30, size=requests), rng.integers(1, 60, size=requests),
                      num_q_heads=4, num_kv_heads=2, head_dim=128, dtype="f16", seed=64)
    kp = H.to_dev_bits(kpool.reshape(case.k_pool0.shape), b.dtype)
    vp = H.to_dev_bits(vpool.reshape(case.v_pool0.shape), b.dtype)
    q = H.to_dev_bits(case.q, b.dtype)
    table = torch.from_numpy(b.page_table).cuda()
    desc = pv.pool_desc(b.num_pages, b.num_kv_heads, b.head_dim, b.dtype)
    ws = torch.empty(pv.attn_workspace_bytes(desc, 4, b.num_reqs, b.total_q, int(b.kv_lens.max())),
                     dtype=torch.uint8, device="cuda")
    out = torch.zeros_like(q)
    plan = pv.plan_create(desc, 4, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    lists = pv.plan_device_bytes(plan)
    small = torch.empty((pv.plan_workspace_bytes(plan) + 255) // 256 * 256 + lists - 256,
                        dtype=torch.uint8, device="cuda")
    plan.destroy()
    assert (lists > 2 * 3840) == (requests == 300)

    def call(space):
        pv.multi_token_paged_attn(desc, 4, q, kp, vp, table, b.max_pages_per_req, b.ctx_lens, b.q_lens,
                                  b.q_start, b.scale, out, space)

    g = torch.cuda.CUDAGraph()
    cap = torch.cuda.Stream()
    with torch.cuda.graph(g, stream=cap):
        with pytest.raises(pv.PvError):
            call(small)
        call(ws)
    for rep in range(4):
        out.zero_()
        ws.fill_(0xA5)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(H.from_dev_bits(out), planned), rep
        H.gpu_run(H.make_case(other), one_shot=True)
        torch.cuda.synchronize()


@pytest.mark.parametrize("scale", [-0.25, 0.0, 3.0])
def test_unusual_scales(oracle, scale):
    """`scale` is any finite multiplier: negative (the kernels negate the queries), zero (uniform
    weights over the visible positions) and large (near one-hot)."""
    b = wl.custom([70, 300, 9], [1, 45, 140], num_q_heads=4, num_kv_heads=2, head_dim=64,
                  dtype="f16", seed=67, value_std=0.5)
    case = H.make_case(b, fill="nan")
    got_bits, _, _ = H.gpu_run(case, scale=scale)
    got = H.bits_to_f64(got_bits, b.dtype)
    want = oracle_out(oracle, case, scale=scale)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= H.TOL[b.dtype]


def test_long_prefill_from_empty_cache(oracle):
    """A 1500-token prompt with nothing cached (12 row tiles, causal diagonal in every one) next to
    requests that bring nothing."""
    b = wl.custom([0, 33, 0], [1500, 0, 1], num_q_heads=2, num_kv_heads=1, head_dim=128,
                  dtype="bf16", seed=71)
    check_case(oracle, H.make_case(b, fill="nan"))


def _random_batch(rng, idx):
    hkv = int(rng.choice([1, 2, 3, 5]))
    g = int(rng.choice([1, 1, 2, 4, 8, 16]))
    d = int(rng.choice([64, 128]))
    dt = str(rng.choice(["f16", "bf16"]))
    r = int(rng.integers(1, 7))
    ctx = [int(x) for x in rng.choice([0, 1, 15, 16, 17, 31, 32, 33, 100, 255, 256, 600, 1100], size=r)]
    qn = [int(x) for x in rng.choice([0, 1, 1, 2, 3, 5, 16, 17, 40, 129, 200], size=r)]
    if sum(qn) == 0:
        qn[0] = 1
    return wl.custom(ctx, qn, num_q_heads=hkv * g, num_kv_heads=hkv, head_dim=d, dtype=dt,
                     seed=1000 + idx, name=f"random{idx}")


@pytest.mark.parametrize("idx", range(24))
def test_random_batches(oracle, idx):
    """Seeded random mixes of lengths, head groupings, head sizes and dtypes: both attention
    kernels, masked/unmasked blocks, empty requests, partial pages."""
    rng = np.random.default_rng(500 + idx)
    check_case(oracle, H.make_case(_random_batch(rng, idx), fill="nan"))


def test_long_contexts_with_split_kv(oracle):
    """One generation step over 60 K cached tokens (GQA 8:1) and a 64-token prompt over 20 K
    tokens: few items, so the plan cuts the KV range into many parts for both kernels."""
    from paper_2312_05516_amd import binding as pv
    b = wl.custom([60000], [1], num_q_heads=8, num_kv_heads=1, head_dim=128, dtype="bf16", seed=83)
    desc = pv.pool_desc(b.num_pages, 1, 128, "bf16")
    plan = pv.plan_create(desc, 8, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    assert pv.plan_num_work_items(plan, 0) > 50 and pv.plan_num_work_items(plan, 2) == 1
    plan.destroy()
    check_case(oracle, H.make_case(b, fill="nan"))
    b = wl.custom([20000], [64], num_q_heads=2, num_kv_heads=1, head_dim=64, dtype="f16", seed=85)
    desc = pv.pool_desc(b.num_pages, 1, 64, "f16")
    plan = pv.plan_create(desc, 2, b.ctx_lens, b.q_lens, b.max_pages_per_req)
    pv.plan_upload(plan)
    assert pv.plan_num_work_items(plan, 1) > 20 and pv.plan_num_work_items(plan, 2) == 1
    plan.destroy()
    check_case(oracle, H.make_case(b, fill="nan"))


def test_outlier_in_a_long_work_list_is_split(oracle):
    """More than 1024 items, one of them forty times longer than the rest: the plan cuts only that
    one (both kernels: a batch of generation steps, and a mixed batch in one launch)."""
    from paper_2312_05516_amd import binding as pv
    ctx = [40 + 3 * i for i in range(135)] + [9000]
    for qn, kinds, merges in (([1] * 136, (0,), 8), ([1] * 135 + [200], (1,), 16)):
        b = wl.custom(ctx, qn, num_q_heads=8, num_kv_heads=8, head_dim=64, dtype="f16", seed=87)
        desc = pv.pool_desc(b.num_pages, 8, 64, "f16")
        plan = pv.plan_create(desc, 8, b.ctx_lens, b.q_lens, b.max_pages_per_req)
        pv.plan_upload(plan)
        for kind in (0, 1):
            n = pv.plan_num_work_items(plan, kind)
            assert (n > 1024) == (kind in kinds), (kind, n)
        assert pv.plan_num_work_items(plan, 2) == merges  # the long request's items only
        plan.destroy()
        check_case(oracle, H.make_case(b, fill="nan"))


def test_two_plans_on_two_streams(oracle):
    """Two batches launched back to back on different streams (each with its own plan, workspace
    and pools) do not disturb each other."""
    import torch
    from paper_2312_05516_amd import binding as pv
    cases, runs = [], []
    for seed, shape in ((91, ([700, 33], [1, 150])), (93, ([64, 2000, 5], [40, 1, 3]))):
        b = wl.custom(*shape, num_q_heads=8, num_kv_heads=2, head_dim=128, dtype="f16", seed=seed)
        case = H.make_case(b, fill="nan")
        desc = pv.pool_desc(b.num_pages, 2, 128, "f16")
        plan = pv.plan_create(desc, 8, b.ctx_lens, b.q_lens, b.max_pages_per_req)
        pv.plan_upload(plan)
        t = dict(plan=plan, table=torch.from_numpy(b.page_table).cuda(),
                 q=H.to_dev_bits(case.q, "f16"), kn=H.to_dev_bits(case.k_new, "f16"),
                 vn=H.to_dev_bits(case.v_new, "f16"), kp=H.to_dev_bits(case.k_pool0, "f16"),
                 vp=H.to_dev_bits(case.v_pool0, "f16"), stream=torch.cuda.Stream(),
                 ws=torch.empty(max(pv.plan_workspace_bytes(plan), 256), dtype=torch.uint8,
                                device="cuda"))
        t["out"] = torch.zeros((b.total_q, 8, 128), dtype=t["q"].dtype, device="cuda")
        cases.append(case)
        runs.append(t)
    torch.cuda.synchronize()
    for _ in range(3):
        for case, t in zip(cases, runs):
            with torch.cuda.stream(t["stream"]):
                pv.kv_append_planned(t["plan"], t["kn"], t["vn"], t["table"], t["kp"], t["vp"])
                pv.multi_token_paged_attn_planned(t["plan"], t["q"], t["kp"], t["vp"], t["table"],
                                                  case.batch.scale, t["out"], t["ws"])
    torch.cuda.synchronize()
    for case, t in zip(cases, runs):
        got = H.bits_to_f64(H.from_dev_bits(t["out"]), "f16")
        want = oracle_out(oracle, case)
        assert np.abs(got - want).max() <= H.TOL["f16"]
        assert np.array_equal(H.from_dev_bits(t["kp"]).ravel(), case.k_pool1)
        t["plan"].destroy()

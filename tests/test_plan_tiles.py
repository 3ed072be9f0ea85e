"""Which kernel a batch's long multi-token units go to (host only)."""
import pytest

from paper_2312_05516_amd import binding as pv


@pytest.mark.parametrize("heads,new,reqs,tiles", [
    ((10, 10), 365, 1, 0), ((64, 8), 188, 2, 0), ((40, 40), 700, 1, 0),
    ((40, 10), 64 * 6 + 5, 2, 0),        # 120 tiles
    ((64, 8), 32 * 22, 1, 0),            # 176 tiles
    ((64, 8), 32 * 23, 1, 184), ((64, 8), 32 * 23 + 31, 1, 184), ((64, 8), 512, 8, 1024)])
def test_few_tiles_go_to_the_128_row_kernel(monkeypatch, heads, new, reqs, tiles):
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 17, heads[1], 128, "bf16")
    plan = pv.plan_create(desc, heads[0], [20000] * reqs, [new] * reqs, 2048)
    items = [pv.plan_work_item(plan, 3, i) for i in range(pv.plan_num_work_items(plan, 3))]
    assert len({(int(i[0]), int(i[1]), int(i[2])) for i in items}) == tiles
    plan.destroy()
    # a limit set by hand still sends the tiles to the 256-row kernel
    monkeypatch.setenv("PV_TILE_MIN_KEYS", "8192")
    plan = pv.plan_create(desc, heads[0], [20000] * reqs, [new] * reqs, 2048)
    assert pv.plan_num_work_items(plan, 3) > 0
    plan.destroy()


@pytest.mark.parametrize("heads,new,ctx,tiles", [
    ((64, 8), 640, 14000, 0), ((64, 8), 640, 17000, 160),     # 2.3 and 2.8 M tile keys, 640 slots
    ((64, 8), 704, 22000, 0), ((64, 8), 704, 23000, 176),     # 4.0 and 4.2 M, 704 slots
    ((64, 8), 448, 32000, 112), ((16, 2), 64 * 8, 128000, 32), ((40, 40), 768, 60000, 120),
    ((40, 10), 64 * 6 + 20, 70000, 0),                        # 60 tiles and a rest: 4.2 M
    ((40, 10), 64 * 6 + 20, 90000, 60),                       # 5.4 M
    ((10, 10), 365, 120000, 0)])                              # 1.2 M
def test_few_tiles_over_many_keys_go_to_the_256_row_kernel(monkeypatch, heads, new, ctx, tiles):
    """Below 180 tiles what counts is tiles times keys: the merge of the 256-row kernel's parts costs
    the same over 16 K and over 120 K keys."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 20, heads[1], 128, "bf16")
    plan = pv.plan_create(desc, heads[0], [ctx], [new], 1 << 14)
    items = [pv.plan_work_item(plan, 3, i) for i in range(pv.plan_num_work_items(plan, 3))]
    assert len({(int(i[0]), int(i[1]), int(i[2])) for i in items}) == tiles
    plan.destroy()


@pytest.mark.parametrize("new,ctx,reqs,tiles", [
    (32 * 13, 12000, 20, 0), (32 * 14, 12000, 20, 0), (32 * 13, 12000, 2, 0),
    (32 * 20, 12000, 20, 0),                                  # 160 tiles, 2.0 M tile keys
    (32 * 16, 20000, 20, 128),                                # 2.6 M
    (32 * 8, 40000, 10, 0), (32 * 8, 80000, 10, 64)])         # more than half: 2.6 and 5.1 M
def test_few_tiles_beside_other_work(monkeypatch, new, ctx, reqs, tiles):
    """One long prompt beside `reqs` short ones, 64/8 heads."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 17, 8, 128, "f16")
    plan = pv.plan_create(desc, 64, [1000] * reqs + [ctx], [400] * reqs + [new], 8192)
    items = [pv.plan_work_item(plan, 3, i) for i in range(pv.plan_num_work_items(plan, 3))]
    assert len({(int(i[0]), int(i[1]), int(i[2])) for i in items}) == tiles
    assert pv.plan_num_work_items(plan, 1) > 0
    plan.destroy()


@pytest.mark.parametrize("heads,new,reqs", [
    ((8, 8, 64), 128, 32),                  # 256 items: a CU each
    ((8, 8, 64), 128 * 2 + 1, 11),          # 264
    ((64, 8, 128), 88, 8),                  # 352
    ((40, 40, 128), 700, 2), ((12, 12, 64), 500, 13),
    ((64, 8, 128), 330, 4),                 # 672
    ((64, 8, 128), 16 * 24, 4),             # 768: the last that runs at once
    ((8, 8, 64), 128, 97), ((5, 5, 64), 300, 20), ((1, 1, 128), 128, 300)])
@pytest.mark.parametrize("uneven", [False, True])
def test_items_that_run_at_once_share_the_cus_evenly(monkeypatch, heads, new, reqs, uneven):
    """Workgroup i goes to XCD i % 8, and workgroup k of an XCD to its CU k % 32."""
    for name in ("PV_XCDS", "PV_TILE_MIN_KEYS", "PV_SPLIT_TARGET"):
        monkeypatch.delenv(name, raising=False)
    group = heads[0] // heads[1]
    desc = pv.pool_desc(1 << 17, heads[1], heads[2], "f16")
    ctx = [(97 * r * r) % 1400 if uneven else 0 for r in range(reqs)]
    q = [new - (29 * r) % (new // 3) if uneven else new for r in range(reqs)]
    plan = pv.plan_create(desc, heads[0], ctx, q, 1024)
    items = [pv.plan_work_item(plan, 1, i) for i in range(pv.plan_num_work_items(plan, 1))]
    n = len(items)
    # every row of every (request, KV head) once, over all keys that it sees
    rows = [0] * reqs
    for req, _, begin, count, kv_begin, kv_end, _, parts in (map(int, i) for i in items):
        if parts == 1:
            assert kv_begin == 0 and kv_end == ctx[req] + (begin + count - 1) // group + 1
        rows[req] += (kv_end - kv_begin) * count
    for r in range(reqs):
        tiles = [(b, min(128, q[r] * group - b)) for b in range(0, q[r] * group, 128)]
        assert rows[r] == heads[1] * sum(c * (ctx[r] + (b + c - 1) // group + 1) for b, c in tiles)
    if not 256 < n <= 768 or any(int(i[7]) > 1 for i in items):
        plan.destroy()
        return
    # No CU has much more to do than one that takes as many items, beyond its longest item: the
    # longest are dealt first, each to the CU with the least.
    cost = [int(i[5] - i[4]) + 96 for i in items]
    for x in range(8):
        mine = [cost[i] for i in range(x, n, 8)]
        per_cu = [mine[c::32] for c in range(32)]
        for a in per_cu:
            for b in per_cu:
                if len(a) == len(b):
                    assert sum(a) - sum(b) <= max(a) + max(b) // 16, (x, a, b)
    plan.destroy()

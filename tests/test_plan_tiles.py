"""Which kernel a batch's long multi-token units go to (host only)."""
from fractions import Fraction

import pytest

from paper_2312_05516_amd import binding as pv

STREAMS, SCALES_SCORES = 8, 16  # of pv_plan_kernel_variants


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
    ((64, 8), 640, 20000, 0), ((64, 8), 640, 22000, 160),     # 3.3 and 3.6 M tile keys, 640 slots
    ((64, 8), 704, 32000, 0), ((64, 8), 704, 35000, 176),     # 5.8 and 6.3 M, 704 slots
    ((64, 8), 448, 32000, 112), ((16, 2), 64 * 8, 190000, 32), ((40, 40), 768, 60000, 120),
    ((40, 10), 64 * 6 + 20, 90000, 0),                        # 60 tiles and a rest: 5.4 M
    ((40, 10), 64 * 6 + 20, 120000, 60),                      # 7.2 M
    ((10, 10), 365, 120000, 0)])                              # 1.2 M
def test_few_tiles_over_many_keys_go_to_the_256_row_kernel(monkeypatch, heads, new, ctx, tiles):
    """Below 180 tiles what counts is tiles times keys: the merge of the 256-row kernel's parts costs
    the same over 16 K and over 120 K keys."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 20, heads[1], 128, "bf16")
    plan = pv.plan_create(desc, heads[0], [ctx], [new], 1 << 14)
    items = [pv.plan_work_item(plan, 3, i) for i in range(pv.plan_num_work_items(plan, 3))]
    assert len({(int(i[0]), int(i[1]), int(i[2])) for i in items}) == tiles
    assert (pv.plan_kernel_variants(plan) & SCALES_SCORES != 0) == (tiles > 0)
    plan.destroy()


@pytest.mark.parametrize("new,ctx,reqs,tiles", [
    (32 * 13, 12000, 20, 0), (32 * 14, 12000, 20, 0), (32 * 13, 12000, 2, 0),
    (32 * 20, 12000, 20, 0),                                  # 160 tiles, 2.0 M tile keys
    (32 * 16, 20000, 20, 128),                                # 2.6 M
    (32 * 8, 80000, 10, 0), (32 * 8, 112000, 10, 64)])        # more than half: 5.1 and 7.2 M
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
    cut = any(int(i[7]) > 1 for i in items)
    # lists of an item for each CU, of more than run at once, or with cut items: nothing more to hold
    exempt = reqs == 97 or (heads, new) == ((8, 8, 64), 128) or uneven and heads in (
        (8, 8, 64), (5, 5, 64), (1, 1, 128))
    assert exempt == (cut or not 256 < n <= 768), (n, cut)
    if exempt:
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


def _items(pv, plan):
    """(req, KV head, first row, rows, first key, end, part, parts) in the order of dispatch."""
    return [tuple(map(int, pv.plan_work_item(plan, 1, i)))
            for i in range(pv.plan_num_work_items(plan, 1))]


def _list_order(items):
    """The order that groups (the row tiles of one request, KV head and part) have by themselves: by
    length, each to the XCD with the least to do, the XCDs' queues in turn."""
    groups = {}
    for i in sorted(items, key=lambda i: (i[0], i[1], i[6], i[2])):
        groups.setdefault((i[0], i[1], i[6]), []).append(i)
    keys = {g: sum(i[5] - i[4] for i in v) for g, v in groups.items()}
    queues, load = [[] for _ in range(8)], [0] * 8
    for g in sorted(groups, key=lambda g: (-Fraction(keys[g], len(groups[g])), g)):
        x = load.index(min(load))
        queues[x] += groups[g]
        load[x] += keys[g]
    out, x = [], 0
    while any(queues):
        while not queues[x]:
            x = (x + 1) % 8
        out.append((x, queues[x].pop(0)))
        x = (x + 1) % 8
    return out


def _fullest(items):
    """Keys of the CU that has most to do, a set-up of 96 for each item: workgroup i goes to XCD
    i % 8, workgroup k of an XCD to its CU k % 32."""
    load = [0] * 256
    for i, it in enumerate(items):
        load[i % 8 * 32 + i // 8 % 32] += it[5] - it[4] + 96
    return max(load)


@pytest.mark.parametrize("heads,new,reqs,gain", [
    # `gain`: what dealing must take off the fullest CU at least (0: the list keeps its own order)
    ((8, 8, 64), (128, 128), 32, 0),          # 256 items: a CU each
    ((8, 8, 64), (128, 128), 97, 0),          # 776: more than run at once
    ((5, 5, 64), (80, 80), 60, 0),            # 300 of one length
    ((8, 8, 64), (1, 257), 24, 0.10), ((64, 8, 128), (60, 90), 8, 0.03),
    ((40, 40, 128), (300, 700), 2, 0.20), ((12, 12, 64), (200, 500), 13, 0.08),
    ((10, 10, 128), (30, 120), 45, 0.10), ((64, 8, 128), (16, 380), 5, 0.15),
    ((12, 12, 64), (60, 256), 35, 0.05)])
@pytest.mark.parametrize("ctx", [0, 1400])
def test_items_that_run_at_once_are_dealt_to_the_cus(monkeypatch, heads, new, reqs, gain, ctx):
    """Lists that gain nothing keep the order of the groups; in the others the fullest CU has less to
    do than in that order."""
    for name in ("PV_XCDS", "PV_TILE_MIN_KEYS", "PV_SPLIT_TARGET"):
        monkeypatch.delenv(name, raising=False)
    group = heads[0] // heads[1]
    desc = pv.pool_desc(1 << 17, heads[1], heads[2], "f16")
    # cutting is another matter: a target set by hand, which no list here is short of
    monkeypatch.setenv("PV_SPLIT_TARGET", "1")
    same = new[0] == new[1]
    c = [ctx if same else (97 * r * r) % (ctx + 1) for r in range(reqs)]
    q = [new[1] - (29 * r * r) % (new[1] - new[0] + 1) for r in range(reqs)]
    plan = pv.plan_create(desc, heads[0], c, q, 1024)
    items = _items(pv, plan)
    plan.destroy()
    want = sorted((r, h, b, min(128, q[r] * group - b), 0,
                   c[r] + (min(b + 128, q[r] * group) - 1) // group + 1, 0, 1)
                  for r in range(reqs) for h in range(heads[1])
                  for b in range(0, q[r] * group, 128))
    assert sorted(items) == want
    own = [i for _, i in _list_order(items)]
    print(f"{len(items)} items, fullest CU {_fullest(own)} -> {_fullest(items)}")
    if gain == 0:
        assert items == own
    else:
        assert 256 < len(items) <= 768
        assert _fullest(items) <= (1 - gain) * _fullest(own)


@pytest.mark.parametrize("long_new,long_reqs,short_reqs,streams", [
    (512, 4, 30, True),     # 4096 rows: full tiles only, none of which the 128-row kernel reads
    (512 + 16, 4, 30, False),  # 128 rows left of each: their K/V are read by tiles of both kernels
    (512 + 17, 4, 30, False),  # 136 rows
    (512 + 16, 4, 1, False), (512, 4, 1, True)])
def test_units_of_the_256_row_kernel_do_not_count_for_the_hint(monkeypatch, long_new, long_reqs,
                                                               short_reqs, streams):
    """Whether the 128-row kernel's items of one-tile units read their K/V with the streaming hint goes
    by the K/V that this kernel reads: 512 tiles over 30 K keys go to the other kernel."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 17, 8, 128, "bf16")
    plan = pv.plan_create(desc, 64, [30000] * long_reqs + [1000] * short_reqs,
                          [long_new] * long_reqs + [16] * short_reqs, 2048)
    tiles = {tuple(map(int, pv.plan_work_item(plan, 3, i)[:3]))
             for i in range(pv.plan_num_work_items(plan, 3))}
    assert len(tiles) == long_reqs * 8 * 16
    assert (pv.plan_kernel_variants(plan) & STREAMS != 0) == streams
    plan.destroy()


@pytest.mark.parametrize("one_tile,three_tiles,streams", [(24, 0, True), (24, 12, True),
                                                          (6, 24, False), (2, 0, False)])
def test_units_of_one_tile_stream_in_large_batches(monkeypatch, one_tile, three_tiles, streams):
    """At least a quarter of the K/V read once, and more than 96 MiB of it in all."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    reqs = one_tile + three_tiles
    plan = pv.plan_create(pv.pool_desc(1 << 14, 40, 128, "f16"), 40, [1000] * reqs,
                          [100] * one_tile + [300] * three_tiles, 128)
    assert (pv.plan_kernel_variants(plan) & STREAMS != 0) == streams
    plan.destroy()

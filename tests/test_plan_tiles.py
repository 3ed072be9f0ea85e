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


@pytest.mark.parametrize("new,reqs,tiles", [(32 * 13, 20, 0), (32 * 14, 20, 112), (32 * 13, 2, 0)])
def test_few_tiles_beside_other_work(monkeypatch, new, reqs, tiles):
    """One long prompt beside `reqs` short ones, 64/8 heads: 104 and 112 tiles."""
    monkeypatch.delenv("PV_TILE_MIN_KEYS", raising=False)
    desc = pv.pool_desc(1 << 17, 8, 128, "f16")
    plan = pv.plan_create(desc, 64, [1000] * reqs + [12000], [400] * reqs + [new], 1024)
    items = [pv.plan_work_item(plan, 3, i) for i in range(pv.plan_num_work_items(plan, 3))]
    assert len({(int(i[0]), int(i[1]), int(i[2])) for i in items}) == tiles
    assert pv.plan_num_work_items(plan, 1) > 0
    plan.destroy()

"""Workgroups that change places from round to round of tiles (tensors of twelve rounds and more): every tile is
taken exactly once, whatever the last round is short of.  Host only: the index map walks the tiles the way a
launch of 96 workgroups does and fails on a tile that is missed or taken twice."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B


@pytest.mark.parametrize("rows,turns", [(12 * 96 * 16, 88), (12 * 96 * 16 + 1, 88), (13 * 96 * 16 - 16, 88), (20 * 96 * 16 + 95 * 16, 88),
                                        (12 * 96 * 16 - 16, 88), (11 * 96 * 16 + 1, 88), (11 * 96 * 16, 0)])
@pytest.mark.parametrize("kw", [dict(), dict(grid_mode=-1), dict(grid_mode=1), dict(grid_mode=3)],
                         ids=lambda k: "-".join("%s%s" % x for x in k.items()) or "default")
def test_every_tile_once_when_workgroups_change_places(rows, turns, kw):
    for elem in (4, 8):
        dims, perm = (16, rows), (1, 0)                         # a single counter of rows / 16 tiles, and more
        plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_TILED, m=1, tile_in=16, k=1, tile_out=16, vec2=1, align_out=1, **kw)
        assert plan.describe().num_tiles == -(-rows // 16)
        assert B.tperm_plan_launch_info(plan, workgroups=96).turns == turns
        ref = oracle.transpose(np.arange(16 * rows, dtype=np.int64), dims, perm)
        assert np.array_equal(B.tperm_plan_index_map(plan), ref)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("dims,perm,m,tile_in,k,tile_out,turns", [
    ((4, 9, 11, 108, 13), (4, 1, 0, 2, 3), 2, 5, 2, 5, 88),      # counters 2 and 1188: gcd(96, 2376) = 24
    ((9, 4, 6, 5, 70), (3, 1, 4, 2, 0), 1, 5, 1, 2, 0),          # 2 and 3: gcd(96, 6) = 6 is below 8
])
def test_every_tile_once_under_counters_in_step_with_the_grid(dims, perm, m, tile_in, k, tile_out, turns, elem):
    plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=m, tile_in=tile_in, k=k, tile_out=tile_out, align_out=1,
                                  vec2=1)
    assert plan.describe().num_tiles >= 12 * 96
    assert B.tperm_plan_launch_info(plan, workgroups=96).turns == turns
    ref = oracle.transpose(np.arange(int(np.prod(dims)), dtype=np.int64), dims, perm)
    assert np.array_equal(B.tperm_plan_index_map(plan), ref)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("slots", [1, 2, 3, 4, 6, 24])
def test_launches_that_keep_places_run_without_the_code_for_turns(slots, elem):
    """Up to four slots, below twelve rounds.  Not row copies, which never had that code; 24 slots of 8 bytes keep
    their places at any number of rounds, and so do small tensors of 6 to 16 slots, which run without masks."""
    def info(tiles, kind=B.KERNEL_TILED, **kw):
        plan = B.tperm_plan_create_ex((16, 16 * slots * tiles), (1, 0), elem, kernel_class=kind, m=1, tile_in=16, k=1, tile_out=16 * slots,
                                      **{**dict(align_out=1, vec2=1, loads_first=1), **kw})
        assert plan.describe().nreg == slots
        i = B.tperm_plan_launch_info(plan, workgroups=256)
        return i.turns, i.steady
    assert info(11 * 256) == (0, int(slots <= 4))
    assert info(11 * 256 + 1) == ((0, 0) if slots == 6 or (slots, elem) == (24, 8) else (88, 0))
    assert info(40 * 256) == ((0, 0) if (slots, elem) == (24, 8) else (88, 0))      # 6 slots: above 40 MB, with masks
    row = B.tperm_plan_create((512 * 16, 3, 100), (0, 2, 1), elem)
    assert row.describe().kernel_class == B.KERNEL_ROWCOPY and B.tperm_plan_launch_info(row, workgroups=256).steady == 0

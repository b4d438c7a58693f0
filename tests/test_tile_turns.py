"""Workgroups that change places from round to round of tiles (tensors of twelve rounds and more): every tile is
taken exactly once, whatever the last round is short of.  Host only: the index map walks the tiles the way a
launch of 96 workgroups does and fails on a tile that is missed or taken twice."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B


@pytest.mark.parametrize("rows", [12 * 96 * 16, 12 * 96 * 16 + 1, 13 * 96 * 16 - 16, 20 * 96 * 16 + 95 * 16, 12 * 96 * 16 - 16])
@pytest.mark.parametrize("kw", [dict(), dict(grid_mode=-1), dict(grid_mode=1), dict(grid_mode=3), dict(cache_policy=2)],
                         ids=lambda k: "-".join("%s%s" % x for x in k.items()) or "default")
def test_every_tile_once_when_workgroups_change_places(rows, kw):
    for elem in (4, 8):
        dims, perm = (16, rows), (1, 0)                         # a single counter of rows / 16 tiles, and more
        tile_out = 128 // elem if kw.get("align_out") == 2 else 16
        plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_TILED, m=1, tile_in=16, k=1, tile_out=tile_out, vec2=1,
                                      **{**dict(align_out=1), **kw})
        assert plan.describe().num_tiles == -(-rows // tile_out)
        ref = oracle.transpose(np.arange(16 * rows, dtype=np.int64), dims, perm)
        assert np.array_equal(B.tperm_plan_index_map(plan), ref)


@pytest.mark.parametrize("elem", [4, 8])
def test_every_tile_once_under_counters_in_step_with_the_grid(elem):
    dims, perm = (9, 4, 6, 5, 70), (3, 1, 4, 2, 0)
    plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=5, k=1, tile_out=2, align_out=1)
    assert plan.describe().num_tiles >= 12 * 96
    ref = oracle.transpose(np.arange(int(np.prod(dims)), dtype=np.int64), dims, perm)
    assert np.array_equal(B.tperm_plan_index_map(plan), ref)

"""Rules of the planner that depend on a size, on both sides of their lines, and the binding's
argument arrays.  Host only."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B


@pytest.mark.parametrize("d0,d1,elem,policy", [
    (256, 248, 8, 3), (256, 264, 8, 2),                            # 512 KiB lies at 256 x 256 elements of 8 bytes
    (512, 240, 4, 3), (512, 272, 4, 2), (1024, 2040, 8, 2), (2048, 2032, 4, 2),
])
def test_cached_loads_below_512_kib(d0, d1, elem, policy):
    """Line-aligned input rows, output rows on 64-byte boundaries."""
    info = B.tperm_plan_create_ex((d0, d1), (1, 0), elem, kernel_class=B.KERNEL_TILED, m=1, tile_in=128 // elem, k=1,
                                  tile_out=64, align_out=1, vec2=1).describe()
    assert info.cache_policy == policy, B.info_dict(info)
    # line-aligned on both sides: nontemporal loads at any size
    assert B.tperm_plan_create((512, 512), (1, 0), 8).describe().cache_policy == 2


@pytest.mark.parametrize("dims,perm,nreg,vec2,align_out", [
    # above 320 MB tiles of 24 single elements displace neither pairs and windows nor smaller tiles (measured,
    # us with them / with 24 slots: 971 / 1177, 364 / 457, 218 / 234, 335 / 368, 697 / 846)
    ((479, 2315, 525), (2, 0, 1), 12, 1, 1), ((42, 1142, 4617), (2, 1, 0), 12, 1, 1), ((407012, 310), (1, 0), 8, 1, 0),
    ((21, 6, 70, 9, 37, 76), (2, 0, 1, 5, 3, 4), 12, 1, 0), ((6861, 155, 371), (2, 0, 1), 16, 0, 0),
    # below they are taken (68 -> 54 us), and 32 slots at any size (301 -> 267 us)
    ((15, 12, 38, 5, 8, 19, 6), (5, 4, 1, 6, 3, 0, 2), 24, 0, 0), ((231, 23, 62, 11, 37), (3, 1, 4, 2, 0), 32, 0, 0),
])
def test_many_slots_of_single_elements(dims, perm, nreg, vec2, align_out):
    info = B.tperm_plan_create(dims, perm, 4).describe()
    assert (info.nreg, info.vec2, info.align_out) == (nreg, vec2, align_out), B.info_dict(info)


@pytest.mark.parametrize("elem,nreg,mb,form", [
    (4, 12, 39, 1), (4, 12, 41, 0), (8, 12, 39, 1), (8, 12, 41, 0),
    # 24 slots of 4-byte elements: masks cost 2 to 19 % on average below the line, save 2 % above it (23 % at most)
    (4, 24, 639, 3), (4, 24, 641, 2), (8, 24, 641, 3), (4, 32, 641, 3), (8, 32, 641, 3),
])
def test_form_without_masks_by_slots_and_size(elem, nreg, mb, form):
    t0, t1 = {12: (61, 50), 24: (77, 79), 32: (89, 71)}[nreg]
    info = B.tperm_plan_create_ex((t0, t1, mb * 1_000_000 // elem // (t0 * t1)), (1, 0, 2), elem, kernel_class=B.KERNEL_PACKED,
                                  m=1, tile_in=t0, k=1, tile_out=t1, vec2=1).describe()
    assert info.nreg == nreg and info.without_masks == form


@pytest.mark.parametrize("pad", [-1, 0, 1])
@pytest.mark.parametrize("elem", [4, 8])
def test_index_maps_of_the_slot_counts_without_masks(elem, pad):
    """Tiles of 6 to 32 slots per thread with edges on both split dims: the map of positions stays
    inside the tensors and inside the LDS image, and no element lies on the place that slots beyond
    the tile write (the map fails if one does)."""
    for t0, t1 in ((48, 32), (61, 25), (64, 64), (77, 79), (89, 71)):
        dims, perm = (2 * t0 - 1, 3, t1 + 1), (2, 0, 1)
        plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1, vec2=1,
                                      align_out=1, lds_buffers=2, lds_pad=pad)
        ref = oracle.transpose(np.arange(int(np.prod(dims)), dtype=np.int64), dims, perm)
        assert np.array_equal(B.tperm_plan_index_map(plan), ref)


@pytest.mark.parametrize("elem", [4, 8])
def test_lds_image_holds_the_tile_and_its_padding_only(elem):
    """One more element only where slots beyond the tile need a place to write and the rows have no
    padding: not for tiles that fill their slots, padded rows, pairs, windows or 64 threads."""
    def lds_bytes(t0, t1, pad, **kw):
        kw = {**dict(vec2=1, align_out=1, lds_buffers=2), **kw}
        dims = (2 * t0, 3, 2 * t1)
        return B.tperm_plan_create_ex(dims, (2, 0, 1), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1,
                                      lds_pad=pad, pair_elems=1, **kw).describe().lds_bytes
    assert lds_bytes(64, 64, 0) == 64 * 64 * elem          # two images of 8-byte elements: 64 KiB, and no more
    assert lds_bytes(61, 50, 0) == (61 * 50 + 1) * elem
    assert lds_bytes(61, 50, 1) == 62 * 50 * elem
    assert lds_bytes(60, 50, 0, vec2=2) == 60 * 50 * elem
    assert lds_bytes(61, 32, 0, align_out=2) == 61 * (32 + 128 // elem) * elem
    assert lds_bytes(30, 50, 0, threads=64) == 30 * 50 * elem


def test_argument_arrays_are_taken_by_value():
    dims = [6, 5, 4]
    a = B.tperm_plan_create(dims, [2, 0, 1], 8)
    dims[0] = 7                                            # a list changed after the call names another problem
    b = B.tperm_plan_create(dims, np.array([2, 0, 1]), 8)
    c = B.tperm_plan_create(tuple(np.array([6, 5, 4])), (2, 0, 1), 8)
    assert [B.tperm_plan_describe(p).volume for p in (a, b, c)] == [120, 140, 120]
    for bad in ([6, 5, 0], []):
        with pytest.raises((B.TpermError, ValueError)):
            B.tperm_plan_create(bad, [2, 0, 1] if len(bad) != 0 else [], 8)
    with pytest.raises(TypeError):
        B.tperm_plan_create(iter((6, 5, 4)), (2, 0, 1), 8)


@pytest.mark.parametrize("n,tile_in,workgroups", [
    (1279, 16, 4), (1281, 16, 8),        # tiles of 2 KiB, eight to a compute unit: four below 2.5 rounds of 2048
    (959, 32, 4), (961, 32, 5),          # tiles of 4 KiB, five: four below 1.5 rounds of 1280
])
def test_workgroups_of_small_tensors(n, tile_in, workgroups):
    info = B.tperm_plan_create_ex((32, 32, n), (1, 0, 2), 8, kernel_class=B.KERNEL_TILED, m=1, tile_in=tile_in, k=1,
                                  tile_out=16, align_out=1, vec2=1).describe()
    assert info.blocks_per_cu == workgroups, B.info_dict(info)


@pytest.mark.parametrize("elem", [4, 8])
def test_a_launch_asks_for_the_lds_of_the_kernel_that_runs(elem):
    """A tile of 3 x 5 x 333 elements: its tables are larger than its image of 4-byte elements.  Loads first has no kernel
    with tables, so such a launch asks for the image alone; accumulation runs stores first, with tables."""
    def plan(**kw):
        return B.tperm_plan_create_ex((2, 3, 700, 5), (2, 1, 3, 0), elem, kernel_class=B.KERNEL_PACKED, m=2, tile_in=3, k=1, tile_out=333,
                                      align_out=1, vec2=1, pair_elems=1, **kw)
    p = plan(loads_first=1)
    image = p.describe().lds_bytes
    info, acc = (B.tperm_plan_launch_info(p, accumulate=a) for a in (False, True))
    assert info.tables == acc.tables == 1 and info.lds_bytes == acc.lds_bytes >= image
    assert info.lds_bytes > image or elem == 8
    p = plan(loads_first=2)
    info, acc = (B.tperm_plan_launch_info(p, accumulate=a) for a in (False, True))
    assert (info.tables, info.lds_bytes) == (0, image) and acc.tables == 1
    assert acc.lds_bytes > image or elem == 8
    assert B.tperm_plan_launch_info(plan(lds_buffers=2, loads_first=2)).lds_bytes == 2 * image
    with pytest.raises(B.TpermError):
        B.tperm_plan_launch_info(B.tperm_plan_create((8, 8), (0, 1), elem))    # a copy has no tiles
    with pytest.raises(B.TpermError):
        B.tperm_plan_launch_info(B.tperm_plan_create_ex((64, 640), (1, 0), elem, vec2=2, align_out=1, tile_in=32, tile_out=32, m=1, k=1,
                                                        kernel_class=B.KERNEL_TILED), accumulate=True)


@pytest.mark.parametrize("tile_out,slots", [(9, 6), (37, 24), (43, 32)])
@pytest.mark.parametrize("elem", [4, 8])
def test_accumulating_32_slots_of_4_byte_elements_take_no_tables(tile_out, slots, elem):
    """They lose 8 % by them (up to 22); every other count and the 8-byte form keep theirs."""
    plan = B.tperm_plan_create_ex((31, 16, 7, 5, 2 * tile_out - 1), (4, 3, 0, 2, 1), elem, kernel_class=B.KERNEL_PACKED, m=2, tile_in=5,
                                  k=1, tile_out=tile_out, align_out=1, vec2=1, pair_elems=1)
    assert plan.describe().nreg == slots
    for acc in (False, True):
        assert B.tperm_plan_launch_info(plan, accumulate=acc).tables == int(not (acc and elem == 4 and slots == 32))


@pytest.mark.parametrize("elem,t0,t1,align_out,slots", [(4, 128, 64, 1, 16), (8, 64, 90, 1, 12), (4, 64, 96, 2, 16)])
def test_largest_tiles_of_pairs_have_16_slots(elem, t0, t1, align_out, slots):
    """A tile has at most 8192 elements, with the halo of line-aligned windows; larger slot counts are not instantiated for pairs."""
    def info(t1):
        return B.tperm_plan_create_ex((3 * t0, 5, 4 * t1), (2, 1, 0), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1,
                                      align_out=align_out, vec2=2).describe()
    i = info(t1)
    assert (i.nreg, i.vec2, i.align_out) == (slots, 1, align_out - 1)
    with pytest.raises(B.TpermError):
        info(t1 + 32)

"""Positions inside a tile taken from tables (tiles of three dims and more with four slots per thread and more,
of four dims and more with three): tiles of three to five dims on both sides of that line, edges on either split dim and on both,
tables of one dim against the rest either way, pairs, every slot count with several tiles per workgroup (the image goes where
the tables were).  Bit-exact against the CPU oracle (the largest tensors: against torch's permute), with guard bands."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B
from paper_1705_01598_amd import workloads as wl

torch = pytest.importorskip("torch")
from gpu_util import GuardedOut, np_uint, to_device  # noqa: E402

# dims, perm, m, tile_in, k, tile_out, positions from tables (256 threads, single elements)
CASES = [
    ((9, 5, 14, 6, 13), (3, 1, 4, 0, 2), 2, 5, 3, 5, 1),           # 9 x 5 x 6 x 5: 6 slots of four dims
    ((9, 5, 14, 6, 13), (4, 1, 3, 0, 2), 3, 3, 1, 4, 1),           # 9 x 5 x 3 x 4: 3 slots of four
    ((17, 9, 5, 37), (3, 0, 2, 1), 2, 8, 1, 7, 1),                 # 17 x 8 x 7: 4 slots of three
    ((17, 7, 5, 37), (3, 0, 2, 1), 2, 6, 1, 7, 0),                 # 17 x 6 x 7: 3 slots of three: dim by dim
    ((3, 5, 2, 7, 4, 31, 3), (4, 1, 5, 2, 6, 0, 3), 4, 6, 3, 9, 1),  # 3 x 5 x 2 x 6 x 4 x 9: 26 slots of six
    ((311, 3, 3, 8), (3, 2, 1, 0), 1, 140, 3, 2, 1),               # one long dim and three short ones
    ((2, 3, 700, 5), (2, 1, 3, 0), 2, 3, 1, 333, 1),               # one long dim behind two short ones
]

# Pairs: even extents and even tile extents along input dim 0 and output dim 0, edges on one split dim and on both
PAIRS = [
    ((14, 9, 21, 6, 26), (3, 1, 4, 0, 2), 2, 5, 3, 4, 1),          # 14 x 9 x 6 x 4: 6 slots of four dims
    ((10, 7, 14, 6, 26), (4, 1, 3, 0, 2), 3, 4, 1, 6, 1),          # 10 x 7 x 4 x 6: 4 slots of four
    ((14, 9, 210, 6, 26), (3, 1, 4, 0, 2), 2, 5, 3, 4, 1),         # several tiles per workgroup
]

# Several tiles per workgroup: slots, and the dims of a tensor whose tiles take them.  Thirteen rounds of one workgroup per compute
# unit, an edge along dim 1; the last in several rounds only
MANY = [(4, (31, 16003, 6)), (5, (31, 41603, 8)), (6, (31, 16003, 9)), (8, (31, 16003, 12)), (10, (31, 41603, 15)), (12, (31, 41603, 17)),
        (14, (31, 16003, 21)), (16, (31, 16003, 25)), (24, (31, 16003, 37)), (32, (31, 16003, 43)), (3, (9, 5, 14, 60, 13))]


def _plan(case, elem, **kw):
    dims, perm, m, tin, k, tout = case[:6]
    return B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=m, tile_in=tin, k=k, tile_out=tout, align_out=1,
                                  pair_elems=1, **kw)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("case", CASES + PAIRS, ids=lambda c: "x".join(map(str, c[0])))
def test_tables_agree_with_the_positions_dim_by_dim(case, elem):
    """The index map of a plan with tables fails unless every pair of entries adds up to its position."""
    for vec2 in (1, 2):
        plan = _plan(case, elem, vec2=vec2)
        assert plan.describe().vec2 == int(vec2 == 2 and case in PAIRS)
        assert B.tperm_plan_launch_info(plan).tables == case[6]
        ref = oracle.transpose(np.arange(int(np.prod(case[0])), dtype=np.int64), case[0], case[1])
        assert np.array_equal(B.tperm_plan_index_map(plan), ref)


def test_forms_without_tables():
    for kw in (dict(large=1), dict(loads_first=2), dict(threads=64)):
        assert B.tperm_plan_launch_info(_plan(CASES[0], 4, vec2=1, **kw)).tables == 0


@pytest.mark.gpu
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("case", CASES + PAIRS, ids=lambda c: "x".join(map(str, c[0])))
def test_tiles_with_positions_from_tables(case, elem):
    dims, perm = case[0], case[1]
    wcase = wl.make_case(0, 93, dims, perm, elem)
    a = wl.bitpattern_values(wcase)
    ref = oracle.transpose(a, dims, perm)
    ftype = np.float64 if elem == 8 else np.float32
    stream = torch.cuda.current_stream().cuda_stream
    for kw in (dict(), dict(vec2=2), dict(large=1), dict(loads_first=2), dict(lds_buffers=2, cache_policy=2), dict(threads=64)):
        try:
            plan = _plan(case, elem, **kw)
        except B.TpermError as e:
            assert e.status == B.ERR_KERNEL and kw.get("threads") == 64     # tile too large for one wavefront
            continue
        a_dev, out = to_device(a), GuardedOut(wcase.volume, elem)
        B.tperm_execute(plan, a_dev.data_ptr(), out.ptr, stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), ref), (dims, kw)
        assert out.guards_intact()
    rng = np.random.default_rng(7)
    x, y = (rng.standard_normal(wcase.volume).astype(ftype) for _ in range(2))
    x_dev, out = to_device(x), GuardedOut(wcase.volume, elem)
    out.view().copy_(to_device(y))
    B.tperm_execute_accumulate(_plan(case, elem, vec2=1), x_dev.data_ptr(), out.ptr, stream)
    torch.cuda.synchronize()
    assert np.array_equal(np_uint(out.view().cpu().numpy()), np_uint(y + oracle.transpose(x, dims, perm)))
    assert out.guards_intact()


@pytest.mark.gpu
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("slots,dims", MANY, ids=lambda x: str(x) if isinstance(x, int) else "")
def test_several_tiles_per_workgroup(slots, dims, elem):
    grid = torch.cuda.get_device_properties(0).multi_processor_count
    case = (dims, (2, 1, 0), 2, 5, 1, dims[2]) if len(dims) == 3 else (dims, CASES[1][1], 3, 3, 1, 4)
    perm = case[1]
    a = wl.bitpattern_values(wl.make_case(0, 95, dims, perm, elem))
    ref = oracle.transpose(a, dims, perm)
    a_dev = to_device(a)
    stream = torch.cuda.current_stream().cuda_stream
    for kw in (dict(), dict(lds_buffers=2, cache_policy=2), dict(cache_policy=3), dict(cache_policy=4)):
        plan = _plan(case, elem, vec2=1, blocks_per_cu=1, **kw)
        info, launch = plan.describe(), B.tperm_plan_launch_info(plan, workgroups=grid)
        assert info.nreg == slots and info.num_tiles > 2 * grid and launch.tables == 1
        if slots > 3:                              # 16 and 24 slots of 8 bytes keep their places, and small tensors of 6 to 16 slots
            assert (launch.turns == 0) == ((elem == 8 and slots in (16, 24)) or (slots <= 16 and info.without_masks & 1 == 1))
        out = GuardedOut(a.size, elem)
        for _ in range(2):
            B.tperm_execute(plan, a_dev.data_ptr(), out.ptr, stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), ref), kw
        assert out.guards_intact()
    rng = np.random.default_rng(slots)
    x, y = (rng.standard_normal(a.size).astype(np.float64 if elem == 8 else np.float32) for _ in range(2))
    ref = np_uint(y + oracle.transpose(x, dims, perm))
    x_dev = to_device(x)
    for policy in (1, 2):
        out = GuardedOut(a.size, elem)
        out.view().copy_(to_device(y))
        B.tperm_execute_accumulate(_plan(case, elem, vec2=1, blocks_per_cu=1, cache_policy=policy), x_dev.data_ptr(), out.ptr, stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), ref), policy
        assert out.guards_intact()


@pytest.mark.gpu
@pytest.mark.parametrize("dims,perm,slots,masks", [
    ((231, 23, 62, 11, 37), (3, 1, 4, 2, 0), 32, 3),                # the plan as selected
    ((31, 140803, 37), (2, 1, 0), 24, 2),                     # 24 slots above 640 MB: with masks
    ((31, 139203, 37), (2, 1, 0), 24, 3),
])
def test_large_tensors_of_24_and_32_slots(dims, perm, slots, masks):
    plan = B.tperm_plan_create(dims, perm, 4) if slots == 32 else _plan((dims, perm, 2, 5, 1, dims[2]), 4, vec2=1)
    info = plan.describe()
    assert (info.nreg, info.vec2, info.without_masks) == (slots, 0, masks)
    assert [B.tperm_plan_launch_info(plan, accumulate=a).tables for a in (False, True)] == [1, int(slots == 24)]
    n = int(np.prod(dims))
    moved = lambda t: t.reshape(dims[::-1]).permute([len(dims) - 1 - perm[len(dims) - 1 - i] for i in range(len(dims))]).reshape(-1)  # noqa: E731
    a = torch.arange(n, dtype=torch.int64, device="cuda").mul_(-1640531527).to(torch.int32)     # every element its own value
    stream = torch.cuda.current_stream().cuda_stream
    out = GuardedOut(n, 4)
    B.tperm_execute(plan, a.data_ptr(), out.ptr, stream)
    torch.cuda.synchronize()
    assert torch.equal(out.view(), moved(a)) and out.guards_intact()
    x = torch.empty(n, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=torch.Generator(device="cuda").manual_seed(5))
    y = a.to(torch.float32)
    ref = y + moved(x)
    B.tperm_execute_accumulate(plan, x.data_ptr(), y.data_ptr(), stream)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int32), ref.view(torch.int32))

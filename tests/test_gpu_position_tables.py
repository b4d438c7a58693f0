"""Positions inside a tile taken from tables (tiles of three dims and more with four slots per thread and more,
of four dims and more with three): tiles of three to five dims on both sides of that line, edges on either split dim and on both,
tables of one dim against the rest either way.  Bit-exact against the CPU oracle, with guard bands."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B
from paper_1705_01598_amd import workloads as wl

torch = pytest.importorskip("torch")
from gpu_util import GuardedOut, np_uint, to_device  # noqa: E402

# dims, perm, m, tile_in, k, tile_out, slots * (dims - 1) with 256 threads and single elements
CASES = [
    ((9, 5, 14, 6, 13), (3, 1, 4, 0, 2), 2, 5, 3, 5, 18),           # 9 x 5 x 6 x 5: 6 slots of four dims
    ((9, 5, 14, 6, 13), (4, 1, 3, 0, 2), 3, 3, 1, 4, 9),            # 9 x 5 x 3 x 4: 3 slots of four
    ((17, 9, 5, 37), (3, 0, 2, 1), 2, 8, 1, 7, 8),                  # 17 x 8 x 7: 4 slots of three
    ((17, 7, 5, 37), (3, 0, 2, 1), 2, 6, 1, 7, 6),                  # 17 x 6 x 7: 3 slots of three: dim by dim
    ((3, 5, 2, 7, 4, 31, 3), (4, 1, 5, 2, 6, 0, 3), 4, 6, 3, 9, 130),  # 3 x 5 x 2 x 6 x 4 x 9: 26 slots of six
    ((311, 3, 3, 8), (3, 2, 1, 0), 1, 140, 3, 2, 81),               # one long dim and three short ones
    ((2, 3, 700, 5), (2, 1, 3, 0), 2, 3, 1, 333, 16),               # one long dim behind two short ones
]


def _plan(case, elem, **kw):
    dims, perm, m, tin, k, tout, _ = case
    return B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=m, tile_in=tin, k=k, tile_out=tout, align_out=1,
                                  pair_elems=1, **kw)


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
def test_tables_agree_with_the_positions_dim_by_dim(case, elem):
    """The index map of a plan with tables fails unless every pair of entries adds up to its position."""
    for vec2 in (1, 2):
        plan = _plan(case, elem, vec2=vec2)
        info = plan.describe()
        if case[6] and not info.vec2:
            n = sum(t > 1 for t in B.info_dict(info)["tile"])
            assert -(-info.tile_volume // 256) * (n - 1) == case[6]
        ref = oracle.transpose(np.arange(int(np.prod(case[0])), dtype=np.int64), case[0], case[1])
        assert np.array_equal(B.tperm_plan_index_map(plan), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
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

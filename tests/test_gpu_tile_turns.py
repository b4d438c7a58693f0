"""Kernels with and without the code by which workgroups change places from round to round of tiles: one to four slots per
thread in every form that has both, launches just below and above twelve rounds.  Bit-exact against the CPU oracle, with
guard bands."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B
from paper_1705_01598_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_util import GuardedOut, np_uint, to_device  # noqa: E402

FORMS = [dict(), dict(cache_policy=2), dict(cache_policy=3), dict(cache_policy=4), dict(loads_first=2), dict(vec2=2), dict(vec2=2, cache_policy=2)]


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("slots", [1, 2, 3, 4])
@pytest.mark.parametrize("turning", [False, True])
def test_both_kernels_of_a_form(slots, elem, turning):
    grid = torch.cuda.get_device_properties(0).multi_processor_count       # one workgroup per compute unit
    stream = torch.cuda.current_stream().cuda_stream
    rng = np.random.default_rng(slots + elem)
    for kw in FORMS:
        pairs = 2 if kw.get("vec2") else 1
        width = 16 * slots * pairs
        dims, perm = (16, width * (11 * grid + 5 * turning) - 2 * turning), (1, 0)   # the last tile is short of two
        plan = B.tperm_plan_create_ex(dims, perm, elem, kernel_class=B.KERNEL_TILED, m=1, tile_in=16, k=1, tile_out=width, blocks_per_cu=1,
                                      **{**dict(align_out=1, vec2=1), **kw})
        info = plan.describe()
        assert (info.nreg, info.vec2) == (slots, pairs - 1)
        launch = B.tperm_plan_launch_info(plan, workgroups=grid)
        assert (launch.turns, launch.steady) == ((88, 0) if turning else (0, 1))
        a = wl.bitpattern_values(wl.make_case(0, 97, dims, perm, elem))
        ref = oracle.transpose(a, dims, perm)
        a_dev, out = to_device(a), GuardedOut(a.size, elem)
        for _ in range(2):
            B.tperm_execute(plan, a_dev.data_ptr(), out.ptr, stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), ref), kw
        assert out.guards_intact()
        if kw.get("vec2") or kw.get("cache_policy", 2) != 2:
            continue
        x, y = (rng.standard_normal(a.size).astype(np.float64 if elem == 8 else np.float32) for _ in range(2))
        assert B.tperm_plan_launch_info(plan, accumulate=True, workgroups=grid).steady == int(not turning)
        x_dev, out = to_device(x), GuardedOut(a.size, elem)
        out.view().copy_(to_device(y))
        B.tperm_execute_accumulate(plan, x_dev.data_ptr(), out.ptr, stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), np_uint(y + oracle.transpose(x, dims, perm)))
        assert out.guards_intact()

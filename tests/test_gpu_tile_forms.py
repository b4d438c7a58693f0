"""Forms of the tile kernel that a rule on size picks, at the sizes where they can go wrong: tiles
that exactly fill their slots and tiles one element short, edges of the tensor on either split dim
and on both, one tile for the whole tensor.  Every test asserts which form ran.  Bit-exact against
the CPU oracle, with guard bands."""
import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import binding as B
from paper_1705_01598_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from gpu_util import GuardedOut, np_uint, to_device  # noqa: E402


def _run(dims, perm, elem, **kw):
    case = wl.make_case(0, 91, dims, perm, elem)
    a = wl.bitpattern_values(case)
    plan = B.tperm_plan_create_ex(dims, perm, elem, **kw)
    a_dev, out = to_device(a), GuardedOut(case.volume, elem)
    B.tperm_execute(plan, a_dev.data_ptr(), out.ptr, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(np_uint(out.view().cpu().numpy()), oracle.transpose(a, dims, perm)), B.info_dict(plan.describe())
    assert out.guards_intact()
    return plan.describe()


# tile of t0 x t1 elements; slots per thread the kernel is instantiated for: 6, 8, 12, 16, 24, 32
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("t0,t1,nreg", [(48, 32, 6), (61, 25, 6), (64, 32, 8), (43, 43, 8), (48, 64, 12), (61, 50, 12),
                                        (64, 64, 16), (63, 65, 16), (96, 64, 24), (77, 79, 24), (89, 71, 32)])
def test_form_without_masks_on_small_tensors(t0, t1, nreg, elem):
    for i, (d0, d1) in enumerate([(t0, t1), (2 * t0, 3 * t1), (3 * t0 + 1, 2 * t1), (2 * t0, 2 * t1 - 1), (2 * t0 - 1, t1 + 1)]):
        info = _run((d0, 3, d1), (2, 0, 1) if i % 2 else (2, 1, 0), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1,
                    tile_out=t1, vec2=1, align_out=1, cache_policy=1 + i % 4, lds_buffers=1 + i % 2, lds_pad=(0, 0, -1, -1, 1)[i],
                    loads_first=1,
                    window_in=(0, 2)[i % 2], window_out=(0, 3)[i // 2 % 2])
        assert info.nreg == nreg and info.loads_first == 0 and info.without_masks & 1


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("t0,t1,nreg", [(48, 32, 6), (61, 50, 12)])
def test_masked_form_where_loads_go_first(t0, t1, nreg, elem):
    """The order with the loads first exists with masks only."""
    info = _run((2 * t0 - 1, 3, t1 + 1), (2, 0, 1), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1,
                vec2=1, align_out=1, loads_first=2)
    assert info.nreg == nreg and info.loads_first == 1 and info.without_masks == 0


@pytest.mark.parametrize("policy", [1, 2, 3, 4])
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("t0,t1,nreg", [(61, 50, 12), (77, 79, 24), (89, 71, 32)])
def test_form_of_large_tensors(t0, t1, nreg, elem, policy):
    """The kernels that address every tile from its own origin."""
    for dims, perm in (((2 * t0 - 1, 3, t1 + 1), (2, 0, 1)), ((t0 + 1, 3, 2 * t1 - 1), (2, 1, 0))):
        info = _run(dims, perm, elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1, vec2=1, align_out=1,
                    large=1, cache_policy=policy, lds_pad=0)
        assert info.nreg == nreg and info.large == 1
        assert info.without_masks == (3 if nreg == 32 or (nreg, elem) == (24, 8) else 0)


@pytest.mark.parametrize("elem,t0,t1,nreg,line", [(4, 61, 50, 12, 40_000_000), (8, 61, 50, 12, 40_000_000), (4, 77, 79, 24, 640_000_000)])
def test_both_sides_of_the_small_tensor_lines(elem, t0, t1, nreg, line):
    """The same tile just below and just above the size where the form changes."""
    for more, form in ((0, 1), (1, 0)):
        info = _run((t0, t1, line // elem // (t0 * t1) + more), (1, 0, 2), elem, kernel_class=B.KERNEL_PACKED, m=1,
                    tile_in=t0, k=1, tile_out=t1, vec2=1)
        assert info.nreg == nreg and info.without_masks & 1 == form


@pytest.mark.parametrize("large", [0, 1])
@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("policy", [1, 2, 3, 4])
def test_accumulation_under_every_cache_policy(policy, elem, large):
    """Staged tiles with edges on both sides, few slots and as many as the form without masks takes, and
    the LDS-free row copy, at output pointers on and off a sector boundary (which changes the policy
    of the kernel that runs)."""
    ftype = np.float64 if elem == 8 else np.float32
    tile = lambda t0, t1: dict(kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1, align_out=1)  # noqa: E731
    for dims, perm, kw, nreg in [((70, 45, 33), (2, 0, 1), tile(33, 16), 3), ((64, 40, 48), (1, 2, 0), tile(32, 40), 6),
                                 ((153, 3, 80), (2, 0, 1), tile(77, 79), 24), ((90, 3, 141), (2, 1, 0), tile(89, 71), 32),
                                 ((96, 3, 128), (2, 1, 0), tile(96, 64), 24),
                                 ((48, 21, 34), (0, 2, 1), {} if large else dict(kernel_class=B.KERNEL_ROWCOPY), 0)]:
        vol = int(np.prod(dims))
        rng = np.random.default_rng(vol + policy)
        a, b = (rng.standard_normal(vol).astype(ftype) for _ in range(2))
        for offset in (0, 1):
            plan = B.tperm_plan_create_ex(dims, perm, elem, cache_policy=policy, large=large, vec2=1, pair_elems=1, **kw)
            info = plan.describe()
            assert nreg == 0 or (info.nreg == nreg and info.without_masks & 2 == (2 if nreg == 32 or (nreg == 24 and (elem == 8 or not large)) else 0))
            a_dev, out = to_device(a), GuardedOut(vol, elem, offset)
            out.view().copy_(to_device(b))
            B.tperm_execute_accumulate(plan, a_dev.data_ptr(), out.ptr, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            ref = b + oracle.transpose(a, dims, perm)      # one IEEE addition per element: exact
            assert np.array_equal(np_uint(out.view().cpu().numpy()), np_uint(ref)), (dims, perm, offset)
            assert out.guards_intact()


@pytest.mark.parametrize("elem", [4, 8])
@pytest.mark.parametrize("t0,t1,nreg", [(56, 32, 7), (58, 29, 7), (64, 40, 10), (47, 49, 10), (64, 56, 14), (59, 60, 14)])
def test_slot_counts_between_the_powers(t0, t1, nreg, elem):
    """7, 10 and 14 slots, filled to the last and with the last few empty: without masks, with masks and the loads
    first, for large tensors, in line-aligned windows and accumulating, with edges on either dim and on both."""
    ftype = np.float64 if elem == 8 else np.float32
    tile = dict(kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1, vec2=1, align_out=1)
    for i, (d0, d1) in enumerate([(t0, t1), (3 * t0 + 1, 2 * t1), (2 * t0, 2 * t1 - 1), (2 * t0 - 1, t1 + 1)]):
        dims, perm = (d0, 3, d1), (2, 0, 1) if i % 2 else (2, 1, 0)
        for policy in (1, 2, 3, 4):
            info = _run(dims, perm, elem, **tile, cache_policy=policy, lds_buffers=1 + i % 2, lds_pad=(0, -1, -1, 1)[i], loads_first=1)
            assert info.nreg == nreg and info.without_masks & 1 and info.large == 0
            info = _run(dims, perm, elem, **tile, cache_policy=policy, large=1)
            assert info.nreg == nreg and info.large == 1
        info = _run(dims, perm, elem, **tile, loads_first=2)
        assert info.nreg == nreg and info.loads_first == 1
        plan = B.tperm_plan_create_ex(dims, perm, elem, **tile)
        vol = d0 * 3 * d1
        rng = np.random.default_rng(vol)
        a, b = (rng.standard_normal(vol).astype(ftype) for _ in range(2))
        a_dev, out = to_device(a), GuardedOut(vol, elem)
        out.view().copy_(to_device(b))
        B.tperm_execute_accumulate(plan, a_dev.data_ptr(), out.ptr, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(np_uint(out.view().cpu().numpy()), np_uint(b + oracle.transpose(a, dims, perm)))
        assert out.guards_intact()


@pytest.mark.parametrize("elem,t0,t1,nreg", [(4, 28, 32, 7), (4, 24, 64, 10), (4, 39, 32, 10), (4, 56, 32, 14),
                                             (8, 56, 16, 7), (8, 47, 32, 10), (8, 55, 48, 14)])
def test_windows_of_the_slot_counts_between(elem, t0, t1, nreg):
    """Windows read a line more along the output run than they write."""
    line = 128 // elem
    for d1 in (5 * line + 5, 2 * t1 + 1):
        for policy in (1, 2, 3, 4):
            info = _run((3 * t0 + 1, 3, d1), (2, 0, 1), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=t0, k=1, tile_out=t1,
                        vec2=1, align_out=2, cache_policy=policy)
            assert info.align_out == 1 and info.nreg == nreg


@pytest.mark.parametrize("elem", [4, 8])
def test_five_slots_from_the_size_of_masked_forms_on(elem):
    for mb, nreg in ((39, 6), (41, 5)):
        info = _run((61, 20, mb * 1_000_000 // elem // (61 * 20)), (1, 0, 2), elem, kernel_class=B.KERNEL_PACKED, m=1, tile_in=61,
                    k=1, tile_out=20, vec2=1)
        assert info.nreg == nreg

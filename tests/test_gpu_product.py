"""Matrix product added into a permuted tensor (tperm_product_accumulate).

Reference: the product in float64, laid out by torch's permute.  Bound per element: K products, each
rounded in the working precision (unit roundoff eps), summed in any order with one rounding per step,
err <= 2 K eps sum_k |l||r| (the standard bound for recursive summation, K eps to first order, doubled
for the higher orders and for products that are not fused), plus the roundings of the final addition
and of the reference, 2 eps (|ref| + sum_k |l||r|)."""
import math

import pytest

from paper_1705_01598_amd import binding as B

# (left dims, right dims, perm, K): tiles are 128 x 32 (fp64) and 128 x 64 (fp32); thin ones 16 x 128,
# 16 x 256, 256 x 16.  dims count from the stride-1 one, left first.
CASES = [
    ((128,), (64,), (0, 1), 16),
    ((127,), (65,), (0, 1), 15),               # odd edges, odd runs
    ((129,), (31,), (1, 0), 17),               # the right operand is the fast one
    ((4, 33), (6, 11), (0, 2, 1, 3), 33),      # runs of 4, digits interleaved
    ((6, 22), (5, 13), (0, 3, 2, 1), 48),      # runs of 2
    ((8, 8, 4), (27, 3), (0, 1, 3, 2, 4), 70),
    ((3, 50), (7, 40), (3, 0, 1, 2), 1),
    ((5,), (700,), (0, 1), 300),               # few fast indices
    ((16,), (9, 60), (0, 2, 1), 40),
    ((17,), (300,), (0, 1), 500),
    ((600,), (3,), (0, 1), 129),               # few slow indices
    ((64, 9), (16,), (0, 2, 1), 24),
    ((605,), (3,), (0, 1), 20),
    ((602,), (5,), (0, 1), 31),
    ((40,), (24,), (1, 0), 4096),              # the summed index in pieces
    ((8,), (9,), (0, 1), 5003),
    ((300,), (70,), (0, 1), 1000),
    ((1,), (100,), (1, 0), 20),
    ((150, 40), (30, 25), (2, 0, 3, 1), 24),   # many tiles to a workgroup
    ((130,), (7, 6), (2, 1, 0), 20),           # the stride-1 dimension is not the first one of its operand
    ((9, 20), (33,), (1, 0, 2), 35),
    ((5,), (3, 400), (2, 0, 1), 18),
]
GUARD = 64


def _operand(torch, mat, k_first, offset):
    """mat (n x K, double, on the host) in memory as the call wants it, `offset` elements into a buffer."""
    flat = (mat if k_first else mat.t()).contiguous().reshape(-1)
    buf = torch.full((flat.numel() + offset,), float("nan"), dtype=mat.dtype)
    buf[offset:] = flat
    return buf


def _run(torch, left, right, perm, k, dtype, lk, rk, offset=0, values=None):
    m, n = math.prod(left), math.prod(right)
    gen = torch.Generator().manual_seed(m * 1000 + n + k)
    rand = lambda *s: torch.rand(*s, generator=gen, dtype=torch.float64).mul_(2).sub_(1).to(dtype)  # noqa: E731
    l, r, d = (rand(m, k), rand(n, k), rand(m * n)) if values is None else values(rand)
    dims = list(left) + list(right)
    prod = B.tperm_product_create(dims, perm, len(left), k, d.element_size(), lk, rk)
    info = B.tperm_product_describe(prod)
    ls, rs = (_operand(torch, x, f, offset).cuda() for x, f in ((l, lk), (r, rk)))
    out = torch.full((m * n + 2 * GUARD + offset,), 7.0, dtype=dtype)
    lo = GUARD + offset
    out[lo:lo + m * n] = d
    out = out.cuda()
    ws = torch.full((max(1, info.workspace_bytes // d.element_size()),), float("nan"), dtype=dtype, device="cuda")
    esz = d.element_size()
    B.tperm_product_accumulate(prod, ls.data_ptr() + offset * esz, rs.data_ptr() + offset * esz, out.data_ptr() + lo * esz,
                               torch.cuda.current_stream().cuda_stream, ws.data_ptr(), info.workspace_bytes)
    torch.cuda.synchronize()
    out = out.cpu()
    assert bool((out[:lo] == 7.0).all()) and bool((out[lo + m * n:] == 7.0).all()), "wrote outside the destination"

    def arranged(t):                                     # (m x n) -> flat destination order
        rank = len(dims)
        axes = [rank - 1 - perm[rank - 1 - i] for i in range(rank)]
        return t.t().reshape(tuple(reversed(dims))).permute(axes).reshape(-1)
    ld, rd = l.double(), r.double()
    ref = d.double() + arranged(ld @ rd.t())
    size = arranged(ld.abs() @ rd.abs().t())
    return info, out[lo:lo + m * n], ref, size


def _check(torch, got, ref, size, k, dtype):
    eps = torch.finfo(dtype).eps
    err = (got.double() - ref).abs()
    bound = 2 * k * eps * size + 2 * eps * (ref.abs() + size)
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("left,right,perm,k", CASES)
def test_product_matches_the_reference(left, right, perm, k, dtype_name):
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    for lk, rk, offset in ((0, 0, 0), (0, 1, 1), (1, 0, 0), (1, 1, 3)):
        _, got, ref, size = _run(torch, left, right, perm, k, dtype, lk, rk, offset)
        _check(torch, got, ref, size, k, dtype)


def test_the_cases_reach_every_form():
    seen = set()
    for elem in (8, 4):
        for left, right, perm, k in CASES:
            i = B.tperm_product_describe(B.tperm_product_create(left + right, perm, len(left), k, elem))
            seen.add((elem, i.shape, i.vec if i.pieces == 1 else 0))
    # (element, shape, neighbours moved together; 0: in pieces)
    need = {(8, 0, 1), (8, 0, 2), (8, 0, 0), (8, 1, 1), (8, 1, 0)}
    need |= {(4, 0, v) for v in (0, 1, 2, 4)} | {(4, 1, v) for v in (0, 1)} | {(4, 2, v) for v in (0, 1, 2, 4)}
    assert need <= seen, need - seen


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
def test_large_destination(dtype_name):
    """More than 128 MiB: nontemporal accesses to the destination."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    elem = torch.finfo(dtype).bits // 8
    left, right, perm, k = (8, 8, 61), (27, 40 * 8 // elem), (0, 1, 3, 2, 4), 5
    left = (8, 8, 61 * 4)
    info, got, ref, size = _run(torch, left, right, perm, k, dtype, 0, 0)
    assert math.prod(left) * math.prod(right) * elem > 128 << 20
    _check(torch, got, ref, size, k, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("lines,extra,offset", [(1, 0, 0), (1, 0, 3), (3, 0, 0), (1, 1, 0), (0, 3, 0), (0, 2, 0)])
def test_large_destination_in_runs(lines, extra, offset, dtype_name):
    """More than 128 MiB in runs of whole lines (nontemporal accesses from an aligned pointer, else cached) and
    of other lengths (cached), wide tiles and thin ones, both layouts of the fast operand."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    elem = torch.finfo(dtype).bits // 8
    run = lines * 128 // elem + extra
    for slow, k, lk in ((45, 5, 0), (13, 3, 1)):
        mid = (136 << 20) // elem // run // slow // 3 + 1
        info, got, ref, size = _run(torch, (run, 3, mid), (slow,), (0, 2, 3, 1), k, dtype, lk, 0, offset)
        assert got.numel() * elem > 128 << 20 and info.pieces == 1
        _check(torch, got, ref, size, k, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
def test_special_values(dtype_name):
    """Subnormal products are not flushed; an infinity or a NaN reaches its own row or column only."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    tiny = torch.finfo(dtype).tiny / 1024

    def small(rand):
        return ((rand(50, 13) * 8).round().to(dtype) * tiny, (rand(21, 13) * 4).round().to(dtype), torch.zeros(50 * 21, dtype=dtype))
    _, got, ref, _ = _run(torch, (50,), (21,), (1, 0), 13, dtype, 0, 0, values=small)
    assert torch.equal(got, ref.to(dtype))            # multiples of tiny: every sum is exact
    assert bool((got != 0).any())

    def odd(rand):
        l, r, d = rand(130, 9), rand(40, 9), rand(130 * 40)
        l[129, 8], r[39, 0] = float("inf"), float("nan")
        return l, r, d
    _, got, ref, _ = _run(torch, (130,), (40,), (0, 1), 9, dtype, 0, 0, values=odd)
    assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("left,right,perm,k", [c for c in CASES if c[3] > 16])
def test_whole_numbers_are_exact(left, right, perm, k, dtype_name):
    """Whole numbers of -2 to 2: every sum is below 2^24 and exact in either type, in any order, so that a summed
    index that is left out or taken twice (at the edge of a stage or of a piece) shows."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)

    def whole(rand):
        n, m = math.prod(right), math.prod(left)
        return tuple((rand(*s) * 2.49).round() for s in ((m, k), (n, k), (m * n,)))
    for lk, rk, offset in ((0, 0, 1), (0, 1, 0), (1, 0, 3), (1, 1, 0)):
        _, got, ref, size = _run(torch, left, right, perm, k, dtype, lk, rk, offset, values=whole)
        assert float(size.max()) < 1 << 24 and torch.equal(got.double(), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("left,right,perm,k", [((131,), (37,), (0, 1), 41), ((37,), (131,), (1, 0), 50), ((13,), (301,), (0, 1), 43),
                                               ((301,), (13,), (0, 1), 35), ((40,), (24,), (1, 0), 4096), ((300,), (70,), (0, 1), 1003)])
def test_special_values_behind_a_vector(left, right, perm, k, dtype_name):
    """Infinities and NaN where loads of several elements run past the end of a row (they fetch the start of the
    next one), in the last stage and at the edges of pieces, in either layout: the rows and columns that hold
    them, and no other, are infinite or NaN."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    inf, nan = float("inf"), float("nan")

    def odd(rand):
        l, r, d = rand(*left, k), rand(*right, k), rand(left[0] * right[0])
        l[0, 1::7], l[1, 5], l[left[0] - 1, k - 1] = nan, inf, inf
        r[0, 2::5], r[2, k - 1], r[right[0] - 1, 0] = nan, -inf, inf
        return l, r, d
    for lk, rk in ((0, 0), (0, 1), (1, 0), (1, 1)):
        info, got, ref, _ = _run(torch, left, right, perm, k, dtype, lk, rk, values=odd)
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf()) and (info.pieces > 1) == (k > 1000)
        assert torch.equal(got[got.isinf()].sign(), ref[ref.isinf()].sign().to(dtype)) and bool(got.isfinite().any())


@pytest.mark.parametrize("dims,perm,left,left_fast", [
    ((1024, 64, 64), (2, 1, 0), 1, 0), ((64, 64, 1024), (1, 0, 2), 2, 1), ((5, 3, 400), (2, 0, 1), 1, 0),   # not its first dimension
    ((5, 1, 7), (1, 0, 2), 1, 1), ((1, 5, 7), (0, 2, 1), 1, 0), ((5, 7), (1, 0), 1, 0), ((5, 7), (0, 1), 1, 1),  # extents of 1 do not count
    ((4, 5), (1, 0), 2, 1), ((4, 5), (1, 0), 0, 0), ((1, 1), (1, 0), 1, 1)])
def test_the_fast_operand_owns_the_stride_1_dimension(dims, perm, left, left_fast):
    for elem in (4, 8):
        info = B.tperm_product_describe(B.tperm_product_create(dims, perm, left, 30, elem))
        assert info.left_fast == left_fast


def test_arguments():
    make = B.tperm_product_create
    for bad, status in ((dict(left_dims=3), B.ERR_RANK), (dict(left_dims=-1), B.ERR_RANK), (dict(k=0), B.ERR_DIMS),
                        (dict(elem_size=2), B.ERR_ELEM_SIZE), (dict(perm=(0, 0)), B.ERR_PERM), (dict(dims=(0, 4)), B.ERR_DIMS),
                        (dict(dims=(1 << 15, 1 << 15)), B.ERR_TOO_LARGE), (dict(k=1 << 28), B.ERR_TOO_LARGE)):
        args = dict(dims=(5, 4), perm=(1, 0), left_dims=1, k=3, elem_size=8)
        args.update(bad)
        with pytest.raises(B.TpermError) as e:
            make(**args)
        assert e.value.status == status, bad
    p = make((5, 4), (1, 0), 1, 3, 8)
    for ptrs, status in (((0, 8, 4096), B.ERR_NULL), ((4096, 0, 8), B.ERR_NULL), ((4100, 8192, 16384), B.ERR_ALIGN),
                         ((4096, 8192, 4096 + 8), B.ERR_ALIAS), ((4096, 8192, 8192 - 8), B.ERR_ALIAS)):
        with pytest.raises(B.TpermError) as e:
            B.tperm_product_accumulate(p, *ptrs)
        assert e.value.status == status, ptrs
    p = make((40, 24), (1, 0), 1, 4096, 8)                     # in pieces: wants a workspace
    need = B.tperm_product_describe(p).workspace_bytes
    assert need > 0
    base = 1 << 30
    for ws, n, status in ((0, 0, B.ERR_NULL), (4 * base, need - 1, B.ERR_TOO_LARGE), (4 * base + 4, need, B.ERR_ALIGN),
                          (base, need, B.ERR_ALIAS), (3 * base, need, B.ERR_ALIAS)):
        with pytest.raises(B.TpermError) as e:
            B.tperm_product_accumulate(p, base, 2 * base, 3 * base, 0, ws, n)
        assert e.value.status == status, (ws, n)


def test_which_contractions_run_in_one_kernel():
    pays = lambda m, n, k, elem: B.tperm_product_describe(B.tperm_product_create((m, n), (1, 0), 1, k, elem)).pays  # noqa: E731
    for elem in (4, 8):
        assert pays(11264, 1728, 70, elem) and pays(64, 100000, 256, elem)
    assert not pays(64, 8085, 2048, 4)                         # 83 us against 60
    assert pays(80, 64, 115620, 8)                             # the library's product runs along the summed index


@pytest.mark.parametrize("elem", [4, 8])
def test_orders_in_which_one_kernel_does_not_pay(elem):
    pays = lambda dims, perm, left, k=30: B.tperm_product_describe(B.tperm_product_create(dims, perm, left, k, elem)).pays  # noqa: E731
    # the stride-1 dimension is not the first of its operand: lanes 512 and more bytes apart
    assert not pays((1024, 64, 64), (2, 1, 0), 1) and not pays((64, 64, 1024), (1, 0, 2), 2)
    assert pays((1024, 64, 64), (1, 2, 0), 1) and pays((64, 64, 1024), (0, 1, 2), 2)
    # short runs: an operand whose dimensions are listed in another order than the destination's
    short, long_ = 32 // elem, 64 // elem
    n = (8 << 20) // elem // short // 30 + 1
    assert pays((short, n, 6, 5), (0, 2, 3, 1), 2) and pays((short, n, 6, 5), (0, 2, 1, 3), 2)
    assert not pays((short, n, 6, 5), (0, 3, 2, 1), 2)
    assert not pays((short, 6, n, 5), (0, 3, 2, 1), 3)
    assert pays((short, n - 1, 6, 5), (0, 3, 2, 1), 2)         # up to 8 MiB
    assert pays((long_, n, 6, 5), (0, 3, 2, 1), 2)


def test_small_fp64_products_that_fill_the_librarys_tiles():
    pays = lambda m, n, k, elem: B.tperm_product_describe(B.tperm_product_create((m, n), (0, 1), 1, k, elem)).pays  # noqa: E731
    assert not pays(297, 1579, 186, 8) and not pays(617, 703, 1046, 8)    # 18.0 us against 21.3, 30.2 against 36.4
    assert pays(297, 1579, 186, 4) and pays(149, 1579, 186, 8)


@pytest.mark.gpu
@pytest.mark.parametrize("library", [False, True])
@pytest.mark.parametrize("d,l,r,ext", [("ab", "ak", "kb", dict(a=24, k=24, b=24)),      # operands in place
                                       ("acb", "akc", "kb", dict(a=6, c=5, b=24, k=24)),  # one transposed first
                                       ("bca", "kac", "kb", dict(a=6, c=5, b=24, k=24))])
def test_contraction_whose_operand_is_its_destination(d, l, r, ext, library):
    """d += l r with d in place of l: the operand is read, or the product finished, before d changes."""
    torch = pytest.importorskip("torch")
    from paper_1705_01598_amd.contraction import Contraction
    con = Contraction(d, l, r, ext, torch.float64)
    if library:
        con._product = None
    g = torch.Generator(device="cuda").manual_seed(4)
    size = lambda s: math.prod(ext[c] for c in s)  # noqa: E731
    x, y = (torch.rand(size(s), dtype=torch.float64, device="cuda", generator=g) for s in (l, r))
    # row-major views of column-major data: labels in reverse
    view = lambda t, s: t.cpu().reshape([ext[c] for c in reversed(s)])  # noqa: E731
    prod = torch.einsum(f"{l[::-1]},{r[::-1]}->{d[::-1]}", view(x, l), view(y, r))
    want = view(x, d) + prod
    t = {}
    con.run(x, y, x, t)
    err = (view(x, d) - want).abs()
    assert bool((err <= 2 * 24 * 2.3e-16 * want).all()), float((err / want).max())     # all terms are positive
    assert set(t) == {"transpose_l_ms", "transpose_r_ms", "gemm_ms", "transpose_d_ms", "total_ms"}

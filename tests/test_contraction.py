"""Tensor contraction through transposes + product (application layer on top of the library).

The checker is the oracle's direct loop nest (oracle.contract: one output element at a time,
products summed in double precision in a fixed order; pinned in test_oracle_pins.py on a
hand-computed case, the matrix product, nested Python loops and the transpose oracle).
CPU part: the label bookkeeping is checked by emulating the four steps with the oracle's
transposes and numpy's matrix product.  GPU part: both real paths (tperm transposes, then the
product that is added straight into the destination, or the vendor GEMM through torch.mm and an
accumulating transpose) against the oracle; a product sums in another order than the loop
nest, so this comparison has a tolerance, unlike every transpose test: with K
products per output element, each rounded in the working precision (unit roundoff eps), the
error of either summation order is at most about K * eps * sum_k |l||r| (the standard bound
for recursive summation), so |difference| <= 2 * 8 * K * eps * sum_k |l||r| + 8 * eps * |ref|
per output element (factor 8: slack for fused multiply-adds and blocked partial sums)."""
import math

import numpy as np
import pytest

import oracle
from paper_1705_01598_amd import contraction as C
from paper_1705_01598_amd import workloads as wl

SMALL = [
    ("ab", "ak", "kb", dict(a=5, b=7, k=3)),                       # plain matrix product
    ("ba", "ak", "kb", dict(a=5, b=7, k=3)),                       # transposed result
    ("abef", "abcd", "cdef", dict(a=3, b=4, c=2, d=5, e=3, f=2)),  # no transposes needed
    ("ebfa", "cadb", "fdce", dict(a=3, b=4, c=2, d=5, e=3, f=2)),  # all four steps permute
    ("cab", "bkc", "ak", dict(a=4, b=3, c=5, k=6)),
]


def _oracle_ref(lay, l, r, d):
    """d + l * r by the oracle's loop nest (first label = stride-1 dimension)."""
    return oracle.contract(lay.d_labels, lay.l_labels, lay.r_labels, dict(lay.extents), l, r, d)


@pytest.mark.parametrize("d,l,r,ext", SMALL)
def test_layout_bookkeeping_reproduces_the_oracle(d, l, r, ext):
    lay = C.layout(d, l, r, ext)
    rng = np.random.default_rng(3)
    lv = rng.standard_normal(math.prod(lay.dims(l)))
    rv = rng.standard_normal(math.prod(lay.dims(r)))
    dv = rng.standard_normal(math.prod(lay.dims(d)))
    lp = oracle.transpose(lv, lay.dims(l), lay.l_perm)                 # (free_l, summed): m x k
    rp = oracle.transpose(rv, lay.dims(r), lay.r_perm)                 # (summed, free_r): k x n
    t = (lp.reshape((lay.m, lay.k), order="F") @ rp.reshape((lay.k, lay.n), order="F")).ravel(order="F")
    got = oracle.transpose_accumulate(t, dv, lay.dims(lay.free_l + lay.free_r), lay.t_perm)
    assert np.allclose(got, _oracle_ref(lay, lv, rv, dv), rtol=1e-12, atol=1e-12)
    assert lay.flops == 2 * lay.m * lay.n * lay.k


def test_layout_rejects_bad_specifications():
    for d, l, r in [("ab", "ak", "kk"), ("ab", "ak", "jb"), ("abk", "ak", "kb"), ("ab", "akc", "kb"), ("ab", "ab", "ab")]:
        with pytest.raises(ValueError):
            C.layout(d, l, r, dict(a=2, b=2, c=2, j=2, k=2))
    with pytest.raises(ValueError):
        C.layout("ab", "ak", "kb", dict(a=2, b=2))


def test_arithmetic_intensity_formula():
    lay = C.layout("ab", "ak", "kb", dict(a=100, b=100, k=100))
    assert lay.arithmetic_intensity == pytest.approx(2 * math.sqrt(1e12) / 3e4)
    for case in wl.contraction_cases():
        lay = C.layout(case["d"], case["l"], case["r"], case["extents"])
        assert max(len(case["d"]), len(case["l"]), len(case["r"])) <= 8
        assert max(lay.m * lay.n, lay.m * lay.k, lay.k * lay.n) < 1 << 26


def test_operands_that_the_library_product_has_to_see():
    """An operand that is used in place reaches the one kernel by its address alone: what torch keeps beside
    the memory (lazy negation, gradients of either mode) and what overlaps the destination goes to torch.mm."""
    torch = pytest.importorskip("torch")
    from torch.autograd import forward_ad
    con = C.Contraction("ab", "ak", "kb", dict(a=6, k=6, b=6), torch.float64, "cpu")
    assert con._product is not None and all(perm is None for perm, _ in con._operands)
    both = lambda x: {con._in_one_kernel(x, y, d), con._in_one_kernel(y, x, d)}  # noqa: E731
    mem = torch.rand(120, dtype=torch.float64)
    x, y, d = mem[:36], torch.rand(36, dtype=torch.float64), torch.zeros(36, dtype=torch.float64)
    assert both(x) == {True}
    assert both(torch._neg_view(x)) == {False}
    grad = x.clone().requires_grad_()
    assert both(grad) == {False}
    with torch.no_grad():
        assert both(grad) == {True}
    with forward_ad.dual_level():
        assert both(x) == {True} and both(forward_ad.make_dual(x, y)) == {False}
    assert con._in_one_kernel(x, y, mem[35:71]) is False and con._in_one_kernel(x, y, mem[36:72]) is True
    one = C.Contraction("ab", "ak", "kb", dict(a=1, k=1, b=1), torch.float64, "cpu")
    z = torch.ones(1, dtype=torch.complex128).conj().imag              # negated lazily, one element: contiguous
    assert z.is_contiguous() and not one._in_one_kernel(z, y[:1], d[:1])


@pytest.mark.gpu
def test_gpu_contraction_of_lazily_negated_operands():
    torch = pytest.importorskip("torch")
    g = torch.Generator(device="cuda").manual_seed(6)
    x, y = (torch.rand(36, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    d = torch.ones(36, dtype=torch.float64, device="cuda")
    C.Contraction("ab", "ak", "kb", dict(a=6, k=6, b=6), torch.float64).run(torch._neg_view(x), y, d)
    want = 1 - y.view(6, 6) @ x.view(6, 6)                             # row-major views of column-major data
    assert torch.allclose(d.view(6, 6), want, rtol=1e-13, atol=1e-14)


MORE = [
    ("ebfa", "cadb", "fdce", dict(a=30, b=14, c=12, d=9, e=20, f=16)),
    ("dabfec", "aghcbi", "efdghi", dict(a=4, b=6, c=5, d=3, e=4, f=3, g=7, h=2, i=5)),
]


def _against_the_oracle(con, dtype):
    torch = pytest.importorskip("torch")
    lay = con.lay
    rng = np.random.default_rng(5)
    npdt = np.float64 if dtype == torch.float64 else np.float32
    values = lambda labels: (rng.random(math.prod(lay.dims(labels))) * 2 - 1).astype(npdt)  # noqa: E731
    lv, rv, dv = values(lay.l_labels), values(lay.r_labels), values(lay.d_labels)
    d_dev = torch.from_numpy(dv.copy()).cuda()
    con.run(torch.from_numpy(lv).cuda(), torch.from_numpy(rv).cuda(), d_dev)
    con.run(torch.from_numpy(lv).cuda(), torch.from_numpy(rv).cuda(), d_dev)      # accumulates twice
    torch.cuda.synchronize()
    l64, r64 = lv.astype(np.float64), rv.astype(np.float64)
    ref = _oracle_ref(lay, l64, r64, _oracle_ref(lay, l64, r64, dv.astype(np.float64)))
    bound = _oracle_ref(lay, np.abs(l64), np.abs(r64), np.zeros_like(ref))         # sum_k |l||r|
    eps = np.finfo(npdt).eps
    err = np.abs(d_dev.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= 2 * 8 * lay.k * eps * bound + 8 * eps * np.abs(ref) + 1e-300), float(err.max())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("d,l,r,ext", SMALL + MORE)
def test_gpu_contraction_matches_the_oracle(d, l, r, ext, dtype_name):
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    con = C.Contraction(d, l, r, ext, dtype)
    assert con._product is not None
    _against_the_oracle(con, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name", ["float64", "float32"])
@pytest.mark.parametrize("d,l,r,ext", SMALL + MORE)
def test_gpu_library_path_matches_the_oracle(d, l, r, ext, dtype_name):
    """The library product and the accumulating transpose, where the plan would take the one kernel."""
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    con = C.Contraction(d, l, r, ext, dtype)
    con._product = None                       # the library path's buffers are made by the first call
    _against_the_oracle(con, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype_name,d,l,r,ext", [
    ("float64", "bcad", "akb", "dkc", dict(a=33, b=9, c=20, d=79, k=186)),        # 297 x 1580, in pieces: the library is faster
    ("float32", "cab", "bkla", "klc", dict(a=21, b=41, c=1344, k=32, l=16)),       # 861 x 1344, K = 512
])
def test_gpu_contraction_that_takes_the_library_path(d, l, r, ext, dtype_name):
    torch = pytest.importorskip("torch")
    dtype = getattr(torch, dtype_name)
    con = C.Contraction(d, l, r, ext, dtype)
    assert con._product is None
    _against_the_oracle(con, dtype)


@pytest.mark.gpu
def test_gpu_benchmark_names_the_path_of_every_row(monkeypatch, capsys):
    """Figures of the one kernel (which has no time of the product alone, and two transposes) and of the library
    path stand under names of their own; --library measures the latter everywhere."""
    import json
    pytest.importorskip("torch")
    cases = [dict(name=str(i), seed=i, d="bcad", l="akb", r="dkc", extents=dict(a=33, b=9, c=20, d=79, k=k)) for i, k in enumerate((186, 30))]
    monkeypatch.setattr(wl, "contraction_cases", lambda: cases)
    for argv, paths in ((["--reps", "1"], ["library", "one kernel"]), (["--reps", "1", "--library"], ["library", "library"])):
        C._bench(argv)
        lines = [json.loads(x) for x in capsys.readouterr().out.splitlines()]
        rows, summaries = lines[:2], lines[2:]
        assert [x["path"] for x in rows] == paths and [x["path"] for x in summaries] == sorted(set(paths))
        for x in rows:
            assert ("gemm_gflops" in x, "transpose_share" in x, "transpose_d_ms" in x) == (x["path"] == "library",) * 3
            assert ("product_gflops" in x, "operand_transpose_share" in x, "product_ms" in x) == (x["path"] == "one kernel",) * 3
        assert sum(x["cases"] for x in summaries) == 2

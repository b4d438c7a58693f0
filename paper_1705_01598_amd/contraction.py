"""Tensor contraction D += L * R through transposes and one product (application layer).

The use the paper makes of its transpose library (Section 3.4: the indirect, "transpose -
transpose - GEMM - transpose" implementation of a binary tensor contraction): the left input is
brought to the layout (uncontracted dims, contracted dims), the right input to (contracted dims,
uncontracted dims), a matrix product gives the result in the layout (left uncontracted, right
uncontracted), and that is transposed and accumulated into the destination.  The first two
transposes run through the tperm library.  The last two steps are one kernel of it, which adds the
product straight into the destination (``tperm_product_accumulate``), where its plan says that pays;
else, and for operands it does not take, the product is the vendor GEMM reached through ``torch.mm``
(hipBLASLt / rocBLAS) and the last step ``tperm_execute_accumulate``.  Everything here is argument
bookkeeping around those.

Conventions as everywhere in this package: a tensor is a flat buffer, the FIRST label / extent
is the stride-1 dimension.  A contraction is given by three label strings, e.g.
``D="abef", L="abcd", R="cdef"``: labels shared by L and R and absent from D are summed over; every
other label must occur in D and in exactly one of L, R.
"""
from __future__ import annotations

import math
from dataclasses import dataclass
from typing import Dict, List, Sequence, Tuple


@dataclass(frozen=True)
class ContractionLayout:
    """Index bookkeeping of one contraction (pure host logic, no GPU needed)."""
    d_labels: str
    l_labels: str
    r_labels: str
    extents: Tuple[Tuple[str, int], ...]
    free_l: str          # uncontracted labels of L, in D's order
    free_r: str          # uncontracted labels of R, in D's order
    summed: str          # contracted labels, in L's order
    l_perm: Tuple[int, ...]   # gather permutation L -> (free_l, summed)
    r_perm: Tuple[int, ...]   # gather permutation R -> (summed, free_r)
    t_perm: Tuple[int, ...]   # gather permutation (free_l, free_r) -> D
    m: int
    n: int
    k: int

    def dims(self, labels: str) -> Tuple[int, ...]:
        e = dict(self.extents)
        return tuple(e[c] for c in labels)

    @property
    def flops(self) -> int:
        return 2 * self.m * self.n * self.k

    @property
    def arithmetic_intensity(self) -> float:
        """2 sqrt(vol(D) vol(L) vol(R)) / (vol(D) + vol(L) + vol(R)), the paper's measure."""
        vd, vl, vr = self.m * self.n, self.m * self.k, self.k * self.n
        return 2.0 * math.sqrt(float(vd) * vl * vr) / (vd + vl + vr)


def layout(d_labels: str, l_labels: str, r_labels: str, extents: Dict[str, int]) -> ContractionLayout:
    """Work out which labels are summed and the three gather permutations."""
    for s in (d_labels, l_labels, r_labels):
        if len(set(s)) != len(s):
            raise ValueError(f"repeated label in '{s}'")
        for c in s:
            if c not in extents or int(extents[c]) < 1:
                raise ValueError(f"label '{c}' has no positive extent")
    summed = "".join(c for c in l_labels if c in r_labels)
    if any(c in d_labels for c in summed):
        raise ValueError("a label shared by both inputs must not occur in the result")
    free_l = "".join(c for c in d_labels if c in l_labels)
    free_r = "".join(c for c in d_labels if c in r_labels)
    if len(free_l) + len(free_r) != len(d_labels):
        raise ValueError("every result label must come from exactly one input")
    if set(free_l) | set(summed) != set(l_labels) or set(free_r) | set(summed) != set(r_labels):
        raise ValueError("every input label must be summed or occur in the result")
    if not summed:
        raise ValueError("nothing to sum over")
    l_target, r_target, t_labels = free_l + summed, summed + free_r, free_l + free_r
    e = {c: int(extents[c]) for c in set(d_labels + l_labels + r_labels)}
    prod = lambda s: math.prod(e[c] for c in s)
    return ContractionLayout(
        d_labels, l_labels, r_labels, tuple(sorted(e.items())), free_l, free_r, summed,
        tuple(l_labels.index(c) for c in l_target), tuple(r_labels.index(c) for c in r_target),
        tuple(t_labels.index(c) for c in d_labels), prod(free_l), prod(free_r), prod(summed))


class Contraction:
    """A planned contraction, workspace included: transposes that bring the operands to matrix layout,
    then a product that is added straight into the destination (``tperm_product_accumulate``), or,
    where that is expected to be slower, a library product and an accumulating transpose."""

    def __init__(self, d_labels: str, l_labels: str, r_labels: str, extents: Dict[str, int], dtype, device="cuda"):
        import torch
        from torch.autograd.forward_ad import unpack_dual
        from . import binding as B
        self._torch, self._B, self._unpack_dual = torch, B, unpack_dual
        self.lay = layout(d_labels, l_labels, r_labels, extents)
        if dtype not in (torch.float32, torch.float64):
            raise ValueError("float32 or float64 only")
        self.dtype = dtype
        self.elem = 4 if dtype == torch.float32 else 8
        self._device = torch.empty(0, dtype=dtype, device=device).device
        self._t = None
        self._product, operands, n = self._one_kernel()
        if self._product is not None:
            self._operands = self._buffers(operands)
            self._workspace = torch.empty(n // self.elem, dtype=dtype, device=self._device) if n else None
        else:
            self._library_buffers()

    def _one_kernel(self):
        """The product that adds into the destination, the permutations its operands need (None where an
        operand is in either of the two matrix layouts already) and its workspace in bytes."""
        lay = self.lay
        if not 1 <= len(lay.d_labels) <= self._B.TPERM_MAX_RANK:
            return None, None, 0

        def place(labels, free, summed):    # (permutation, summed index first)
            if labels == free + summed:
                return None, False
            if labels == summed + free:
                return None, True
            return tuple(map(labels.index, free + summed)), False

        best = least = None
        for summed in dict.fromkeys((lay.summed, "".join(c for c in lay.r_labels if c in lay.l_labels))):
            ops = place(lay.l_labels, lay.free_l, summed), place(lay.r_labels, lay.free_r, summed)
            moved = (lay.m if ops[0][0] else 0) + (lay.n if ops[1][0] else 0)    # times k
            if best is None or moved < least:
                best, least = ops, moved
        try:
            product = self._B.tperm_product_create(lay.dims(lay.free_l + lay.free_r), lay.t_perm, len(lay.free_l),
                                                   lay.k, self.elem, best[0][1], best[1][1])
        except self._B.TpermError:    # tensors of 4 GiB and more
            return None, None, 0
        info = self._B.tperm_product_describe(product)
        if not info.pays:
            return None, None, 0
        return product, (best[0][0], best[1][0]), info.workspace_bytes

    def _buffers(self, perms):
        """(permutation, buffer) of either operand; inputs already in matrix layout are used in place."""
        lay, torch = self.lay, self._torch
        sizes = (lay.m * lay.k, lay.k * lay.n)
        return [(p, None if p is None else torch.empty(n, dtype=self.dtype, device=self._device))
                for p, n in zip(perms, sizes)]

    def _library_buffers(self):
        lay = self.lay
        ident = lambda p: tuple(p) == tuple(range(len(p)))
        self._library = self._buffers([None if ident(p) else p for p in (lay.l_perm, lay.r_perm)])
        self._t = self._torch.empty(lay.m * lay.n, dtype=self.dtype, device=self._device)

    def _in_one_kernel(self, l, r, d) -> bool:
        """Whether this call may add into d while it reads its operands.  Operands that are used in place
        have to be plain memory on this object's device, apart from d; the others go the way of the library
        product, which reads a tensor that is negated lazily as such and refuses those that carry gradients
        (backward or forward mode)."""
        if self._product is None:
            return False
        for (perm, _), t in zip(self._operands, (l, r)):
            if perm is None:
                a, b = t.data_ptr(), d.data_ptr()
                if t.device != self._device or t.is_neg() or (t.requires_grad and self._torch.is_grad_enabled()) or \
                        self._unpack_dual(t).tangent is not None or \
                        (a < b + d.numel() * self.elem and b < a + t.numel() * self.elem):
                    return False
        return True

    def run(self, l, r, d, timings: dict = None) -> None:
        """d += l * r; all three are flat device tensors of the contraction's dtype.  ``timings`` receives
        the milliseconds of the steps (transpose_d_ms is 0 where gemm_ms includes that step)."""
        torch, B, lay = self._torch, self._B, self.lay
        for t, labels in ((l, lay.l_labels), (r, lay.r_labels), (d, lay.d_labels)):
            if t.dtype != self.dtype or t.numel() != math.prod(lay.dims(labels)) or not t.is_contiguous():
                raise ValueError("operand does not match the planned contraction")
        one_kernel = self._in_one_kernel(l, r, d)
        if not one_kernel and self._t is None:
            self._library_buffers()
        stream = torch.cuda.current_stream().cuda_stream
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(5)] if timings is not None else None
        mark = (lambda i: ev[i].record()) if ev else (lambda i: None)
        mark(0)
        ops = []
        for i, (t, labels) in enumerate(((l, lay.l_labels), (r, lay.r_labels))):
            perm, buffer = (self._operands if one_kernel else self._library)[i]
            if perm is not None:
                B.tperm_transpose(lay.dims(labels), perm, self.elem, t.data_ptr(), buffer.data_ptr(), stream)
                t = buffer
            ops.append(t)
            mark(1 + i)
        if one_kernel:
            ws = self._workspace
            B.tperm_product_accumulate(self._product, ops[0].data_ptr(), ops[1].data_ptr(), d.data_ptr(), stream,
                                       0 if ws is None else ws.data_ptr(), 0 if ws is None else ws.numel() * self.elem)
            mark(3)
        else:
            # column-major (m x k)(k x n) = (m x n)  is  row-major (n x k)(k x m) = (n x m)
            torch.mm(ops[1].view(lay.n, lay.k), ops[0].view(lay.k, lay.m), out=self._t.view(lay.n, lay.m))
            mark(3)
            t_dims = lay.dims(lay.free_l + lay.free_r)
            B.tperm_transpose(t_dims, lay.t_perm, self.elem, self._t.data_ptr(), d.data_ptr(), stream, accumulate=True)
        mark(4)
        if ev:
            ev[4].synchronize()
            names = ("transpose_l_ms", "transpose_r_ms", "gemm_ms", "transpose_d_ms")
            for i, name in enumerate(names):
                timings[name] = 0.0 if one_kernel and i == 3 else ev[i].elapsed_time(ev[i + 1])
            timings["total_ms"] = ev[0].elapsed_time(ev[4])


def contract(d_labels: str, l_labels: str, r_labels: str, extents: Dict[str, int], l, r, d) -> None:
    """One-shot d += l * r (plans and workspace are built on every call; keep a Contraction
    object around when the same contraction repeats)."""
    Contraction(d_labels, l_labels, r_labels, extents, d.dtype, d.device).run(l, r, d)


def _bench(argv: Sequence[str] = None) -> None:
    """Times the seeded contraction sample: GFLOP/s and the share of time spent transposing,
    against arithmetic intensity.  One JSON line per case with the path it took, then a summary line for each
    path: "library" (transposes, library product, accumulating transpose; --library takes it everywhere), or
    "one kernel", whose product_ms covers the destination's update too and whose transposes are the operands' only."""
    import argparse
    import json
    import numpy as np
    import torch
    from . import workloads as wl
    ap = argparse.ArgumentParser(description=_bench.__doc__)
    ap.add_argument("--dtype", choices=["f32", "f64"], default="f64")
    ap.add_argument("--reps", type=int, default=5)
    ap.add_argument("--library", action="store_true", help="take the library product for every contraction")
    args = ap.parse_args(argv)
    dtype = torch.float64 if args.dtype == "f64" else torch.float32
    paths = {"library": [], "one kernel": []}
    for case in wl.contraction_cases():
        c = Contraction(case["d"], case["l"], case["r"], case["extents"], dtype)
        if args.library:
            c._product = None
        lay = c.lay
        g = torch.Generator(device="cuda").manual_seed(case["seed"])
        l = torch.rand(lay.m * lay.k, dtype=dtype, device="cuda", generator=g) * 2 - 1
        r = torch.rand(lay.k * lay.n, dtype=dtype, device="cuda", generator=g) * 2 - 1
        d = torch.zeros(lay.m * lay.n, dtype=dtype, device="cuda")
        c.run(l, r, d)
        best = None
        for _ in range(args.reps):
            t = {}
            c.run(l, r, d, t)
            if best is None or t["total_ms"] < best["total_ms"]:
                best = t
        one = c._in_one_kernel(l, r, d)
        ops = best["transpose_l_ms"] + best["transpose_r_ms"]
        row = {"case": case["name"], "path": "one kernel" if one else "library", "d": case["d"], "l": case["l"], "r": case["r"],
               "m": lay.m, "n": lay.n, "k": lay.k,
               "arithmetic_intensity": round(lay.arithmetic_intensity, 1),
               "gflops": round(lay.flops / best["total_ms"] / 1e6, 1)}
        if one:
            row.update(product_gflops=round(lay.flops / best["gemm_ms"] / 1e6, 1),
                       operand_transpose_share=round(ops / best["total_ms"], 4),
                       transpose_l_ms=round(best["transpose_l_ms"], 4), transpose_r_ms=round(best["transpose_r_ms"], 4),
                       product_ms=round(best["gemm_ms"], 4), total_ms=round(best["total_ms"], 4))
        else:
            row.update(gemm_gflops=round(lay.flops / best["gemm_ms"] / 1e6, 1),
                       transpose_share=round((ops + best["transpose_d_ms"]) / best["total_ms"], 4),
                       **{k: round(v, 4) for k, v in best.items()})
        paths[row["path"]].append(row)
        print(json.dumps(row), flush=True)
    for path, rows in paths.items():
        if not rows:
            continue
        by = sorted(rows, key=lambda x: x["arithmetic_intensity"])
        third = max(1, len(by) // 3)
        share = "transpose_share" if path == "library" else "operand_transpose_share"
        summary = {"metric": "tensor contraction through transposes + " + ("GEMM" if path == "library" else "product into the destination"),
                   "path": path, "dtype": args.dtype, "cases": len(rows),
                   "low_ai": {"ai_max": by[third - 1]["arithmetic_intensity"],
                              "median_" + share: float(np.median([x[share] for x in by[:third]]))},
                   "high_ai": {"ai_min": by[-third]["arithmetic_intensity"],
                               "median_" + share: float(np.median([x[share] for x in by[-third:]])),
                               "median_gflops": float(np.median([x["gflops"] for x in by[-third:]]))}}
        print(json.dumps(summary), flush=True)


if __name__ == "__main__":
    _bench()

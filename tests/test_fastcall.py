"""Argument conversion of the execute calls (the CPython extension behind binding.py): the same objects
are taken and refused as by ctypes, statuses come back as TpermError.  Host only: every call here is
refused before anything is launched."""
import os
import subprocess
import sys
import sysconfig
import threading

import numpy as np
import pytest

from paper_1705_01598_amd import binding as B

A, O = 1 << 32, 1 << 33                                     # addresses that are never touched


def _status(f, *args, **kw):
    with pytest.raises(B.TpermError) as e:
        f(*args, **kw)
    return e.value.status


@pytest.fixture(scope="module")
def plan():
    return B.tperm_plan_create((6, 5, 4), (2, 0, 1), 8)


@pytest.mark.parametrize("f", [B.tperm_execute, B.tperm_execute_accumulate])
def test_execute_statuses_and_types(f, plan):
    assert _status(f, plan, None, O) == B.ERR_NULL and _status(f, plan, A, 0) == B.ERR_NULL
    assert _status(f, plan, A + 4, O) == B.ERR_ALIGN
    assert _status(f, plan, A, A) == B.ERR_ALIAS and _status(f, plan, A, A + 8, stream=0) == B.ERR_ALIAS
    assert _status(f, plan=plan, in_ptr=A, out_ptr=A, stream=None) == B.ERR_ALIAS
    for bad in ("1", 1.0, b"x", np.int64(A), [A]):
        with pytest.raises(TypeError):
            f(plan, bad, O)
        with pytest.raises(TypeError):
            f(plan, A, A, bad)
    with pytest.raises(TypeError):
        f(plan, A)
    gone = B.tperm_plan_create((6, 5), (1, 0), 8)
    gone.destroy()
    assert _status(f, gone, A, O) == B.ERR_NULL


def test_verified_statuses(plan):
    n = B.verify_workspace_bytes(120)
    f = lambda v, w, b: _status(B.tperm_execute_verified, plan, A, O, 0, v, w, b)  # noqa: E731
    assert f(0, 1 << 34, n) == B.ERR_NULL and f(1 << 35, 1 << 34, n - 1) == B.ERR_TOO_LARGE
    assert f(1 << 35, (1 << 34) + 4, n) == B.ERR_ALIGN and f(1 << 35, A, np.int64(n)) == B.ERR_ALIAS
    with pytest.raises((TypeError, ValueError)):
        B.tperm_execute_verified(plan, A, O, 0, 1 << 35, 1 << 34, "many")


def test_one_call_interface_arguments():
    t = B.tperm_transpose
    ok = ((6, 5, 4), (2, 0, 1), 8)
    assert _status(t, *ok, A, A) == B.ERR_ALIAS
    for dims, perm, elem in (([6, 5, 4], [2, 0, 1], 8), (np.array([6, 5, 4]), np.array([2, 0, 1], np.int32), np.int64(8)),
                             (("6", 5.7, 4), iter((2, 0, 1)), "8"), (range(4, 7), (2, 0, 1), True + 7)):
        assert _status(t, dims, perm, elem, A, A, accumulate=True) == B.ERR_ALIAS
    assert _status(t, (), (), 8, A, O) == B.ERR_RANK and _status(t, (2,) * 17, tuple(range(17)), 8, A, O) == B.ERR_RANK
    assert _status(t, (6, 5, 4), (2, 0), 8, A, O) == B.ERR_PERM and _status(t, (6, 0), (1, 0), 8, A, O) == B.ERR_DIMS
    assert _status(t, (6, 5), (1, 0), 3, A, O) == B.ERR_ELEM_SIZE
    with pytest.raises(IndexError):
        t((6, 5), (1, 0, 2), 8, A, O)
    for bad in ((iter((6, 5)), (1, 0)), (7, (0,)), ((6, None), (1, 0)), ((6, 5), 3)):
        with pytest.raises(TypeError):
            t(*bad, 8, A, O)
    with pytest.raises(ValueError):
        t(("six", 5), (1, 0), 8, A, O)
    with pytest.raises(TypeError):
        t((6, 5), (1, 0), 8, "A", O)


@pytest.mark.parametrize("change,kept", [(lambda x: x.clear(), 1), (lambda x: x.__delitem__(slice(2, None)), 2),
                                         (lambda x: x.extend([1] * 1000), 1013)])
def test_a_list_that_changes_while_it_is_converted(change, kept):
    """Converting an entry may run Python code: the entries are those that iterating the list gives."""
    class Entry:
        def __init__(self, owner, value):
            self.owner, self.value = owner, value

        def __int__(self):
            if self.owner is not None:
                change(self.owner)
                self.owner = None
            return self.value

    def fresh(values):
        entries = []
        entries += [Entry(entries if i == 0 else None, v) for i, v in enumerate(values)]
        return entries
    rank = 13
    for dims, perm, n, given in ((fresh([2] * rank), tuple(range(rank)), kept, rank), ((2,) * rank, fresh(range(rank)), rank, kept)):
        if given > n:                                     # more permutation entries than extents
            with pytest.raises(IndexError):
                B.tperm_transpose(dims, perm, 8, A, A)
        else:                                             # too many extents, or too few entries
            assert _status(B.tperm_transpose, dims, perm, 8, A, A) == (B.ERR_RANK if n > 16 else B.ERR_PERM)


def test_the_extension_belongs_to_this_interpreter():
    """Its file name holds the interpreter's ABI; where there is none for this one, loading says so."""
    from paper_1705_01598_amd import _fastcall, build
    assert B.FASTCALL_PATH == build.FASTCALL == _fastcall.__file__
    assert os.path.basename(B.FASTCALL_PATH) == "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX") != "_fastcall.so"
    src = ("from paper_1705_01598_amd import binding as B\n"
           "B.FASTCALL_PATH = B.FASTCALL_PATH.replace('cpython-', 'cpython-0')\n"
           "try:\n    B.lib()\nexcept FileNotFoundError as e:\n    print(e)\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, cwd=root)
    assert out.returncode == 0 and "paper_1705_01598_amd.build" in out.stdout


def test_calls_from_several_threads(plan):
    seen = []

    def work(i):
        for _ in range(200):
            seen.append(_status(B.tperm_transpose, (6 + i, 5), (1, 0), 8, A, A))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for x in threads:
        x.start()
    for x in threads:
        x.join()
    assert seen == [B.ERR_ALIAS] * 800

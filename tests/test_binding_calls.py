"""The calls of the path as the binding makes them (csrc/mw_py.c), without a GPU: what they take, what they refuse, and that the
library's own answer comes back.  A context of None is refused by every call before anything touches a device."""
import ctypes as C
import inspect
import os
import re
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2605_22428_amd import binding as B


def _calls():
    return sorted(set(re.findall(r"_native\(\)\.(mw_\w+)", inspect.getsource(B))))


def test_every_call_has_the_same_arguments_in_both_forms():
    source = open(os.path.join(B.HERE, "csrc", "mw_py.c")).read()
    assert dict(re.findall(r'CALL\((mw_\w+), "(\w+)"', source)) == B._KINDS and sorted(B._KINDS) == _calls()


@pytest.mark.parametrize("form", ["module", "ctypes"])
@pytest.mark.parametrize("name", _calls())
def test_arguments_reach_the_library(name, form):
    calls = B._native() if form == "module" else B._CtypesCalls(B.load())
    assert (form == "module") == (getattr(calls, "__name__", "").endswith("_mwcall"))
    call, kinds = getattr(calls, name), B._KINDS[name]
    t = torch.zeros(8, dtype=torch.int32)
    good = [{"h": None, "t": t, "p": 0, "i": 1, "l": 16}[k] for k in kinds]
    assert call(*good) == B.MW_ERR_INVALID_ARG                       # no context
    assert call(*[C.c_void_p(0) if k == "h" else a for k, a in zip(kinds, good)]) == B.MW_ERR_INVALID_ARG
    assert call(*[None if k == "t" else a for k, a in zip(kinds, good)]) == B.MW_ERR_INVALID_ARG
    with pytest.raises(TypeError):
        call(*good[:-1])
    for at, kind in enumerate(kinds):
        for bad, error in {"h": [(7, AttributeError)], "t": [(7, AttributeError), ("x", AttributeError)], "p": [(None, TypeError), (t, TypeError)],
                           "i": [(1.5, TypeError), (None, TypeError)], "l": [(1.5, TypeError), ("3", TypeError)]}[kind]:
            if kind == "p" and bad is t:
                bad = torch.zeros(2)                                 # (a tensor of one whole number is an index)
            with pytest.raises(error):
                call(*(good[:at] + [bad] + good[at + 1:]))


def test_every_method_of_a_context_that_is_closed_is_refused():
    ctx = B.Context.__new__(B.Context)
    ctx._h = None
    t = torch.zeros(8, dtype=torch.int32)
    B_stream, B._stream_handle = B._stream_handle, lambda: 0
    try:
        for call, args in ((ctx.mw_plan, (t, t, t, t, t)), (ctx.mw_unpack, (t, 1, t, None, 4, t, t, t, t)), (ctx.mw_relay, (t, t, 4, t))):
            with pytest.raises(B.MwError) as e:
                call(*args)
            assert e.value.status == B.MW_ERR_INVALID_ARG
    finally:
        B._stream_handle = B_stream


OTHER_INTERPRETER = """
import sys, sysconfig, ctypes
sysconfig.get_config_vars()["EXT_SUFFIX"] = ".cpython-999-x86_64-linux-gnu.so"
sys.path.insert(0, sys.argv[1])
from paper_2605_22428_amd import binding as B
calls = B._native()
assert isinstance(calls, B._CtypesCalls), calls
assert calls.mw_plan_allgather(None, 16, None, None, 0) == B.MW_ERR_INVALID_ARG
"""


def test_an_interpreter_without_the_module_calls_through_ctypes():
    assert os.path.basename(B.CALLS_PATH) != "_mwcall.so"            # (which any interpreter would import)
    subprocess.run([sys.executable, "-c", OTHER_INTERPRETER, os.path.dirname(B.HERE)], check=True)


TWO_TREES = """
import sys
sys.path[:0] = sys.argv[1:]
from paper_2605_22428_amd import binding as first
first._native()
from other import binding as second
assert second._native().mw_allgather_step(None, None, 0, None, None, None, None, None, 0) == -77
assert first._native().mw_allgather_step(None, None, 0, None, None, None, None, None, 0) == first.MW_ERR_INVALID_ARG
"""


def test_calls_reach_the_library_of_their_own_tree(tmp_path):
    """A second tree in the process, whose library answers everything with -77."""
    shutil.copytree(B.HERE, tmp_path / "other", ignore=shutil.ignore_patterns("libmw.so*", "csrc", "__pycache__"))
    (tmp_path / "stub.c").write_text("".join("int %s(void) { return -77; }\n" % name for name in B.EXPORTS))
    subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / "stub.c"), "-o", str(tmp_path / "other" / "libmw.so")], check=True)
    subprocess.run([sys.executable, "-c", TWO_TREES, os.path.dirname(B.HERE), str(tmp_path)], check=True)

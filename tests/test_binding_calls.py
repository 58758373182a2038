"""The two executor calls of the Python binding: the C functions take what the ctypes functions take, with the same
results and errors, and the binding works without them.  Host-only plans: every call ends in the library's argument
checks, before anything is launched."""
import ctypes
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest

from paper_2008_11849_amd import sparsert as sp, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _plans():
    csr = synth.uniform_csr(16, 18, 0.5, 3)
    return (sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 16, 18, 20, host_only=True),
            sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 16, 18, 20, host_only=True, conv=(2, 4, 5)))


def _outcome(call, args, kw):
    try:
        return call(*args, **kw)
    except Exception as e:
        return type(e).__name__, str(e).replace("_spmm", "spmm").replace("_conv3x3", "conv3x3"), getattr(e, "status", None)


@pytest.mark.parametrize("fast,general,which", [(sp.spmm, sp._spmm, 0), (sp.conv3x3, sp._conv3x3, 1)])
def test_the_calls_take_the_same_arguments_as_ctypes_does(fast, general, which):
    plan, other = _plans()[which], _plans()[1 - which]
    there = 1 << 20   # an address that is only looked at

    class HalfOpen:
        handle = None

    class Wide:
        handle = ctypes.c_void_p(plan.handle)

    forms = [((plan, there, there), {}), ((plan, there, there, 0), {}), ((plan, there, there, None), {}),
             ((plan, there, there, 7), {}), ((plan, None, there), {}), ((plan, there, 0, 0), {}),
             ((plan, there + 4, there), {}), ((plan, there, there + 8), {}),                        # not on 16 bytes
             ((other, there, there), {}), ((HalfOpen, there, there), {}), ((Wide, there, there), {}),
             ((plan, ctypes.c_void_p(there), there), {}), ((plan, ctypes.c_void_p(there), ctypes.c_void_p(None), ctypes.c_void_p(None)), {}),
             ((plan, True, there), {}), ((plan, -16, -32), {}), ((plan, 2 ** 64 + 16, there), {}), ((plan, 2 ** 70 + 4, there), {}),
             ((plan, there, there), {"stream": 0}), ((plan,), {"B_dev" if which == 0 else "X_dev": there, "C_dev" if which == 0 else "Y_dev": there, "stream": 0}),
             ((plan, np.int64(there), there), {}), ((plan, 1.5, there), {}), ((plan, "x", there), {}), ((plan, there, there, "s"), {}),
             ((plan, there), {}), ((), {}), ((plan, there, there, 0, 0), {}), ((plan, there, there), {"streem": 0}),
             ((None, there, there), {}), ((plan.handle, there, there), {})]
    refused = 0
    for args, kw in forms:
        want = _outcome(general, args, kw)
        assert _outcome(fast, args, kw) == want, (args, kw)
        refused += want is not None and want[0] == "SparseRTError"
    assert refused >= 17   # reached the library; a host-only plan is never executed


def test_the_binding_works_without_the_c_functions():
    code = """
import sys
sys.modules["paper_2008_11849_amd._fastcall"] = None   # what an import finds that was not built
from paper_2008_11849_amd import sparsert as sp, synth
assert sp.spmm is sp._spmm and sp.conv3x3 is sp._conv3x3
csr = synth.uniform_csr(16, 18, 0.5, 3)
plan = sp.inspect(csr.row_ptr, csr.col_idx, csr.vals, 16, 18, 20, host_only=True)
for call in (sp.spmm, sp.conv3x3):
    try:
        call(plan, 1 << 20, 1 << 20, stream=0)
    except sp.SparseRTError as e:
        assert e.status == sp.EINVAL
    else:
        raise SystemExit("not refused")
"""
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]


@pytest.mark.skipif(sp._fastcall is None, reason="built without the Python headers")
def test_the_c_functions_are_built_for_this_interpreter_and_refuse_before_they_are_bound():
    assert os.path.basename(sp._fastcall.__file__) == "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX")
    assert sp.spmm is sp._fastcall.spmm and sp.conv3x3 is sp._fastcall.conv3x3
    code = """
from paper_2008_11849_amd import _fastcall
for args, kw in (((1, 2, 3), {}), ((1,), {"stream": 0})):
    try:
        _fastcall.spmm(*args, **kw)
    except RuntimeError:
        continue
    raise SystemExit("not refused")
"""
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]

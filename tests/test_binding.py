"""What the compiled binding takes and refuses, through the public functions of `qsync` (CPU only: every call here returns before
anything is launched -- an empty tensor, or an argument that is refused)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2407_02327_amd import qsync as Q


@pytest.mark.parametrize("integer", [np.int64, np.int32, np.uint8, torch.tensor], ids=lambda f: f.__name__)
def test_integers_are_whatever_has_an_index(integer):
    """Sizes, enumerators, seeds: Python's integers and everything that answers as one (a product of shapes in numpy is no `int`)."""
    i, x, s = integer, torch.empty(4), torch.empty(1)
    Q.qsync_absmax_scale(x, i(0), i(4), i(4), i(Q.PER_TENSOR), i(8), s, s, None, None, None, 0)
    Q.qsync_quantize(x, i(0), i(4), i(4), i(Q.FP16), i(0), i(0), i(Q.ROUND_NEAREST), i(7), i(0), None, x, None, 0)
    rows = i(4)      # one object for sizes that follow each other
    with pytest.raises(Q.QsyncError) as e:
        Q.qsync_quantize(x, rows, rows, i(2), i(Q.FP16), i(0), i(0), i(Q.ROUND_NEAREST), i(7), i(0), None, x, None, 0)
    assert e.value.status == Q.ERR_BAD_SHAPE


@pytest.mark.parametrize("bad", [4.0, "4", None])
def test_other_integers_are_refused(bad):
    x = torch.empty(4)
    with pytest.raises(TypeError):
        Q.qsync_quantize(x, 0, bad, 4, Q.FP16, 0, 0, 0, 0, 0, None, x, None, 0)


def test_an_address_is_no_tensor():
    """A pointer argument is a tensor or None: a number there would be an address that nothing has checked."""
    x, s = torch.empty(4), torch.empty(1)
    for args in ((4096, 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, x, None, 0), (x, 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, 4096, None, 0),
                 (x, 0, 4, 4, Q.INT8, 8, 0, 0, 0, 0, True, x, None, 0)):
        with pytest.raises(AttributeError):
            Q.qsync_quantize(*args)
    with pytest.raises(AttributeError):
        Q.qsync_absmax_scale(x, 0, 4, 4, Q.PER_TENSOR, 8, s, s, None, None, 4096, 0)      # (nor is it a workspace and its size)


class _Holder:
    """Answers for a tensor's memory without being one."""

    def __init__(self, t):
        self.t, self.dtype = t, t.dtype
        self.data_ptr, self.numel, self.element_size = t.data_ptr, t.numel, t.element_size


def test_objects_that_hold_memory():
    """data_ptr() and dtype are what a pointer and its type are read from, numel() and element_size() a workspace's size."""
    h = lambda n, dt=torch.float32: _Holder(torch.empty(n, dtype=dt))
    Q.qsync_quantize(h(4), 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, h(4, torch.float16), None, 0)
    with pytest.raises(Q.QsyncError) as e:                        # an integer tensor is no source: its type was read
        Q.qsync_quantize(h(4, torch.int32), 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, h(4), None, 0)
    assert e.value.status == Q.ERR_BAD_ENUM
    with pytest.raises(KeyError):
        Q.qsync_quantize(h(4, torch.int64), 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, h(4), None, 0)
    need, s = Q.qsync_absmax_quantize_workspace_bytes(4, 8), h(1)
    with pytest.raises(Q.QsyncError) as e:
        Q.qsync_absmax_quantize(h(32), 4, 8, 8, 0, 0, 0, s, s, None, h(32, torch.int8), None, h(need // 4 - 1), -1, 0)
    assert e.value.status == Q.ERR_WORKSPACE


def test_probe_without_an_output():
    with pytest.raises(Q.QsyncError) as e:
        Q.qsync_probe_mfma(Q.INT8, 0, 4, None, 0)
    assert e.value.status == Q.ERR_NULL


FORK = """
import os, sys
import torch
state = {"up": True}                      # stands for torch's own: initialised, and not in a process forked after that
torch.cuda.is_initialized = lambda: state["up"]
def current_stream():
    raise RuntimeError("cannot re-initialize in a forked process")
torch.cuda.current_stream = current_stream
from paper_2407_02327_amd import qsync as Q
x = torch.empty(4)
def call():
    try:
        Q.qsync_quantize(x, 0, 4, 4, Q.FP16, 0, 0, 0, 0, 0, None, x, None)
    except RuntimeError as e:
        return str(e)
    return ""
first = call()
assert "forked" not in first, first       # (no device here: whatever the lookup of its stream says)
pid = os.fork()
if pid == 0:
    state["up"] = False
    os._exit(0 if "forked" in call() else 1)
sys.exit(os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]))
"""


@pytest.mark.skipif(torch.cuda.is_available(), reason="forks after a stand-in for the device's initialisation")
def test_a_forked_process_is_told_so():
    """torch says, at the first use of the device in a process that was forked from one that had used it, that this cannot work;
    the look-up of the current stream has to ask again there."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", FORK], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr

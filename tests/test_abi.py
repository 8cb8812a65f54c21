"""The C-ABI library loads and exports every symbol include/nd.h declares
(no compute calls: this runs without a GPU)."""
import ctypes
import os
import re

import numpy as np
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

from paper_2009_06693_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "nd.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = set(re.findall(r"\b(nd_[a-z_0-9]+)\s*\(", text))
    return names


def test_every_declared_symbol_is_exported():
    L = B.lib()
    names = _declared()
    assert {"nd_graph_create", "nd_sample", "nd_sample_query", "nd_graph_destroy"} <= names
    for n in names:
        assert hasattr(L, n), f"{n} declared in nd.h but not exported"
    assert set(B.EXPORTS) == names


def test_version_and_params_defaults():
    assert B.nd_version() == 100
    p = B.nd_params_init()
    assert p.struct_size == ctypes.sizeof(B.nd_params) == 128
    assert p.n2v_max_attempts == 64 and p.sched_force_class == B.ND_CLASS_AUTO
    assert p.mode == B.ND_MODE_TRANSIT_PARALLEL and p.p == 1.0 and p.q == 1.0


def test_null_arguments_are_errors_not_crashes():
    L = B.lib()
    assert L.nd_graph_destroy(None) == 0
    assert L.nd_sample_query(None, 0, None, 0, None, None, None) == B.ND_ERR_NULL_POINTER
    assert b"NULL" in L.nd_last_error()
    h = ctypes.c_void_p()
    assert L.nd_graph_create(ctypes.byref(h), 4, 0, None, 0, None, None, 0, None) == B.ND_ERR_NULL_POINTER
    assert L.nd_graph_create(None, 4, 0, None, 0, None, None, 0, None) == B.ND_ERR_NULL_POINTER
    assert L.nd_group_workspace_bytes(1000, 50) > 0


@pytest.mark.parametrize("call,complaint", [
    (lambda p, t: B._call.sample(None, 0, p, t, 1, [t], t, 0), "roots must be"),
    (lambda p, t: B._call.sample(None, 0, p, 3, 1, [t], t, 0), "roots must be"),
    (lambda p, t: B._call.sample(None, 0, None, t, 1, [t], t, 0), ""),
    (lambda p, t: B._call.sample(None, 0, b"x", t, 1, [t], t, 0), "nd_params"),
    (lambda p, t: B._call.sample_static(None, 0, p, t, 1.5, [t], None, 0), "integer"),
    (lambda p, t: B._call.sample(None, np.int32(0), p, t, np.int64(1), [t], t, 0), "roots must be"),
    (lambda p, t: B._call.sample(None, 0, p, t, 1, [t], t), "expected 8"),
    (lambda p, t: B._call.pack([t], 3, t, 0), "step arrays must be"),
    (lambda p, t: B._call.pack(t, "3", t, 0), ""),
    (lambda p, t: B._call.record_length([t, 1], 3), "step arrays must be"),
])
def test_marshalling_refuses_what_is_no_gpu_array(call, complaint):
    B.lib()
    with pytest.raises(TypeError, match=complaint):
        call(B.nd_params_init(), torch.zeros(3, dtype=torch.int32))


def _on_gpu(n=3, dtype=torch.int32):
    """What looks like an array on a GPU, without one (its address is null)."""
    with FakeTensorMode():
        return torch.empty(n, dtype=dtype, device="cuda:0")


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
def test_as_many_outputs_as_steps():
    """The library reads an address per step: a shorter list is refused, not read past its end."""
    B.lib()
    t, none = _on_gpu(), _on_gpu(0)
    for steps, call in ((3, lambda r, o: B._call.sample(None, B.ND_KHOP, p, r, 1, o, t, 0)),
                        (4096, lambda r, o: B._call.sample_static(None, B.ND_PPR, p, r, 1, o, None, 0))):
        p = B.nd_params_init(num_steps=steps)
        for n in (0, 1, steps - 1):
            with pytest.raises(ValueError, match=f"{n} arrays for {steps} steps"):
                call(t, [t] * n)
        for r, n in ((t, steps), (t, steps + 1), (none, 0)):  # no roots, nothing written
            assert call(r, [t] * n) == B.ND_ERR_NULL_POINTER  # the library's answer: no graph
    p = B.nd_params_init(num_steps=4097)
    assert B._call.sample(None, B.ND_PPR, p, t, 1, [t], t, 0) == B.ND_ERR_NULL_POINTER


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("bad", [torch.zeros(4096, dtype=torch.int32),                     # the host's own memory
                                 _on_gpu(64)[::2], _on_gpu(1).expand(64), 7])
def test_memory_that_a_kernel_cannot_use_is_refused(bad):
    """Its address would be handed to a kernel, with more bytes behind it than the tensor has where it has gaps."""
    B.lib()
    p, t = B.nd_params_init(num_steps=1), _on_gpu()
    with pytest.raises(TypeError, match="workspace must be"):
        B._call.sample(None, 0, p, t, 1, [t], bad, 0)
    with pytest.raises(TypeError, match="status must be"):
        B._call.sample_static(None, 0, p, t, 1, [t], bad, 0)
    with pytest.raises(TypeError, match="samples must be"):
        B._call.pack([t], 3, bad, 0)


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
def test_memory_that_a_kernel_can_use_is_taken():
    """Whatever the types and shapes of the scratch and the status word; no samples need no records."""
    B.lib()
    p, t = B.nd_params_init(num_steps=1), _on_gpu()
    for ok in (_on_gpu(64, torch.uint8), _on_gpu(64, torch.float64).view(8, 8).t(), _on_gpu(1, torch.int64)):
        assert B._call.sample(None, 0, p, t, 1, [t], ok, 0) == B.ND_ERR_NULL_POINTER
        assert B._call.sample_static(None, 0, p, t, 1, [t], ok, 0) == B.ND_ERR_NULL_POINTER
    assert B._call.pack([t], 0, torch.zeros(0, dtype=torch.int32), 0) == B.ND_OK
    for short in (_on_gpu(0), _on_gpu(3, torch.uint8)):
        with pytest.raises(TypeError, match="status must be"):
            B._call.sample_static(None, 0, p, t, 1, [t], short, 0)

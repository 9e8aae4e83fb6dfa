"""The native marshalling of the binding's asynchronous calls, without a GPU: what it hands to the
library is what the same call through ctypes hands over.  Every input here is refused (or has no
rows) before anything would be enqueued."""
import ctypes as C
import os
import subprocess
import sys

import pytest
import torch

import paper_2403_17017_amd as S
from paper_2403_17017_amd import binding as B


def matrix(rows=4, cols=5, nnz=3):
    return S.DeviceCSR(rows, cols, torch.zeros(rows + 1, dtype=torch.int32), torch.zeros(max(nnz, 1), dtype=torch.int32),
                       torch.zeros(max(nnz, 1)), nnz)


def through_ctypes(call, handle, A, x, y, ws):
    L, cs = S.lib(), A.c_struct()
    tail = (x.data_ptr(), y.data_ptr(), ws.data_ptr() if ws is not None else None, ws.numel() if ws is not None else 0, None)
    if call == "spmv":
        return L.seer_spmv(handle, C.byref(cs), *tail)
    if call == "auto":
        return L.seer_spmv_auto(C.byref(cs), C.byref(handle.c), *tail)
    if call == "model":
        return L.seer_spmv_model(C.byref(cs), C.byref(handle.c), *tail, None, None)
    return L.seer_spmv_prepared(C.byref(handle.c), C.byref(cs), *tail)


def through_marshal(call, handle, A, x, y, ws):
    S.lib()
    if call == "spmv":
        return B._marshal.spmv(handle, A, x, y, ws, 0)
    f = {"auto": B._marshal.spmv_auto, "model": B._marshal.spmv_model, "prepared": B._marshal.spmv_prepared}[call]
    rc = f(C.addressof(handle.c), A, x, y, ws, 0)
    return rc[0] if call == "model" else rc


def handles(call):
    if call == "spmv":
        return [0, 3, 4, 5, 6, 8, 9, -1]
    if call == "prepared":
        return [S.Plan(B.seer_plan(k, rows, 3, 1, split, 0, None, 0), None) for k in (3, 5, 6, 7, 8, 99) for rows in (4, 5)
                for split in (0, 1)]
    deep = S.Tree([0, -1, -1], [1.0, 0, 0], [1, -1, -1], [7, -1, -1], [-1, 0, 1])          # a child that is not there
    trees = [S.Tree.constant(S.CSR_MP), S.Tree.constant(S.CSR_A), deep]
    return trees if call == "auto" else [S.Model(t) for t in trees]


@pytest.mark.parametrize("call", ["spmv", "auto", "model", "prepared"])
def test_same_status_as_through_ctypes(call):
    both = torch.zeros(16)
    aligned = torch.zeros(64, dtype=torch.uint8)
    seen = set()
    for h in handles(call):
        for A in (matrix(), matrix(nnz=0), matrix(rows=0, nnz=0)):
            for x, y in ((both[:5], both[2:6]), (both[:5], both[4:9])):             # overlapping: refused in every call
                for ws in (None, aligned, aligned[1:]):
                    if A.rows and not B.lib().seer_num_kernels() == S.NUM_KERNELS:
                        continue
                    want = through_ctypes(call, h, A, x, y, ws)
                    assert through_marshal(call, h, A, x, y, ws) == want
                    assert want <= 0 and (want < 0 or A.rows == 0)
                    seen.add(want)
    assert len(seen) >= 3                                                              # accepted, and refused in several ways


def test_errors_of_the_objects_come_through():
    S.lib()
    x = torch.zeros(8)
    with pytest.raises(AttributeError):
        B._marshal.spmv(0, object(), x, x, None, 0)
    with pytest.raises(AttributeError):
        B._marshal.spmv(0, matrix(), 3, x, None, 0)
    with pytest.raises(TypeError):
        B._marshal.spmv(0, matrix(), x, x, None)
    with pytest.raises(S.SeerError):
        S.seer_spmv_prepared(handles("prepared")[0], matrix(), x, x, workspace=torch.zeros(64, dtype=torch.uint8), stream=0)


def test_first_call_of_a_process_may_name_a_kernel_that_does_not_exist():
    """The library is loaded by whatever call comes first, also one that asks it for no size."""
    code = ("import torch, paper_2403_17017_amd as S\n"
            "A = S.DeviceCSR(4, 5, torch.zeros(5, dtype=torch.int32), torch.zeros(3, dtype=torch.int32), torch.zeros(3), 3)\n"
            "try:\n"
            "    S.seer_spmv(99, A, torch.zeros(5), torch.zeros(4), stream=0)\n"
            "except S.SeerError as e:\n"
            "    print('status', e.status)\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert out.stdout.strip() == "status -2", out.stderr


def test_a_structure_of_another_type_is_refused():
    """A Model where a Tree belongs (and so on) is an error, not memory read as something else."""
    A, x, ws = matrix(), torch.zeros(16), torch.zeros(64, dtype=torch.uint8)
    tree = S.Tree.constant(S.CSR_MP)
    model, plan = S.Model(tree), handles("prepared")[0]
    for call, right in ((S.seer_spmv_auto, tree), (S.seer_spmv_model, model), (S.seer_spmv_prepared, plan)):
        for h in (tree, model, plan):
            with pytest.raises(S.SeerError if h is right else C.ArgumentError):
                if call is S.seer_spmv_prepared:
                    call(h, A, x[:5], x[2:6], workspace=ws, stream=0)
                else:
                    call(A, h, x[:5], x[2:6], ws, stream=0)


class Odd:
    """Something with an address and a size of any type."""
    def __init__(self, address, size=64):
        self.address, self.size = address, size

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.size


@pytest.mark.parametrize("what", ["rows", "cols", "nnz"])
@pytest.mark.parametrize("value", [None, 4.0, "4"])
def test_sizes_that_are_no_integers_are_refused(what, value):
    A, x = matrix(), torch.zeros(16)
    setattr(A, what, value)
    with pytest.raises(TypeError):
        A.c_struct()
    with pytest.raises(TypeError):
        S.seer_spmv_auto(A, S.Tree.constant(S.CSR_MP), x[:5], x[2:6], torch.zeros(64, dtype=torch.uint8), stream=0)


def test_addresses_and_workspaces_that_are_none_are_refused():
    import numpy as np
    tree, x, ws = S.Tree.constant(S.CSR_MP), torch.zeros(16), torch.zeros(64, dtype=torch.uint8)

    def auto(A=None, xx=x[:5], w=ws):
        S.seer_spmv_auto(A or matrix(), tree, xx, x[2:6], w, stream=0)
    for bad in (Odd(16.0), Odd(np.int64(16)), Odd(ws.data_ptr(), None), Odd(ws.data_ptr(), 64.0)):
        with pytest.raises(TypeError):
            auto(w=bad)
    for w in (None, 3):                                                  # no optional argument of these two calls
        with pytest.raises(AttributeError):
            auto(matrix(rows=0, nnz=0), w=w)
        with pytest.raises(AttributeError):
            S.seer_spmv_model(matrix(rows=0, nnz=0), S.Model(tree), x[:5], x[2:6], w, stream=0)
    with pytest.raises(TypeError):
        auto(xx=Odd(16.0))
    A = matrix()
    A.row_ptr = Odd(16.0)
    with pytest.raises(TypeError):
        auto(A)
    for A, xx in ((matrix(), Odd(None)), (matrix(), x[:5])):              # a null x; x and y that overlap
        A.cols = np.int32(5)
        with pytest.raises(S.SeerError) as e:
            auto(A, xx)
        assert e.value.status == -1


def test_host_calls_work_without_the_native_marshalling():
    """Only the calls that go through it need the module; they say what is missing."""
    code = ("import torch, paper_2403_17017_amd as S\n"
            "from paper_2403_17017_amd import binding as B\n"
            "B._MARSHAL_PATH += '.not-built'\n"
            "print(S.seer_select(S.seer_known_features(4, 5, 3), S.Tree.constant(S.CSR_WO)))\n"
            "S.set_tuning('nt', -1)\n"
            "A = S.DeviceCSR(4, 5, torch.zeros(5, dtype=torch.int32), torch.zeros(3, dtype=torch.int32), torch.zeros(3), 3)\n"
            "try:\n"
            "    S.seer_spmv(0, A, torch.zeros(5), torch.zeros(4), stream=0)\n"
            "except ImportError as e:\n"
            "    print('.not-built is missing' in str(e))\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert out.stdout.split() == [str(S.CSR_WO), "True"], out.stderr


def test_the_current_stream_is_asked_for_only_where_torch_has_initialized(monkeypatch):
    """A forked child of a process that used the GPU must be refused by torch, not handed a stream."""
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 4711, raising=False)
    monkeypatch.setattr(torch.cuda, "_initialized", True)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: False)
    assert B._stream_handle(None) == 4711
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    with pytest.raises(RuntimeError, match="forked subprocess"):
        B._stream_handle(None)

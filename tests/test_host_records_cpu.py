"""The nb_system record of a batch keeps the host arrays that it points to, whatever the batch does
meanwhile (another call, another thread, new boxes), and only a record of the right type is taken
as the system argument."""

import ctypes
import threading

import numpy as np
import pytest

import nbtest_util as U
from paper_0902_0827_amd import nbhip as H

torch = pytest.importorskip("torch")


def _batch(**host):
    b = H.device_batch([U.small_chain()], dtype=torch.float64, device="cpu")
    for k, v in host.items():
        setattr(b, k, v)
    return b


def test_record_keeps_converted_arrays():
    # neither array is contiguous int64 / float64, so each record converts its own
    b = _batch(box=np.float32([[20.0, 21.0, 22.0]]))
    n = int(b.atom_offset[-1])
    b.atom_offset = np.int32([0, n])
    first = b.struct()
    b.box = np.float32([[30.0, 31.0, 32.0]])
    b.atom_offset = np.int32([0, n - 1])
    b.struct()
    churn = [np.full((1, 3), 7.0) for _ in range(64)] + [np.full(2, 7) for _ in range(64)]
    assert [first.box[k] for k in range(3)] == [20.0, 21.0, 22.0]
    assert [first.atom_offset[k] for k in range(2)] == [0, n]
    assert len(churn) == 128


def test_record_outlives_its_batch():
    first = _batch(box=[[20.0, 21.0, 22.0]]).struct()
    churn = [np.full((1, 3), 7.0) for _ in range(64)]
    assert [first.box[k] for k in range(3)] == [20.0, 21.0, 22.0]
    assert len(churn) == 64


def test_threads_share_a_batch():
    b = _batch(box=np.float32([[20.0, 21.0, 22.0]]))
    p = H.make_params(9.0, 0.34)
    want, bad = H.workspace_bytes(b, p), []

    def work():
        for _ in range(300):
            if H.workspace_bytes(b, p) != want:
                bad.append(1)

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_a_wrong_system_argument_is_refused():
    lib, p, n = H.load_library(), H.make_params(9.0, 0.34), ctypes.c_size_t()
    other = ctypes.create_string_buffer(4096)
    for wrong in (ctypes.byref(other), other, ctypes.byref(p), 4096, bytes(ctypes.sizeof(H.nb_system))):
        with pytest.raises(ctypes.ArgumentError):
            lib.nb_workspace_bytes(wrong, ctypes.byref(p), ctypes.byref(n))
    s = _batch().struct()
    for right in (s, ctypes.byref(s), ctypes.pointer(s)):
        assert lib.nb_workspace_bytes(right, ctypes.byref(p), ctypes.byref(n)) == H.NB_OK

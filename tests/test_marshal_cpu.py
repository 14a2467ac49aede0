"""A batch's job array without the native module: missing, unreadable or of another torch, it
is left out, and the binding's own loop fills the same array and reads the same codes."""
import ctypes

import pytest

import paper_2402_09481_amd as P
from paper_2402_09481_amd import _lib


class Words:
    def __init__(self, at, count):
        self.at, self.count = at, count

    def numel(self):
        return self.count


class Library:
    """extract_batch on the host: keeps the array, rejects every other job."""

    def extract_batch(self, handle, arr, count, flags, stream):
        self.jobs = [(j.kind, j.flags, j.n, j.m, j.x, j.y, j.z, j.status) for j in arr]
        for i in range(count):
            arr[i].err = -1 if i % 2 else 0
        return -1


@pytest.fixture
def no_module(monkeypatch, tmp_path):
    monkeypatch.setattr(_lib, "_marshal", None)
    monkeypatch.setattr(_lib, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    return tmp_path / "_marshal.so"


@pytest.mark.parametrize("file", [None, b"", b"no library"])
def test_batches_without_the_native_module(no_module, monkeypatch, file):
    if file is not None:
        no_module.write_bytes(file)
    assert _lib.marshal() is None
    monkeypatch.setattr(P, "_ptr", lambda t: t.at)
    ctx = P.Context.__new__(P.Context)
    ctx.handle, ctx.device, ctx._lib = None, 0, Library()
    jobs = [{"kind": "toeplitz", "n": 640, "m": 64, "x": Words(1 << 12, 10), "y": Words(2 << 12, 11), "z": Words(3 << 12, 1),
             "seed_order": "linear"}] * 3
    assert ctx.batch(jobs, stream=0) == (-1, [0, -1, 0])
    assert ctx._lib.jobs == [(0, P.EXT_SEED_LINEAR, 640, 64, 1 << 12, 2 << 12, 3 << 12, None)] * 3


def test_a_module_of_another_torch_is_left_out(monkeypatch):
    import torch
    monkeypatch.setattr(_lib, "_marshal", None)
    if _lib.marshal() is None:
        pytest.skip("the module is not built")
    assert _lib.marshal().fill([], ctypes.addressof((P.ExtJob * 1)()))
    monkeypatch.setattr(_lib, "_marshal", None)
    monkeypatch.setattr(torch, "__version__", "0.0")
    assert _lib.marshal() is None

"""Results of one GPU copied to another (no GPU needed: torch and the library are
stand-ins that record what is called): the copy kernel reads the result's memory,
so it is launched on the result's device, with that device current, and torch
moves the copy."""
import contextlib

import pytest
import torch

import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import _lib


class _Tensor:
    is_cuda = True

    def __init__(self, shape, device, dtype=torch.float32):
        self.shape, self.device, self.dtype = shape, torch.device(device), dtype

    def to(self, device):
        return _Tensor(self.shape, device)

    def dim(self):
        return len(self.shape)

    def contiguous(self):
        return self

    def data_ptr(self):
        return 16


class _Cuda:
    def __init__(self, calls):
        self.calls, self.now = calls, 0

    def current_device(self):
        return self.now

    @contextlib.contextmanager
    def device(self, d):
        d = torch.device(d)
        was, self.now = self.now, d.index
        yield
        self.now = was

    def current_stream(self, device):
        d = torch.device(device)
        if d.type != "cuda":
            raise ValueError("Expected a cuda device")
        index = self.now if d.index is None else d.index
        return type("S", (), {"cuda_stream": 100 + index})()


class _Torch:
    device, int32, float32 = torch.device, torch.int32, torch.float32

    def __init__(self, calls):
        self.cuda = _Cuda(calls)

    def empty(self, shape, dtype=None, device=None):
        return _Tensor(shape, device)


class _Lib:
    def __init__(self, calls, fake):
        self.calls, self.fake = calls, fake

    def ldni_result_axis(self, handle, axis, view):
        view._obj.w, view._obj.n_samples = 4, 10
        return 0

    def ldni_axis_copy(self, view, offsets, depth, normal, tri, stream):
        self.calls.append((stream.value, self.fake.cuda.now))
        return 0

    def _made(self, *args):
        args[-1]._obj.value = 1
        return 0

    ldni_sample = ldni_boolean = ldni_offset = _made

    def ldni_free(self, handle):
        pass


def _result(entry, device):
    """A library-owned result of that entry point from inputs on the device."""
    if entry == "sample":
        return ldni.ldni_sample(_Tensor((3, 3), device), _Tensor((1, 3), device, torch.int32), (0, 0, 0, 1, 1, 1), 4)
    l = ldni.LDNI(2, 4, 2, *[_Tensor((10,), device) for _ in range(4)])
    if entry == "boolean":
        return ldni.ldni_boolean(l, l, "union")
    return ldni.ldni_offset([l, l, l], (0, 0, 0, 1, 1, 1), 0.1)


@pytest.fixture
def calls(monkeypatch):
    log = []
    fake = _Torch(log)
    monkeypatch.setattr(ldni, "_torch", lambda: fake)
    monkeypatch.setattr(_lib, "lib", lambda: _Lib(log, fake))
    return log


@pytest.mark.parametrize("entry", ["sample", "boolean", "offset"])
@pytest.mark.parametrize("owner,asked,out", [
    ("cuda:0", None, "cuda"), ("cuda:0", "cuda:0", "cuda:0"), ("cuda:1", "cuda:1", "cuda:1"),
    ("cuda:1", "cuda:0", "cuda:0"), ("cuda:1", None, "cuda"), ("cuda:0", "cuda:1", "cuda:1")])
def test_copied_where_the_result_lives(calls, entry, owner, asked, out):
    k = torch.device(owner).index
    got = _result(entry, owner).to_torch(2, asked)
    assert calls == [(100 + k, k)]
    for t in (got.offsets, got.depth, got.normal, got.tri):
        assert t.device == torch.device(out)
    assert (got.axis, got.w) == (2, 4) and got.depth.shape == 10


def test_host_memory_stays_refused(calls):
    for owner in ("cuda:0", "cuda:1"):
        with pytest.raises(ValueError):
            _result("sample", owner).to_torch(0, "cpu")
    assert calls == []

"""ldni_axis_copy: all words of the four arrays and none beside them, for
sizes around a workgroup's 4,096 words, destinations off the 16-byte grid, and
the views that it refuses."""
import ctypes

import pytest
import torch

from paper_1009_0794_amd import _lib

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _words(n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-2**31, 2**31 - 1, (n,), dtype=torch.int32, generator=g).to(DEV)


@pytest.mark.parametrize("w,n", [(1, 0), (1, 1), (63, 4095), (64, 4096), (64, 4097), (127, 16385), (200, 100003)])
@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("rgb8", [False, True])
def test_copies(w, n, shift, rgb8):
    sizes = [w * w + 1, n, n if rgb8 else 3 * n, n]
    src = [_words(s + 8, k)[4:4 + s] for k, s in enumerate(sizes)]  # (16-byte aligned)
    dst = [torch.full((s + 16,), 7, dtype=torch.int32, device=DEV) for s in sizes]
    v = _lib.AxisView()
    v.w, v.n_samples = w, n
    v.offsets, v.depth, v.tri = src[0].data_ptr(), src[1].data_ptr(), src[3].data_ptr()
    if rgb8:
        v.normal_rgb8 = src[2].data_ptr()
    else:
        v.normal = src[2].data_ptr()
    _lib.check(_lib.lib().ldni_axis_copy(ctypes.byref(v), *[d[shift:].data_ptr() for d in dst], _stream()))
    for s, d in zip(src, dst):
        assert torch.equal(d[shift:shift + s.numel()], s)
        assert bool((d[:shift] == 7).all()) and bool((d[shift + s.numel():] == 7).all())


def test_refuses_missing_arrays():
    v = _lib.AxisView()
    x = _words(64, 0)
    L = _lib.lib()
    assert L.ldni_axis_copy(ctypes.byref(v), x.data_ptr(), None, None, None, _stream()) != 0  # no offsets
    v.w, v.n_samples, v.offsets = 2, 3, x.data_ptr()
    assert L.ldni_axis_copy(ctypes.byref(v), x.data_ptr(), x.data_ptr(), x.data_ptr(), x.data_ptr(), _stream()) != 0
    assert L.ldni_axis_copy(None, x.data_ptr(), None, None, None, _stream()) != 0

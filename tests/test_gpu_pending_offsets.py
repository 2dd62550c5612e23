"""The offsets of a pending Boolean operation or offset are in the caller's
memory.  If they change before the call is finished, the write pass fails or
writes other samples, but nothing beside the caller's arrays; the call is
released and the next one is right."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle import boolean as ob, offset as oo
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import _lib, meshgen as mg
from tests.test_gpu_offset import _same, _to_gpu

pytestmark = pytest.mark.gpu
BOX = (-1.0, -1.0, -1.0, 1.0, 1.0, 1.0)
W = 40
PAD = 64  # words around every output
DEVICE = 5

CHANGES = {
    "zero": lambda o, n: o.zero_(),
    "shifted": lambda o, n: o.add_(1000000),
    "largest": lambda o, n: o.fill_(-1),
    "reversed": lambda o, n: o.copy_(o.flip(0)),
    "one more at the end": lambda o, n: o[-1:].add_(1),
    "one word": lambda o, n: o[o.numel() // 2].fill_(0x7fffffff),
    "all in one pixel": lambda o, n: o[1:].fill_(n),
    "doubled": lambda o, n: o.mul_(2),
}


def _outputs(sizes):
    """(pointer table, guarded buffers) of arrays of that many words each."""
    bufs = [torch.full((s + 2 * PAD,), 7, dtype=torch.int32, device="cuda:0") for s in sizes]
    ptrs = (ctypes.c_void_p * 3)(*[b[PAD:].data_ptr() for b in bufs])
    return ptrs, bufs


def _untouched(bufs):
    return all(bool((b[:PAD] == 7).all()) and bool((b[b.numel() - PAD:] == 7).all()) for b in bufs)


def _finish(L, p, n):
    outs = [_outputs([k * s for s in n]) for k in (1, 3, 1)]
    rc = L.ldni_pending_finish(p, *[o[0] for o in outs])
    torch.cuda.synchronize()
    assert all(_untouched(o[1]) for o in outs)
    return rc, outs


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("change", [None, *CHANGES])
def test_boolean(change):
    A, B = (oracle.sample(*mg.icosphere(2, r, (x, 0.02, -0.01)), BOX, W, "z")[2] for r, x in ((0.5, -0.1), (0.4, 0.2)))
    ga, gb = _to_gpu(2, A), _to_gpu(2, B)
    L = _lib.lib()
    va, vb = ldni._view(ga), ldni._view(gb)
    offs = torch.empty(W * W + 1, dtype=torch.int32, device="cuda:0")
    p, n, ml = ctypes.c_void_p(), (ctypes.c_uint64 * 3)(), (ctypes.c_uint32 * 3)()
    _lib.check(L.ldni_boolean_begin(ctypes.byref(va), ctypes.byref(vb), 0, 1e-5, offs.data_ptr(), _stream(),
                                    ctypes.byref(p), n, ml))
    assert n[0] > 0
    if change:
        CHANGES[change](offs, int(n[0]))
    rc, outs = _finish(L, p, [int(n[0]), 0, 0])
    ref = ob.boolean(A, B, "union")
    if change in (None, "one word"):  # (the word of a pixel that is not the first of a wave's 64 is not read)
        assert rc == 0
        assert np.array_equal(outs[0][1][0][PAD:-PAD].cpu().numpy().view(np.uint32), ref.depth.view(np.uint32))
    elif change != "all in one pixel":  # (the waves' ranges still cover the outputs in order)
        assert rc == DEVICE
    _same(ldni.boolean(ga, gb, "union"), ref, "after")


@pytest.mark.parametrize("keep", [None, 3 * W * W * 8 * 16, 0])  # 128 end points a ray kept, 16, none
@pytest.mark.parametrize("change", [None, *CHANGES])
def test_offset(change, keep, monkeypatch):
    if keep is not None:
        monkeypatch.setenv("LDNI_OFFSET_KEEP_BYTES", str(keep))
    v, f = mg.concat([mg.icosphere(1, 0.05 + 0.07 * k, (0.0, 0.0, 0.0)) for k in range(12)])
    A = oracle.sample(v, f, BOX, W, "xyz")
    G = {a: _to_gpu(a, A[a]) for a in range(3)}
    L = _lib.lib()
    views = (_lib.AxisView * 3)(*[ldni._view(G[a]) for a in range(3)])
    bb = (ctypes.c_float * 6)(*BOX)
    offs = [torch.empty(W * W + 1, dtype=torch.int32, device="cuda:0") for _ in range(3)]
    optr = (ctypes.c_void_p * 3)(*[o.data_ptr() for o in offs])
    p, n, ml = ctypes.c_void_p(), (ctypes.c_uint64 * 3)(), (ctypes.c_uint32 * 3)()
    r = 0.01
    _lib.check(L.ldni_offset_begin(views, bb, r, 1e-5, optr, _stream(), ctypes.byref(p), n, ml))
    assert max(ml) > 16 and min(n) > 0
    if change:
        CHANGES[change](offs[1], int(n[1]))
    rc, outs = _finish(L, p, [int(x) for x in n])
    ref = oo.offset(A, BOX, W, r)
    if change is None:
        assert rc == 0
        for a in range(3):
            assert np.array_equal(outs[0][1][a][PAD:-PAD].cpu().numpy().view(np.uint32), ref[a].depth.view(np.uint32))
    else:
        assert rc == DEVICE
    got = ldni.offset(G, BOX, r)
    for a in range(3):
        _same(got[a], ref[a], f"after, axis {a}")

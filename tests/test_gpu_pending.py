"""Boolean operations and offsets written into the caller's arrays: the same
as the result that the library owns, empty results included, and a pending
call that is dropped leaves the next one as it was."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle import boolean as ob
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import _lib, meshgen as mg
from tests.test_gpu_boolean import _same, _to_gpu

pytestmark = pytest.mark.gpu
BOX = (-1.0, -1.0, -1.0, 1.0, 1.0, 1.0)


def _ball(r, x, w):
    v, f = mg.icosphere(2, r, (x, 0.02, -0.01))
    return {a: l for a, l in oracle.sample(v, f, BOX, w, "xyz").items()}


def _equal(x, y):
    assert x.w == y.w and x.max_layers == y.max_layers and x.axis == y.axis
    for p, q in ((x.offsets, y.offsets), (x.depth, y.depth), (x.normal, y.normal), (x.tri, y.tri)):
        assert p.dtype == q.dtype and p.shape == q.shape and torch.equal(p, q)


@pytest.mark.parametrize("op", ["union", "intersection", "difference"])
@pytest.mark.parametrize("w,x", [(1, 0.0), (33, 0.3), (64, 1.9)])
def test_boolean_equals_library_owned(op, w, x):
    A, B = _ball(0.5, -0.1, w), _ball(0.4, x, w)
    for a in range(3):
        ga, gb = _to_gpu(a, A[a]), _to_gpu(a, B[a])
        got = ldni.boolean(ga, gb, op)
        _equal(got, ldni.ldni_boolean(ga, gb, op).to_torch(a))
        _same(got, ob.boolean(A[a], B[a], op), f"{op} w={w} axis {a}")


@pytest.mark.parametrize("r", [0.2, -0.2, -0.8])  # (the last leaves nothing)
def test_offset_equals_library_owned(r):
    G = {a: _to_gpu(a, l) for a, l in _ball(0.5, 0.1, 30).items()}
    got, owned = ldni.offset(G, BOX, r), ldni.ldni_offset(G, BOX, r)
    for a in range(3):
        _equal(got[a], owned.to_torch(a))


def test_dropped_call():
    w = 40
    A, B = _ball(0.5, -0.1, w)[2], _ball(0.4, 0.2, w)[2]
    ga, gb = _to_gpu(2, A), _to_gpu(2, B)
    L = _lib.lib()
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    offs = torch.empty(w * w + 1, dtype=torch.int32, device="cuda:0")
    n, ml = (ctypes.c_uint64 * 3)(), (ctypes.c_uint32 * 3)()
    views = [ldni._view(ga), ldni._view(gb)]
    for given in (offs.data_ptr(), offs.data_ptr() + 4, None):
        p = ctypes.c_void_p()
        rc = L.ldni_boolean_begin(ctypes.byref(views[0]), ctypes.byref(views[1]), 0, 1e-5, given, st,
                                  ctypes.byref(p), n, ml)
        assert (rc == 0) == (given == offs.data_ptr()) and bool(p.value) == (rc == 0)
        L.ldni_pending_free(p)
    p = ctypes.c_void_p()
    _lib.check(L.ldni_boolean_begin(ctypes.byref(views[0]), ctypes.byref(views[1]), 0, 1e-5, offs.data_ptr(), st,
                                    ctypes.byref(p), n, ml))
    none = (ctypes.c_void_p * 3)()
    assert n[0] > 0 and L.ldni_pending_finish(p, none, none, none) != 0  # (releases it)
    _same(ldni.boolean(ga, gb, "union"), ob.boolean(A, B, "union"), "after dropped calls")

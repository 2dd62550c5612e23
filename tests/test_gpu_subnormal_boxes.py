"""Boxes of a few hundred of the smallest float32 numbers (2^-149), where the
pixel centres and node depths are rounded to a good part of a pixel: the
estimates of node and pixel numbers must leave room for that.  Bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import nodes as on
import paper_1009_0794_amd as ldni
from tests.test_gpu_nodes import _check as _check_nodes, _to_gpu
from tests.test_gpu_offset_cells import _axis, _check as _check_offset

pytestmark = pytest.mark.gpu
ULP = 2.0 ** -149


@pytest.mark.parametrize("w", [31, 33, 64])
@pytest.mark.parametrize("lo,size", [(0, 70), (0, 333), (-150, 300), (1000, 500), (-7, 5000)])
def test_nodes(w, lo, size):
    bbox = [lo * ULP] * 3 + [(lo + size) * ULP, (lo + size + 1) * ULP, (lo + 2 * size) * ULP]
    b = oracle.bbox_f32(bbox)
    rng = np.random.default_rng(w + size)
    L = []
    for a in range(3):
        d = on.node_depths(b[a], b[3 + a], w).astype(np.float32)
        near = np.concatenate([d, np.nextafter(d, np.float32(np.inf)), np.nextafter(d, np.float32(-np.inf))])
        cnt = rng.integers(0, 7, w * w)
        off = np.zeros(w * w + 1, np.uint32)
        off[1:] = np.cumsum(cnt)
        n = int(off[-1])
        dep = np.concatenate([np.sort(rng.choice(near, c)) for c in cnt]).astype(np.float32)
        L.append(oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=np.zeros((n, 3), np.float32),
                                 tri=np.zeros(n, np.int32)))
    _check_nodes([_to_gpu(a, L[a]) for a in range(3)], L, bbox, f"w={w} lo={lo} size={size}")


@pytest.mark.parametrize("lo,size", [(0, 70), (0, 333), (-150, 300), (-7, 5000)])
def test_offset(lo, size):
    w = 17
    box = [lo * ULP] * 3 + [(lo + size) * ULP] * 3
    rng = np.random.default_rng(size)
    L = {a: _axis(rng, w, size * ULP, 6, False) for a in range(3)}
    for r in (0.11 * size, -0.2 * size, 2 * size / w, 5.5 * size / w):
        _check_offset(L, box, w, float(np.float32(round(r) * ULP)), f"lo={lo} size={size} r={r}", eps=0.0)


@pytest.mark.parametrize("size", [101, 105, 134, 138])
def test_backward(size):
    """A sheet whose left edge is at the rounded-up centre of a tile's last
    column: its samples lie in two tiles (the gradient of the depths only, as
    that of the normals is beyond float32 here)."""
    w, box = 32, [0.0] * 3 + [size * ULP] * 3
    left = float(np.float32(15.5 * size / w * ULP)) / ULP
    assert left > 15.5 * size / w  # (rounded up)
    x1, y0, y1 = round(0.9 * size), round(0.1 * size), round(0.85 * size)
    v = np.array([[left, y0, 5], [x1, y0, 20], [x1, y1, 31], [left, y1, 11]]) * ULP
    v, f = v.astype(np.float32), np.array([[0, 1, 2], [0, 2, 3]], np.int32)
    ref = oracle.sample(v, f, box, w, "z")[2]
    pix = np.repeat(np.arange(w * w), np.diff(ref.offsets.astype(np.int64))) % w
    assert (pix == 15).any() and (pix > 15).any()
    gd = np.random.default_rng(size).normal(size=ref.n).astype(np.float32)
    want = oracle.backward(v, f, box, w, 2, ref, gd, np.zeros((ref.n, 3), np.float32))
    got = ldni.ldni_backward(torch.from_numpy(v).to("cuda:0"), torch.from_numpy(f).to("cuda:0"), box, w,
                             {2: _to_gpu(2, ref)}, {2: torch.from_numpy(gd).to("cuda:0")}).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max()

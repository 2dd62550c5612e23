"""Offsetting where the count pass merges chords by depth cells, bit for bit
against the oracle: rays with many overlapping chords, cell counts at the edges
of the rule that picks the cell size (and beyond it), boxes far from the
origin, and samples in front of and behind the box."""
import numpy as np
import pytest

import oracle
from oracle import offset as oo
import paper_1009_0794_amd as ldni
from tests.test_gpu_offset import BBOX, _random_axis, _same, _to_gpu

pytestmark = pytest.mark.gpu


def _axis(rng, w, size, n_max, dyadic, before=0.0):
    cnt = rng.integers(0, n_max, w * w)
    cnt[rng.random(w * w) < 0.3] = 0
    off = np.zeros(w * w + 1, np.uint32)
    off[1:] = np.cumsum(cnt)
    n = int(off[-1])
    dep = rng.integers(0, 64, n) * (size / 64) if dyadic else rng.uniform(-before, size + before, n)
    dep = dep.astype(np.float32)
    for p in range(w * w):
        dep[off[p]:off[p + 1]].sort()
    return oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=rng.normal(size=(n, 3)).astype(np.float32),
                           tri=rng.integers(0, 1 << 30, n).astype(np.int32))


def _check(L, box, w, r, label, eps=1e-5):
    ref = oo.offset(L, box, w, r, eps)
    got = ldni.offset({a: _to_gpu(a, L[a]) for a in range(3)}, box, r, eps)
    for a in range(3):
        _same(got[a], ref[a], f"{label} axis {a}")


@pytest.mark.parametrize("dyadic", [False, True])
@pytest.mark.parametrize("w,n_max,r", [(10, 30, 0.3), (10, 30, -0.3), (8, 60, 0.25), (12, 24, -0.17), (9, 12, 1.5),
                                       (7, 20, 0.5)])
def test_overlapping_chords(w, n_max, r, dyadic):
    rng = np.random.default_rng(w * n_max)
    _check({a: _axis(rng, w, 2.0, n_max, dyadic) for a in range(3)}, BBOX, w, r, f"w={w} r={r}")


@pytest.mark.parametrize("cells", [766, 767, 768, 1022, 1023, 1025])
def test_number_of_cells(cells):
    """Half-radius cells up to 768, three-quarter-radius cells up to there, then the sweep over all events."""
    w, r = 3, 2.0 / (0.5 * cells)
    rng = np.random.default_rng(cells)
    L = {a: _axis(rng, w, 2.0, 40, False) for a in range(3)}
    for a in range(3):  # neighbours that touch and overlap
        d = L[a].depth
        d[1::2] = np.maximum(d[1::2], d[:-1:2][:len(d[1::2])] + np.float32(0.4 * r))
        for p in range(w * w):
            d[L[a].offsets[p]:L[a].offsets[p + 1]].sort()
    for sign in (1, -1):
        _check(L, BBOX, w, sign * r, f"cells={cells}", eps=0.0)


@pytest.mark.parametrize("lo,size", [((1000.0, -5000.0, 0.1), 1.0), ((3.0e6, 1.0, -2.0e6), 16.0),
                                     ((1e-9, 1e-9, 1e-9), 3e-9)])
def test_boxes_far_from_the_origin(lo, size):
    w = 9
    box = [float(np.float32(x)) for x in lo]
    box += [float(np.float32(x + size)) for x in lo]
    rng = np.random.default_rng(3)
    L = {a: _axis(rng, w, box[3 + a] - box[a], 16, False) for a in range(3)}
    for r in (0.21 * size, -0.13 * size):
        _check(L, box, w, r, f"lo={lo} r={r}", eps=0.0)


@pytest.mark.parametrize("r", [0.3, -0.2])
def test_samples_outside_the_box(r):
    w = 8
    rng = np.random.default_rng(8)
    _check({a: _axis(rng, w, 2.0, 20, False, before=1.5) for a in range(3)}, BBOX, w, r, f"r={r}")

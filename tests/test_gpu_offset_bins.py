"""Offsetting at the edges of the spheres' binning, bit for bit against the
oracle: radii whose pixel ranges are just up to and just beyond the eight
pixels a side that a mask of hits holds, spheres that touch more rays than a
workgroup's table has entries, and rays and samples that do not fill a group
of eight, a wave's 64 pixels or a workgroup's 256 spheres."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_offset_cells import _check
from tests.test_gpu_offset import BBOX

pytestmark = pytest.mark.gpu


def _axis(rng, w, n_max):
    cnt = rng.integers(0, n_max + 1, w * w)
    off = np.zeros(w * w + 1, np.uint32)
    off[1:] = np.cumsum(cnt)
    dep = rng.uniform(0.0, 2.0, int(off[-1])).astype(np.float32)
    for p in range(w * w):
        dep[off[p]:off[p + 1]].sort()
    n = dep.size
    return oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=rng.normal(size=(n, 3)).astype(np.float32),
                           tri=rng.integers(0, 1 << 30, n).astype(np.int32))


@pytest.mark.parametrize("pixels", [0.3, 1.0, 2.0, 3.44, 3.5, 3.9, 3.96, 4.0, 4.5, 7.0])
@pytest.mark.parametrize("w", [1, 15, 32])
def test_radius_in_pixels(w, pixels):
    rng = np.random.default_rng(int(100 * pixels) + w)
    r = pixels * 2.0 / w
    _check({a: _axis(rng, w, 1) for a in range(3)}, BBOX, w, -r, f"w={w} r={pixels} pixels")


@pytest.mark.parametrize("pixels", [2.0, 3.9, 5.0])
def test_more_rays_than_entries(pixels):
    """Few samples all over a wide grid: 256 spheres hit some thousands of groups of rays."""
    w = 150
    rng = np.random.default_rng(7)
    L = {}
    for a in range(3):
        ax = _axis(rng, w, 1)
        keep = rng.random(ax.n) < 0.05
        pix = np.repeat(np.arange(w * w), np.diff(ax.offsets.astype(np.int64)))[keep]
        off = np.zeros(w * w + 1, np.uint32)
        off[1:] = np.cumsum(np.bincount(pix, minlength=w * w))
        L[a] = oracle.AxisLDNI(w=w, offsets=off, depth=ax.depth[keep], normal=ax.normal[keep], tri=ax.tri[keep])
    _check(L, BBOX, w, pixels * 2.0 / w, f"r={pixels} pixels")

"""Sampling where its launches change: bands (rows of tiles) of 4,096 pixels
and just more, cut into two or into up to eight parts, widths that leave a
part's first pixel inside a vector, tile counts around the one-launch tile
scan's 16,384, triangle chunks just below and at the 256 from which on a
workgroup takes all axes, and deep tiles, whose place items come first, beside
shallow ones.  Everything must equal the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import meshgen as mg
from tests.test_gpu_parity import _run, compare

pytestmark = pytest.mark.gpu

BALL = mg.icosphere(2, rot=mg.random_rotation(np.random.default_rng(5)))


@pytest.fixture(autouse=True)
def _auto_tiles():
    yield
    ldni.set_tile_shape(0, 0)


def _check(mesh, w, axes, tile):
    v, f = mesh
    bb = mg.cubic_bbox(v)
    ldni.set_tile_shape(*tile)
    compare(_run(v, f, bb, w, axes), oracle.sample(v, f, bb, w, axes), bb, label=f"w={w} {axes} {tile}")


@pytest.mark.parametrize("w,axes,tile", [
    (1, "xyz", (32, 32)), (128, "xyz", (32, 32)), (129, "xyz", (32, 32)), (255, "y", (32, 32)), (257, "xz", (32, 32)),
    (513, "xyz", (32, 32)), (1031, "xyz", (32, 32)), (1399, "xyz", (32, 32)), (1168, "xyz", (16, 16)),
    (1185, "xyz", (16, 16))])
def test_bands(w, axes, tile):
    _check(BALL, w, axes, tile)


@pytest.mark.parametrize("n_v", [255, 256])
@pytest.mark.parametrize("axes", ["xyz", "yz"])
def test_chunks(n_v, axes):
    """2 x 256 x 255 triangles are 255 chunks of 512, 2 x 256 x 256 are 256."""
    _check(mg.torus(256, n_v, 1.0, 0.4), 150, axes, (0, 0))


@pytest.mark.parametrize("shells", [3, 60, 400])
@pytest.mark.parametrize("w", [33, 200])
def test_deep_tiles(shells, w):
    """Concentric shells beside a ball: tiles of several place items and of one."""
    parts = [mg.icosphere(1, radius=0.1 + 0.2 * k / shells) for k in range(shells)]
    parts.append(mg.icosphere(1, radius=0.5, center=(2.0, 1.0, 0.3)))
    _check(mg.concat(parts), w, "xyz", (0, 0))

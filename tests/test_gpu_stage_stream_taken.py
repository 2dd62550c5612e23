"""Sampling with staged hits that by-pass the caches: at small ragged sizes (a
hook sets the number of entries from which they do to none, so that every staged
tile takes that way), and at a size whose own buffer is large enough, computed
here as the library computes it.  Bit for bit the oracle's samples."""
import numpy as np
import pytest
import torch

import oracle
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import meshgen as mg
from tests.test_gpu_parity import _run, compare

pytestmark = pytest.mark.gpu
EDGE = (256 << 20) // 12  # entries of 12 bytes that the 256 MiB cache holds


def _mesh(shells):
    """Concentric shells (tiles of several place items) beside a torus."""
    parts = [mg.icosphere(1, radius=0.1 + 0.2 * k / shells) for k in range(shells)]
    return mg.concat(parts + [mg.torus(24, 12, 0.7, 0.2, (1.5, 1.0, 0.3))])


@pytest.mark.parametrize("entries", [None, 2000])  # (with 2,000 some tiles are walked again)
@pytest.mark.parametrize("tile", [(16, 16), (32, 32)])
@pytest.mark.parametrize("w,shells", [(1, 3), (33, 60), (129, 3), (200, 300)])
def test_ragged_sizes(w, shells, tile, entries, monkeypatch):
    v, f = _mesh(shells)
    bb = mg.cubic_bbox(v)
    ref = oracle.sample(v, f, bb, w)
    monkeypatch.setenv("LDNI_STREAM_ENTRIES", "0")
    if entries:
        monkeypatch.setenv("LDNI_STAGE_ENTRIES", str(entries))
    try:
        ldni.set_tile_shape(*tile)
        for _ in range(2):
            compare(_run(v, f, bb, w), ref, bb, label=f"{w} {shells} {tile} {entries}")
    finally:
        ldni.set_tile_shape(0, 0)


def test_batch(monkeypatch):
    monkeypatch.setenv("LDNI_STREAM_ENTRIES", "0")
    meshes = [(*_mesh(k), w, tile) for k, w, tile in ((3, 77, (16, 16)), (200, 40, (32, 32)))]
    dev = [(torch.from_numpy(np.ascontiguousarray(v, np.float32)).to("cuda:0"),
            torch.from_numpy(np.ascontiguousarray(f, np.int32)).to("cuda:0"), mg.cubic_bbox(v), w, t)
           for v, f, w, t in meshes]
    b = ldni.sample_batch(dev, "xyz")
    for _ in range(2):
        b.run()
        for k, (v, f, w, _) in enumerate(meshes):
            bb = mg.cubic_bbox(v)
            compare({a: b.to_torch(k, a) for a in range(3)}, oracle.sample(v, f, bb, w), bb, label=f"mesh {k}")
    b.free()


@pytest.mark.parametrize("entries", [EDGE - 8, EDGE + 64])
def test_own_size(entries, monkeypatch):
    """Just below and above the limit, cut to that by the hook for smaller
    buffers; the first call on a shape asks for more."""
    n, w, images = (1200, 401, 3)
    v, f = mg.torus(n, n // 2, 1.0, 0.4, rot=mg.random_rotation(np.random.default_rng(3)))
    f = f[: len(f) - (entries > EDGE)]  # (another shape for either, so that no call has sized it yet)
    asked = min(16 * len(f) * images + 4 * w * w * images, 64 * w * w * images) + 65536
    assert asked > EDGE + 64
    monkeypatch.setenv("LDNI_STAGE_ENTRIES", str(entries))
    bb = mg.cubic_bbox(v)
    compare(_run(v, f, bb, w), oracle.sample(v, f, bb, w), bb, label=f"{entries}")

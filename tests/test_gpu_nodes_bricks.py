"""Node classification where its brick passes can go wrong, bit for bit
against the oracle: boxes whose node depths round together (the search behind
the float64 estimate), an output buffer without 16-byte alignment, rays with
more samples than a brick has nodes, and bricks the surface leaves uniform."""
import numpy as np
import pytest
import torch

import oracle
from oracle import nodes as on
import paper_1009_0794_amd as ldni
from tests.test_gpu_nodes import DEV, _check, _random_axis, _to_gpu, _unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [31, 33, 65])
@pytest.mark.parametrize("lo,size", [(1000.0, 4e-3), (-3.0e5, 1.0), (1e-12, 3e-12)])
def test_coarse_node_depths(w, lo, size):
    """Far from the origin neighbouring nodes share a float32 depth; every
    sample sits at or next to a node depth, below the first and beyond the last."""
    bbox = [lo, lo - size, 2 * lo, lo + size, lo, 2 * lo + 3 * size]
    b = oracle.bbox_f32(bbox)
    if not all(b[d] < b[3 + d] for d in range(3)):
        pytest.skip("the box is empty in float32")
    rng = np.random.default_rng(w)
    L = []
    for a in range(3):
        d = on.node_depths(b[a], b[3 + a], w).astype(np.float32)
        near = np.concatenate([d, np.nextafter(d, np.float32(np.inf)), np.nextafter(d, np.float32(-np.inf))])
        cnt = rng.integers(0, 7, w * w)
        off = np.zeros(w * w + 1, np.uint32)
        off[1:] = np.cumsum(cnt)
        dep = np.concatenate([np.sort(rng.choice(near, c)) for c in cnt]).astype(np.float32)
        n = int(off[-1])
        L.append(oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=np.zeros((n, 3), np.float32),
                                 tri=np.zeros(n, np.int32)))
    _check([_to_gpu(a, L[a]) for a in range(3)], L, bbox, f"w={w} lo={lo}")


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_bits(shift):
    """An output buffer at any 4-byte address is written in full and nothing beside it."""
    w, bbox = 40, [-1.0, -1.0, -1.0, 1.0, 1.0, 1.0]
    rng = np.random.default_rng(shift)
    b = oracle.bbox_f32(bbox)
    L = [_random_axis(rng, w, on.node_depths(b[a], b[3 + a], w)) for a in range(3)]
    inside, votes = on.classify(L[0], L[1], L[2], bbox, w)
    n = ldni.node_words(w)
    buf = torch.full((n + 8,), -1, dtype=torch.int32, device=DEV)
    _, n_in, n_split = ldni.classify_nodes([_to_gpu(a, L[a]) for a in range(3)], bbox, buf[shift:shift + n])
    got = buf.cpu().numpy()
    assert np.array_equal(_unpack(got[shift:shift + n], w), inside)
    assert (got[:shift] == -1).all() and (got[shift + n:] == -1).all()
    assert (n_in, n_split) == on.stats(inside, votes)


@pytest.mark.parametrize("w,deep", [(32, 300), (70, 2000), (257, 64)])
def test_deep_and_uniform_bricks(w, deep):
    """Rays with more samples than a brick holds nodes (many toggles of one
    node), next to rays that run through the grid inside or outside."""
    bbox = [-1.0, -1.0, -1.0, 1.0, 1.0, 1.0]
    rng = np.random.default_rng(w)
    L = []
    for a in range(3):
        cnt = np.where(np.arange(w * w) % w < w // 2, 2, 0)  # half the image: a slab through the whole grid
        cnt[rng.integers(0, w * w, 5)] = deep
        off = np.zeros(w * w + 1, np.uint32)
        off[1:] = np.cumsum(cnt)
        dep = [np.float32([-0.5, 2.5]) if c == 2 else np.sort(rng.uniform(-0.1, 2.1, c)).astype(np.float32)
               for c in cnt]
        n = int(off[-1])
        L.append(oracle.AxisLDNI(w=w, offsets=off, depth=np.concatenate(dep), normal=np.zeros((n, 3), np.float32),
                                 tri=np.zeros(n, np.int32)))
    _check([_to_gpu(a, L[a]) for a in range(3)], L, bbox, f"w={w} deep={deep}")

"""Node classification around the sizes at which its launches change: 512 bricks
(w = 256), up to which every brick is voted on and the vote reports the totals
itself, and 13 x 13 patches of rays (w = 416), up to which 1,024 threads sort a
patch.  Bit for bit against the oracle, totals included, also in calls that
follow each other with other sizes (the counters are cleared in the call)."""
import numpy as np
import pytest

import oracle
from oracle import nodes as on
from tests.test_gpu_nodes import BBOX, _check, _to_gpu

pytestmark = pytest.mark.gpu


def _axes(w, n_max, seed):
    rng = np.random.default_rng(seed)
    L = []
    for a in range(3):
        cnt = rng.integers(0, n_max + 1, w * w)
        cnt[rng.integers(0, w * w, 3)] = 90
        off = np.zeros(w * w + 1, np.uint32)
        off[1:] = np.cumsum(cnt)
        n = int(off[-1])
        dep = rng.uniform(-0.1, 2.1, n).astype(np.float32)
        pix = np.repeat(np.arange(w * w), cnt)
        dep = dep[np.lexsort((dep, pix))]
        L.append(oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=np.zeros((n, 3), np.float32),
                                 tri=np.zeros(n, np.int32)))
    return L


@pytest.mark.parametrize("w,n_max", [(1, 2), (31, 3), (32, 0), (33, 4), (64, 2), (65, 5), (255, 2), (256, 3), (257, 3),
                                     (416, 1), (417, 2)])
def test_sizes(w, n_max):
    L = _axes(w, n_max, w)
    _check([_to_gpu(a, L[a]) for a in range(3)], L, BBOX, f"w={w}")


def test_all_inside():
    """The largest totals of a grid that is voted on brick by brick: every node inside."""
    w = 256
    L = []
    for a in range(3):
        off = np.arange(w * w + 1, dtype=np.uint32) * 2
        dep = np.tile(np.float32([-1.0, 5.0]), w * w)
        L.append(oracle.AxisLDNI(w=w, offsets=off, depth=dep, normal=np.zeros((dep.size, 3), np.float32),
                                 tri=np.zeros(dep.size, np.int32)))
    inside, _ = _check([_to_gpu(a, L[a]) for a in range(3)], L, BBOX, "all inside")
    assert inside.all()


def test_one_after_the_other():
    grids = [(w, _axes(w, 2, w)) for w in (40, 300, 64, 420, 17)]
    G = [[_to_gpu(a, L[a]) for a in range(3)] for _, L in grids]
    for _ in range(2):
        for (w, L), g in zip(grids, G):
            _check(g, L, BBOX, f"w={w}")

"""The backward pass at its edges: tiles with more triangles than the LDS
table has slots (1,024), images of one tile and just more, triangle counts
that end inside a wave or a workgroup, one of the two gradients only, and
samples of triangles that the mesh does not have."""
import numpy as np
import pytest
import torch

import oracle
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import meshgen as mg

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BB = (-1.0, -1.0, -1.0, 1.0, 1.0, 1.0)


def _check(v, f, w, use_gd=True, use_gn=True, foreign=False, seed=0):
    vt = torch.from_numpy(np.ascontiguousarray(v, np.float32)).to(DEV)
    ft = torch.from_numpy(np.ascontiguousarray(f, np.int32)).to(DEV)
    res = ldni.sample(vt, ft, BB, w, "xyz")
    orc = oracle.sample(v, f, BB, w)
    rng = np.random.default_rng(seed)
    ref = np.zeros((len(v), 3))
    gds, gns = {}, {}
    for a in range(3):
        assert res[a].n == orc[a].n
        gd = rng.normal(size=res[a].n).astype(np.float32) * use_gd
        gn = rng.normal(size=(res[a].n, 3)).astype(np.float32) * use_gn
        if foreign:
            tri = res[a].tri.clone()
            tri[::3] = len(f) + 5
            tri[1::7] = -1
            res[a].tri = tri
            out = (tri.cpu().numpy() < 0) | (tri.cpu().numpy() >= len(f))
            ref += oracle.backward(v, f, BB, w, a, orc[a], np.where(out, 0, gd), np.where(out[:, None], 0, gn))
        else:
            ref += oracle.backward(v, f, BB, w, a, orc[a], gd, gn)
        if use_gd:
            gds[a] = torch.from_numpy(gd).to(DEV)
        if use_gn:
            gns[a] = torch.from_numpy(gn).to(DEV)
    g = ldni.ldni_backward(vt, ft, BB, w, res, gds, gns).cpu().numpy().astype(np.float64)
    scale = np.abs(ref).max()
    assert scale > 0 and np.abs(g - ref).max() <= 1e-4 * scale


@pytest.mark.parametrize("w", [16, 17, 48])
@pytest.mark.parametrize("level", [3, 5])
def test_full_tables(w, level):
    v, f = mg.icosphere(level, 0.9, (0.01, 0.02, -0.03), mg.random_rotation(np.random.default_rng(w)))
    _check(v, f, w)


@pytest.mark.parametrize("grads", [(True, False), (False, True)])
def test_one_gradient(grads):
    v, f = mg.torus(40, 20, 0.6, 0.25, rot=mg.random_rotation(np.random.default_rng(2)))
    _check(v, f, 37, *grads)


@pytest.mark.parametrize("n_u,n_v", [(3, 3), (8, 4), (16, 8), (43, 3)])  # 18, 64, 256, 258 triangles
def test_triangle_counts(n_u, n_v):
    v, f = mg.torus(n_u, n_v, 0.6, 0.25, rot=mg.random_rotation(np.random.default_rng(3)))
    _check(v, f, 33)


def test_foreign_triangles():
    v, f = mg.icosphere(2, 0.8, rot=mg.random_rotation(np.random.default_rng(4)))
    _check(v, f, 40, foreign=True)

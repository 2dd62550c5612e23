"""Sampling with a staging buffer just below and above the size from which its
accesses by-pass the caches (the buffer's size by a test hook; what it holds is
less): the same samples as the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1009_0794_amd import meshgen as mg
from tests.test_gpu_parity import _run, compare

pytestmark = pytest.mark.gpu
EDGE = (256 << 20) // 12


@pytest.mark.parametrize("entries", [EDGE - 8, EDGE + 64])
@pytest.mark.parametrize("shells", [1, 40])
def test_streamed_stage(entries, shells, monkeypatch):
    # (a mesh of 1.4 M triangles or more asks for such a buffer on its first call)
    n = 1200
    v, f = mg.concat([mg.torus(n, n // 2, 1.0, 0.4, rot=mg.random_rotation(np.random.default_rng(3)))] +
                     [mg.icosphere(1, 0.1 + 0.005 * k) for k in range(shells)])
    bb, w = mg.cubic_bbox(v), 301
    monkeypatch.setenv("LDNI_STAGE_ENTRIES", str(entries))
    ref = oracle.sample(v, f, bb, w)
    for _ in range(2):  # (the second call's buffer follows the first's demand)
        compare(_run(v, f, bb, w), ref, bb, label=f"{entries} {shells}")

"""A table of place items that is too small (by a test hook; the library sizes it
by a bound that sampling cannot pass) fails the call instead of leaving samples
out, and the next call is right."""
import pytest

import oracle
import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import meshgen as mg
from tests.test_gpu_parity import _run, compare

pytestmark = pytest.mark.gpu
DEVICE = 5


@pytest.mark.parametrize("cap", [0, 1, 5, 11, 12, 1000])
def test_short_table(cap, monkeypatch):
    v, f = mg.icosphere(2)
    bb, w = mg.cubic_bbox(v), 64
    ref = oracle.sample(v, f, bb, w)
    try:
        ldni.set_tile_shape(32, 32)  # 4 tiles of each image, each met by the ball: 12 items
        monkeypatch.setenv("LDNI_PLACE_ITEMS", str(cap))
        if cap < 12:
            with pytest.raises(ldni.LDNIError) as e:
                _run(v, f, bb, w)
            assert e.value.code == DEVICE
            monkeypatch.delenv("LDNI_PLACE_ITEMS")
        compare(_run(v, f, bb, w), ref, bb, label=f"{cap}")
    finally:
        ldni.set_tile_shape(0, 0)

"""A batch whose write pass disagrees with its count pass (by a test hook: the
first image's counts are lost on the device) fails; without it the results are
the single calls'."""
import pytest
import torch

import paper_1009_0794_amd as ldni
from paper_1009_0794_amd import meshgen as mg

pytestmark = pytest.mark.gpu
DEVICE = 5


@pytest.mark.parametrize("axes", ["z", "xyz"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32)])
def test_lost_counts(axes, tile, monkeypatch):
    meshes = []
    for level, w in ((2, 64), (3, 50)):
        v, f = mg.icosphere(level)
        meshes.append((torch.from_numpy(v).to("cuda:0", torch.float32), torch.from_numpy(f).to("cuda:0", torch.int32),
                       mg.cubic_bbox(v), w, tile))
    monkeypatch.setenv("LDNI_FAULT", "counts")
    with pytest.raises(ldni.LDNIError) as e:
        ldni.sample_batch(meshes, axes)
    assert e.value.code == DEVICE
    monkeypatch.delenv("LDNI_FAULT")
    b = ldni.sample_batch(meshes, axes)
    for _ in range(2):
        b.run()
        for k, (v, f, bb, w, _) in enumerate(meshes):
            one = ldni.sample(v, f, bb, w, axes)
            for a in one:
                got = b.to_torch(k, a)
                assert got.max_layers == one[a].max_layers
                for x, y in ((got.offsets, one[a].offsets), (got.depth, one[a].depth), (got.normal, one[a].normal),
                             (got.tri, one[a].tri)):
                    assert torch.equal(x, y)
    b.free()

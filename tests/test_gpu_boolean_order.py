"""Boolean operations on lists with one fault each: two neighbours swapped, or a
NaN, in one pixel deep enough that its wave's samples are merged in equal parts.
Such lists are merged one sample after the other, whichever part the fault lies
in, also when it lies between two pixels (where it is none) or in the unpaired
last sample of a list (which is ignored)."""
import numpy as np
import pytest

import oracle
from oracle import boolean as ob
import paper_1009_0794_amd as ldni
from tests.test_gpu_boolean import OPS, _same, _to_gpu
from tests.test_gpu_boolean_batches import _lists, _merge

pytestmark = pytest.mark.gpu
W = 8  # (one wave)


def _sides(rng, deep):
    """Two images of shallow pixels and one (or two) of `deep` samples a side,
    all lists of disjoint values."""
    sides = []
    for k in range(2):
        cnt = rng.integers(0, 3, W * W)
        cnt[[20, 41]] = deep, deep + k
        sides.append(_lists(rng, cnt, lambda c: np.sort(rng.permutation(4 * max(c, 4))[:c]) * 0.25 + 0.125 * k))
    return sides


def _compare(a, b, label):
    ga, gb = _to_gpu(1, a), _to_gpu(1, b)
    for op in OPS:
        got = ldni.boolean(ga, gb, op, 1e-5)
        off = got.offsets.cpu().numpy().view(np.uint32).astype(np.int64)
        dep, tri = got.depth.cpu().numpy(), got.tri.cpu().numpy()
        for p in range(W * W):
            sa, sb = (slice(int(x.offsets[p]), int(x.offsets[p + 1])) for x in (a, b))
            ref = _merge(a.depth[sa], b.depth[sb], op, float(np.float32(1e-5)))
            assert off[p + 1] - off[p] == len(ref), (label, op, p)
            for k, (side, i) in enumerate(ref):
                x, q = (a, sa.start + i) if side == 0 else (b, sb.start + i)
                o = off[p] + k
                assert dep[o].view(np.uint32) == x.depth[q].view(np.uint32), (label, op, p, k)
                assert tri[o] == (x.tri[q] if side == 0 else -1 - x.tri[q]), (label, op, p, k)


@pytest.mark.parametrize("deep", [12, 31, 64, 200])
@pytest.mark.parametrize("fault", ["swap", "nan"])
def test_one_fault(deep, fault):
    rng = np.random.default_rng(deep)
    for trial in range(24):
        sides = _sides(rng, deep)
        x = sides[trial & 1]
        at = int(x.offsets[20]) + int(rng.integers(0, deep - 1))
        if fault == "swap":
            x.depth[[at, at + 1]] = x.depth[[at + 1, at]]
        else:
            x.depth[at] = np.nan
        _compare(*sides, f"{deep} {fault} {trial}")


def test_no_fault():
    """Falls between pixels and single (unpaired) NaNs are none: the oracle's result."""
    rng = np.random.default_rng(5)
    a, b = _sides(rng, 50)
    _same(ldni.boolean(_to_gpu(1, a), _to_gpu(1, b), "union", 1e-5), ob.boolean(a, b, "union", 1e-5), "plain")
    for x in (a, b):
        one = np.flatnonzero(np.diff(x.offsets.astype(np.int64)) == 1)
        x.depth[x.offsets[one]] = np.nan
    assert len(one) > 0
    _compare(a, b, "unpaired NaN")

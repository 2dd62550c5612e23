"""Boolean operations where the count pass changes its way: pixels around the
LDS batch's 1,024 samples and deeper, batches that end inside a wave, infinite
depths, and lists that are not ascending or hold NaN, which are merged one
sample after the other (the merge written out below)."""
import numpy as np
import pytest

import oracle
from oracle import boolean as ob
import paper_1009_0794_amd as ldni
from tests.test_gpu_boolean import OPS, _same, _to_gpu

pytestmark = pytest.mark.gpu


def _lists(rng, counts, values):
    off = np.zeros(len(counts) + 1, np.uint32)
    off[1:] = np.cumsum(counts)
    n = int(off[-1])
    dep = np.concatenate([values(c) for c in counts] + [np.zeros(0)]).astype(np.float32)
    return oracle.AxisLDNI(w=int(len(counts) ** 0.5), offsets=off, depth=dep,
                           normal=rng.normal(size=(n, 3)).astype(np.float32),
                           tri=rng.integers(0, 1 << 30, n).astype(np.int32))


@pytest.mark.parametrize("deep", [(511, 513), (512, 512), (1023, 1), (1024, 0), (0, 1025), (1025, 1024), (3000, 40)])
def test_deep_pixels(deep):
    """One pixel with that many samples of A and of B among shallow ones."""
    w = 12
    rng = np.random.default_rng(sum(deep))
    sides = []
    for n in deep:
        cnt = rng.integers(0, 20, w * w)
        cnt[70] = n
        sides.append(_lists(rng, cnt, lambda c: np.sort(rng.integers(0, max(8, 2 * c), c)) * 0.125))
    a, b = sides
    ga, gb = _to_gpu(2, a), _to_gpu(2, b)
    for op in OPS:
        for eps in (0.0, 0.2):
            _same(ldni.boolean(ga, gb, op, eps), ob.boolean(a, b, op, eps), f"{deep} {op} eps={eps}")


@pytest.mark.parametrize("per", [8, 15, 16, 17, 33])
def test_batches_end_inside_a_wave(per):
    """64 pixels hold more samples than a batch: 8 to 33 of each list per pixel."""
    w = 16
    rng = np.random.default_rng(per)
    a, b = (_lists(rng, np.full(w * w, per), lambda c: np.sort(rng.uniform(0, 4, c))) for _ in range(2))
    ga, gb = _to_gpu(0, a), _to_gpu(0, b)
    for op in OPS:
        _same(ldni.boolean(ga, gb, op, 1e-2), ob.boolean(a, b, op, 1e-2), f"{per} {op}")


def _merge(da, db, op, eps):
    """The end points of one pixel: (enter, exit) pairs as (list, index)."""
    da, db = da[:len(da) & ~1], db[:len(db) & ~1]
    holds = {"union": lambda x, y: x or y, "intersection": lambda x, y: x and y,
             "difference": lambda x, y: x and not y}[op]
    ia = ib = 0
    ina = inb = res = False
    out, enter = [], None
    while ia < len(da) or ib < len(db):
        first_a = ia < len(da) and (ib >= len(db) or not (db[ib] < da[ia]))
        d, ref = (da[ia], (0, ia)) if first_a else (db[ib], (1, ib))
        if first_a:
            ina, ia = not ina, ia + 1
        else:
            inb, ib = not inb, ib + 1
        while ia < len(da) and da[ia] == d:
            ina, ia = not ina, ia + 1
        while ib < len(db) and db[ib] == d:
            inb, ib = not inb, ib + 1
        r = holds(ina, inb)
        if r == res:
            continue
        res = r
        if r:
            enter = (d, ref)
            continue
        with np.errstate(invalid="ignore"):
            th = float(d) - float(enter[0])
        if th > 0.0 and th >= eps:
            out += [enter[1], ref]
    return out


@pytest.mark.parametrize("kind", ["infinite", "nan", "unsorted"])
@pytest.mark.parametrize("deep", [False, True])
def test_lists_out_of_the_ordinary(kind, deep):
    w = 10
    rng = np.random.default_rng(len(kind) + deep)

    def values(c):
        v = np.sort(rng.integers(0, 12, c) * 0.25)
        if c and rng.random() < 0.3:
            if kind == "infinite":
                v[:rng.integers(0, c + 1)] = -np.inf
                v[rng.integers(0, c + 1):] = np.inf
                v.sort()
            elif kind == "nan":
                v[rng.integers(0, c)] = np.nan
            else:
                rng.shuffle(v)
        return v

    sides = []
    for _ in range(2):
        cnt = rng.integers(0, 9, w * w)
        if deep:
            cnt[[17, 55]] = (700, 1300)
        sides.append(_lists(rng, cnt, values))
    a, b = sides
    ga, gb = _to_gpu(1, a), _to_gpu(1, b)
    for op in OPS:
        got = ldni.boolean(ga, gb, op, 1e-5)
        off = got.offsets.cpu().numpy().view(np.uint32).astype(np.int64)
        dep, nrm, tri = got.depth.cpu().numpy(), got.normal.cpu().numpy(), got.tri.cpu().numpy()
        eps = float(np.float32(1e-5))
        for p in range(w * w):
            sa, sb = (slice(int(x.offsets[p]), int(x.offsets[p + 1])) for x in (a, b))
            ref = _merge(a.depth[sa], b.depth[sb], op, eps)
            assert off[p + 1] - off[p] == len(ref), (op, p)
            for k, (side, i) in enumerate(ref):
                x, q = (a, sa.start + i) if side == 0 else (b, sb.start + i)
                o = off[p] + k
                sign = np.float32(-1 if side and op == "difference" else 1)
                assert dep[o].view(np.uint32) == x.depth[q].view(np.uint32)
                assert np.array_equal(nrm[o], sign * x.normal[q])
                assert tri[o] == (x.tri[q] if side == 0 else -1 - x.tri[q])

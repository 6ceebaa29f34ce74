"""A pair's J does not depend on the pairs beside it in the call, bit for bit:
the paths that share a kind of pair (a wavefront's group, a workgroup, a
wavefront of the launch for large pairs) are chosen by the call's counts."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2511_16576_amd import datagen as dg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_16576_amd import polymh
    polymh.check_device()
    return polymh


def _stars(counts, side, lo, hi, seed):
    rng = np.random.default_rng(seed)
    counts = np.asarray(counts)
    radii = rng.uniform(lo, hi, counts.size) * side
    c = side // 2 + rng.uniform(-0.2, 0.2, (counts.size, 2)) * side
    ps = dg.star_polygons(rng, counts, c.astype(np.int64), radii)
    return [ps.xy[ps.offsets[i]:ps.offsets[i + 1]] for i in range(ps.n)]


def _refine(pm, D, Q, ids, n_cand=None, **kw):
    import torch
    ids = np.asarray(ids, dtype=np.int32)
    off = torch.tensor([0, ids.size], dtype=torch.int64).cuda()
    return pm.refine(D, Q, off, torch.from_numpy(ids).cuda(), n_cand=n_cand, **kw)[:ids.size].cpu().numpy()


@pytest.mark.parametrize("m", [100, 513, 900, 1024])
def test_pairs_beyond_a_group_beside_larger_ones(pm, orc, m):
    """513 to 1,024 edges on one side at least: 512 of them in a call and more,
    with a larger pair beside them and without."""
    side = 1 << 24
    sizes = [513, 514, 520, 600, 700, 767, 768, 800, 1000, 1015, 1016, 1017, 1023, 1024]
    data = _stars(sizes, side, 0.2, 0.3, 3) + _stars([600, 1000], side, 0.01, 0.02, 4) + _stars([900], side, 0.4, 0.45, 5)
    data += [data[3][::-1]] + _stars([1100], side, 0.2, 0.3, 6)
    ds, qs = dg.from_list(data), dg.from_list(_stars([m], side, 0.2, 0.3, 9))
    n = ds.n - 1                                   # the last one is larger
    want = orc.jaccard_candidates(ds, qs, np.array([0, ds.n]), np.arange(ds.n, dtype=np.int32))
    D, Q = pm.to_device(ds), pm.to_device(qs)
    alone = _refine(pm, D, Q, np.arange(n))
    assert np.all(np.abs(alone - want[:n]) <= 1e-9 * want[:n] + 1e-12)
    for count in (n, 512, 513, 2000):
        for larger in (0, 1):
            ids = np.concatenate([np.arange(count) % n, np.full(larger, n)])
            got = _refine(pm, D, Q, ids)
            assert np.array_equal(got[:count], alone[ids[:count]]), (count, larger)


def _clipped_area2(ring, convex):
    """Twice the area of a ring inside a convex counter-clockwise one, exact
    (Sutherland and Hodgman's clipping; the edges it adds cancel)."""
    pts = [(Fraction(int(x)), Fraction(int(y))) for x, y in ring]
    for (ax, ay), (bx, by) in zip(convex, np.roll(convex, -1, axis=0)):
        ax, ay, bx, by = int(ax), int(ay), int(bx), int(by)
        side = [(bx - ax) * (y - ay) - (by - ay) * (x - ax) for x, y in pts]
        out = []
        for i, p in enumerate(pts):
            j = (i + 1) % len(pts)
            q, s, t = pts[j], side[i], side[j]
            if s >= 0:
                out.append(p)
            if (s > 0 > t) or (s < 0 < t):
                u = s / (s - t)
                out.append((p[0] + u * (q[0] - p[0]), p[1] + u * (q[1] - p[1])))
        pts = out
    return sum(a[0] * b[1] - b[0] * a[1] for a, b in zip(pts, pts[1:] + pts[:1]))


@pytest.mark.parametrize("extra", [0, 300])
@pytest.mark.parametrize("many", [False, True])
def test_small_polygons_against_a_thin_query(pm, extra, many):
    """Data polygons of some 100 lattice units against a thin query across a
    box of 2^25: a crossing's term is rounded by the pair's size, not the
    query's (all of a crossing's products here are below 2^18, whose terms the
    refinement knows to 2^-48 relative)."""
    w = 1 << 25
    low = [(8 * i, 7 * i + i % 3) for i in range(24)] + [(w * (i + 1) // (extra + 2), w * (i + 1) // (extra + 2))
                                                         for i in range(extra)] + [(w, w)]
    up = [(x - 20, y + 24) for x, y in low]
    q = np.array(low + up[::-1])
    ring = np.array([(6, 1), (3, 6), (-2, 7), (-6, 2), (-5, -2), (-2, -6), (2, -5), (7, -2)])
    data = [ring + (8 * i + dx, 7 * i + dy) for i in range(2, 20) for dx, dy in ((1, 0), (4, -3), (-18, 21), (-24, 20))]
    aq = sum(int(a[0]) * int(b[1]) - int(b[0]) * int(a[1]) for a, b in zip(q, np.roll(q, -1, axis=0)))
    want = []
    for p in data:
        ap = sum(int(a[0]) * int(b[1]) - int(b[0]) * int(a[1]) for a, b in zip(p, np.roll(p, -1, axis=0)))
        inter = _clipped_area2(q, p)
        assert 0 < inter < ap
        want.append(float(inter / (ap + aq - inter)))
    # `many` beside a larger pair: more than workgroups take
    big = [np.stack([np.rint(2000 * np.cos(t)), np.rint(2000 * np.sin(t))], 1).astype(np.int64)
           for t in [np.arange(1100) * (2 * np.pi / 1100)]]
    ds, qs = dg.from_list(data + big), dg.from_list([q])
    ids = np.concatenate([np.arange(600) % len(data), [len(data)]]) if many else np.arange(len(data))
    got = _refine(pm, pm.to_device(ds), pm.to_device(qs), ids)[:600 if many else len(data)]
    ref = np.array(want)[ids[:got.size]]
    assert np.all(np.abs(got - ref) <= 1e-9 * ref)


def test_more_large_pairs_than_the_list_holds(pm, orc):
    """2^20 list entries, taken a wavefront's lanes at a time, and pairs past
    them, which are computed in place."""
    side = 1 << 20
    data = _stars([600, 40, 530], side, 0.2, 0.3, 31) + [dg.rectangle(0, 0, 9, 9)]
    ds, qs = dg.from_list(data), dg.from_list(_stars([520], side, 0.2, 0.3, 32))
    want = orc.jaccard_candidates(ds, qs, np.array([0, 4]), np.arange(4, dtype=np.int32))
    assert (want[:3] > 0).all()
    ids = np.arange((1 << 20) * 4 // 3 + 3000) % 4    # three of four go to the list
    got = _refine(pm, pm.to_device(ds), pm.to_device(qs), ids)
    assert np.all(np.abs(got - want[ids]) <= 1e-9 * want[ids] + 1e-12)


@pytest.mark.parametrize("count", [1, 40, 2500])
def test_units_of_split_pairs(pm, orc, count):
    """Pairs split into units (from a few a call to more than 64 a wavefront):
    each against the oracle, and the same bits however many there are; pairs
    too wide for the split ones' arithmetic beside them."""
    side = 1 << 24
    data = _stars([3000, 1500, 5000], side, 0.2, 0.3, 41)
    wide = np.rint(data[0].astype(float) * 5).astype(np.int64)      # beyond 2^26 across: split by slices
    ds, qs = dg.from_list(data + [wide]), dg.from_list(_stars([2500], side, 0.2, 0.3, 42))
    want = orc.jaccard_candidates(ds, qs, np.array([0, 4]), np.arange(4, dtype=np.int32))
    assert (want[:3] > 0).all()
    D, Q = pm.to_device(ds), pm.to_device(qs)
    ids = np.concatenate([np.arange(count) % 3, np.full(min(count, 40), 3)])
    got = _refine(pm, D, Q, ids)
    assert np.all(np.abs(got - want[ids]) <= 1e-9 * want[ids] + 1e-12)
    one = np.array([_refine(pm, D, Q, [i])[0] for i in range(4)])
    assert np.array_equal(got, one[ids])

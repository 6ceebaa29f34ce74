"""Refinement where a wavefront's candidates are packed into groups: data
polygons about the sizes that fill a group's chunks, rings far apart in size,
pairs that leave a group (disjoint, degenerate, wide, beyond the tiled form),
more candidates than lanes, and any place in a list.  Against the oracle
(within 1e-9 relative, as elsewhere); a tiled pair's value does not depend on
its neighbours, bit for bit."""
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


def _data(side):
    big = _stars([3, 7, 8, 9, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 504, 505, 511, 512, 513, 700],
                 side, 0.15, 0.3, 1)
    small = _stars([4, 8, 20, 40], side, 0.01, 0.03, 2)
    q = side // 4
    odd = [dg.rectangle(0, 0, side - 1, side - 1),            # around every query
           dg.rectangle(0, 0, 5, 5), dg.rectangle(side - 9, 0, side - 1, 9),
           np.array([[q, q], [2 * q, 2 * q], [3 * q, 3 * q]]),    # no area
           np.array([[q, q], [q, q], [3 * q, q], [2 * q, 3 * q]])]
    return big + small + odd + [p[::-1] for p in big[:6]]


def _refine(pm, D, Q, off, ids):
    import torch
    J = pm.refine(D, Q, torch.from_numpy(off).cuda(), torch.from_numpy(ids.astype(np.int32)).cuda())
    return J.cpu().numpy()


@pytest.mark.parametrize("m", [3, 8, 9, 64, 100, 511, 512, 513])
@pytest.mark.parametrize("side", [1 << 10, 1 << 25])
def test_groups(pm, orc, m, side):
    import torch
    data, queries = _data(side), _stars([m, m], side, 0.15, 0.3, 10 + m)
    wide = [p.astype(np.int64) * 30 for p in data[:4]] if side > 1 << 20 else []
    ds, qs = dg.from_list(data + wide), dg.from_list(queries)
    D, Q = pm.to_device(ds), pm.to_device(qs)
    n = ds.n
    want = orc.jaccard_candidates(ds, qs, np.array([0, n, 2 * n]), np.tile(np.arange(n, dtype=np.int32), 2))
    rng = np.random.default_rng(m)
    first = None
    for per in (n, 70 * n, 700 * n):        # up to 100 candidates a wavefront
        order = np.concatenate([rng.permutation(n) if per > n else np.arange(n) for _ in range(2 * per // n)])
        got = _refine(pm, D, Q, np.array([0, per, 2 * per]), order)
        ref = np.concatenate([want[:n][order[:per]], want[n:][order[per:]]])
        assert np.all(np.abs(got - ref) <= 1e-9 * ref + 1e-12), per
        if first is None:
            first = got
        tiled = (np.diff(ds.offsets)[order] <= 512) & (m <= 512)
        same = np.concatenate([first[:n][order[:per]], first[n:][order[per:]]])
        assert np.array_equal(got[tiled], same[tiled]), per
    assert (want > 0).sum() >= 40


def test_short_lists(pm, orc):
    """1, 2, ... candidates a query, some queries without any."""
    data, side = _data(1 << 12), 1 << 12
    queries = _stars(np.arange(3, 43), side, 0.1, 0.3, 5)
    ds, qs = dg.from_list(data), dg.from_list(queries)
    off = np.concatenate([[0], np.cumsum([i % 9 for i in range(40)])]).astype(np.int64)
    ids = np.random.default_rng(0).integers(0, ds.n, off[-1]).astype(np.int32)
    want = orc.jaccard_candidates(ds, qs, off, ids)
    got = _refine(pm, pm.to_device(ds), pm.to_device(qs), off, ids)
    assert np.all(np.abs(got - want) <= 1e-9 * want + 1e-12)


@pytest.mark.parametrize("m", [3, 513, 700, 1017, 1023, 1024, 1025])
@pytest.mark.parametrize("side", [1 << 18, 1 << 25])
def test_pairs_beyond_a_group(pm, orc, m, side):
    """513 to 1,024 edges a side (a workgroup a pair) beside smaller and larger
    ones: about the chunk edges, contained, containing, apart, without area."""
    data = _stars([3, 9, 512, 513, 520, 767, 768, 1016, 1017, 1023, 1024, 1025, 1600], side, 0.15, 0.3, 3)
    data += _stars([600, 900], side, 0.01, 0.02, 4) + _stars([600, 1000], side, 0.4, 0.45, 6)
    q = side // 4
    flat = np.stack([np.linspace(q, 3 * q, 600).astype(np.int64)] * 2, axis=1)
    data += [flat, dg.rectangle(0, 0, side - 1, side - 1), data[5][::-1]]
    ds, qs = dg.from_list(data), dg.from_list(_stars([m, max(3, m - 1)], side, 0.15, 0.3, 20 + m))
    n = ds.n
    want = orc.jaccard_candidates(ds, qs, np.array([0, n, 2 * n]), np.tile(np.arange(n, dtype=np.int32), 2))
    D, Q = pm.to_device(ds), pm.to_device(qs)
    rng, first = np.random.default_rng(m), None
    for rep in range(3):
        order = np.concatenate([rng.permutation(n) if rep else np.arange(n) for _ in range(2)])
        got = _refine(pm, D, Q, np.array([0, n, 2 * n]), order)
        ref = np.concatenate([want[:n][order[:n]], want[n:][order[n:]]])
        assert np.all(np.abs(got - ref) <= 1e-9 * ref + 1e-12), rep
        first = got if first is None else first
        whole = (np.diff(ds.offsets)[order] <= 1024) & (m <= 1024)
        same = np.concatenate([first[:n][order[:n]], first[n:][order[n:]]])
        assert np.array_equal(got[whole], same[whole]), rep


@pytest.mark.parametrize("larger", [0, 1])
@pytest.mark.parametrize("n", [500, 513, 700])
def test_many_pairs_beyond_a_group(pm, orc, n, larger):
    """As many pairs of 513 to 1,024 edges as workgroups take beside a larger
    pair, more, and more without one."""
    side = 1 << 20
    data = _stars([600, 1024, 1100], side, 0.2, 0.3, 8)
    ds, qs = dg.from_list(data), dg.from_list(_stars([520], side, 0.2, 0.3, 9))
    ids = np.concatenate([np.arange(n) % 2, np.full(larger, 2)]).astype(np.int32)
    want = orc.jaccard_candidates(ds, qs, np.array([0, 3]), np.arange(3, dtype=np.int32))[ids]
    got = _refine(pm, pm.to_device(ds), pm.to_device(qs), np.array([0, ids.size]), ids)
    assert np.all(np.abs(got - want) <= 1e-9 * want + 1e-12)

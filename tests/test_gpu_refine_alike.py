"""A pair's J does not depend on the pairs beside it in the call, bit for bit:
the paths that share a kind of pair (a wavefront's group, a workgroup, a
wavefront of the launch for large pairs) are chosen by the call's counts."""
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

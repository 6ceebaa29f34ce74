"""Pairs of about 512 edges a side in a large call (2^18 candidates, or no
workspace), where a wavefront's group takes them all: its edge numbers, its
chunks and the padding of its last chunk at their limits together."""
import numpy as np
import pytest

from paper_2511_16576_amd import datagen as dg

pytestmark = pytest.mark.gpu


def _stars(counts, side, lo, hi, seed):
    rng = np.random.default_rng(seed)
    counts = np.asarray(counts)
    radii = rng.uniform(lo, hi, counts.size) * side
    c = side // 2 + rng.uniform(-0.2, 0.2, (counts.size, 2)) * side
    ps = dg.star_polygons(rng, counts, c.astype(np.int64), radii)
    return [ps.xy[ps.offsets[i]:ps.offsets[i + 1]] for i in range(ps.n)]


@pytest.mark.parametrize("side", [1 << 16, 1 << 25])
@pytest.mark.parametrize("m", [257, 504, 505, 511, 512])
def test_groups_of_a_large_call(orc, m, side):
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    sizes = [497, 503, 504, 505, 506, 507, 508, 509, 510, 511, 512, 512, 512, 256, 257]
    data = _stars(sizes, side, 0.2, 0.3, 3) + _stars([3, 8, 9, 64, 100, 512], side, 0.01, 0.03, 4)
    queries = _stars([m, m], side, 0.2, 0.3, 9)
    data += [queries[0], queries[1][::-1], np.roll(queries[0], 17, axis=0)]       # every edge a contact
    ds, qs = dg.from_list(data), dg.from_list(queries)
    n = ds.n
    want = orc.jaccard_candidates(ds, qs, np.array([0, n, 2 * n]), np.tile(np.arange(n, dtype=np.int32), 2)).reshape(2, n)
    D, Q = pm.to_device(ds), pm.to_device(qs)
    rng, first = np.random.default_rng(m), None
    for reps in (1, 7):
        ids = np.concatenate([rng.permutation(np.tile(np.arange(n, dtype=np.int32), reps)) for _ in range(2)])
        off = torch.tensor([0, n * reps, 2 * n * reps], dtype=torch.int64).cuda()
        gid = torch.from_numpy(ids).cuda()
        q = np.repeat([0, 1], n * reps)
        for kw in (dict(split_heavy=False), dict(n_cand=1 << 18), dict()):
            got = pm.refine(D, Q, off, gid, **kw)[:ids.size].cpu().numpy()
            ref = want[q, ids]
            assert np.all(np.abs(got - ref) <= 1e-9 * ref + 1e-12), (reps, kw)
            if first is None:
                first = np.zeros((2, n))
                first[q, ids] = got
            assert np.array_equal(got, first[q, ids]), (reps, kw)
    assert (want > 0).sum() >= n

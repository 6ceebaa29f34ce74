"""The walk where its polygons' edges change place (one or two a lane, in LDS
with their products taken out, in LDS as vertices, in memory, 128-bit) and
where its launch changes form: sets that need no order, that are ordered by
one workgroup and by several, and hash counts that the split of a polygon's
hashes leaves a remainder of.  Signatures are whole numbers: equal to the
oracle's."""
import dataclasses

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


def _stars(counts, side, seed=1):
    rng = np.random.default_rng(seed)
    counts = np.asarray(counts)
    radii = rng.uniform(0.1, 0.3, counts.size) * side
    c = np.ceil(radii)[:, None] + rng.random((counts.size, 2)) * (side - 1 - 2 * np.ceil(radii))[:, None]
    return dg.star_polygons(rng, counts, c.astype(np.int64), radii)


def _sign(pm, ps, box, k, cap, **cfg):
    got = pm.sign(pm.to_device(ps), box, 7, k, cap, config=pm.sign_config(**cfg) if cfg else None)
    return got.cpu().numpy().view(np.uint32)


EDGES = [3, 63, 64, 65, 127, 128, 129, 149, 150, 151, 299, 300, 301, 511, 512, 513, 1023, 1024, 1025, 3000]


@pytest.mark.parametrize("cfg", [dict(), dict(lds_edges=300), dict(lds_edges=64), dict(samples_per_lane=2),
                                 dict(persistent=0, block_threads=192)], ids=str)
@pytest.mark.parametrize("bits", [20, 27, 31])      # 27, 31: wider than the exact doubles
def test_edge_places(pm, orc, bits, cfg):
    side, ps = 1 << bits, _stars(EDGES, 1 << bits)
    for x0, y0 in ((0, 0), (-(1 << 30), 5))[:1 if bits == 31 else 2]:
        qs = dataclasses.replace(ps, xy=ps.xy + np.array([x0, y0], ps.xy.dtype))
        box = (x0, y0, x0 + side - 1, y0 + side - 1)
        want = orc.sign(qs, box, 7, 33, 3000)
        assert np.array_equal(_sign(pm, qs, box, 33, 3000, **cfg), want)


@pytest.mark.parametrize("n,k", [(1, 1), (1, 300), (5, 7), (255, 33), (257, 64), (1000, 130), (2048, 4), (8191, 3),
                                 (8192, 9), (8193, 9), (20_000, 5)])
@pytest.mark.parametrize("persistent", [0, 1])
def test_launch_forms(pm, orc, n, k, persistent):
    rng = np.random.default_rng(n)
    ps, box = _stars(rng.integers(3, 90, n), 1 << 16, seed=n), (0, 0, (1 << 16) - 1, (1 << 16) - 1)
    want = orc.sign(ps, box, 7, k, 500)
    assert np.array_equal(_sign(pm, ps, box, k, 500, persistent=persistent), want)

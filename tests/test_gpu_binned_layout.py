"""Binned signing where its bins and launches change form: every grid side in
boxes whose rows are evenly filled, half filled or narrower than the grid,
hash counts about the groups of 256 and the chunk sizes that follow from
them, bins reused by a second call, and launches large enough to be ordered
along the plane.  The signatures equal the walk's, which other tests compare
with the oracle, and the oracle's directly on a part."""
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


def _set(n, side, seed=1, counts=(8, 33)):
    rng = np.random.default_rng(seed)
    radii = rng.uniform(0.02, 0.1, n) * side
    c = np.ceil(radii)[:, None] + rng.random((n, 2)) * (side - 1 - 2 * np.ceil(radii))[:, None]
    return dg.star_polygons(rng, rng.integers(*counts, n), c.astype(np.int64), radii)


@pytest.mark.parametrize("box", [(0, 0, (1 << 20) - 1, (1 << 20) - 1), (0, 0, 1 << 20, 1 << 20),
                                 (-5, 3, 999_990, 700_000), (100, 100, 139, 163), (0, 0, 127, (1 << 20) - 1)])
@pytest.mark.parametrize("bits", [0, 1, 4, 5, 6])
def test_boxes_and_grids(pm, orc, box, bits):
    ps = _set(60, 1 << 20)
    if box[2] < 200:        # polygons of a few lattice points
        ps = dg.from_list([dg.rectangle(100 + i, 100 + 2 * i, 103 + i, 105 + 3 * i) for i in range(20)])
    D = pm.to_device(ps)
    k, cap = 40, 1 << 16
    want = orc.sign(ps, box, 0, k, cap)
    for horizon in (256, 5000, 30_000):
        got = pm.sign_binned(D, box, 0, k, cap, horizon=horizon, bin_bits=bits, walk_ratio=0.0)
        assert np.array_equal(got.cpu().numpy().view(np.uint32), want), horizon


@pytest.mark.parametrize("k", [1, 2, 3, 63, 127, 128, 129, 255, 256, 257, 520])
@pytest.mark.parametrize("bits", [3, 6])
def test_hash_groups(pm, k, bits):
    import torch
    ps, box = _set(150, 1 << 22), (0, 0, (1 << 22) - 1, (1 << 22) - 1)
    D = pm.to_device(ps)
    walk = pm.sign(D, box, 3, k, 1 << 20)
    ws = torch.full((pm.sign_binned_workspace_size(ps.n, k, 1 << 20, 20_000, bits),), 0xC3, dtype=torch.uint8,
                    device="cuda")
    for rebin in (True, False):        # the second call reads the first one's bins
        got = pm.sign_binned(D, box, 3, k, 1 << 20, horizon=20_000, bin_bits=bits, walk_ratio=0.0, ws=ws, rebin=rebin)
        assert torch.equal(got, walk), rebin


@pytest.mark.parametrize("n, box", [(65_536, (0, 0, (1 << 20) - 1, (1 << 20) - 1)),
                                    (65_537, (0, 0, (1 << 20) - 1, (1 << 20) - 1)),
                                    (70_003, (-77, 12, 1_000_000, 650_000))])
def test_large_launches(pm, n, box):
    import torch
    small = _set(2000, 1 << 20, seed=2, counts=(3, 12))
    ids = np.random.default_rng(4).integers(0, small.n, n)
    D = pm.to_device(small.subset(ids))
    k, cap = 70, 1 << 16
    walk = pm.sign(pm.to_device(small), box, 0, k, cap)[torch.from_numpy(ids).cuda()]
    for ratio in (0.0, 600.0):
        got = pm.sign_binned(D, box, 0, k, cap, horizon=4000, bin_bits=6, walk_ratio=ratio)
        assert torch.equal(got, walk), ratio


@pytest.mark.parametrize("k", [1, 4, 64, 65])
@pytest.mark.parametrize("frac", [0.02, 0.25, 1.0])
def test_first_samples_alone(pm, k, frac):
    """Polygons whose first hits are expected in the first samples of a chunk,
    among them slivers that fill little of their MBR."""
    import torch
    side = 1 << 22
    rng = np.random.default_rng([k, int(100 * frac)])
    star = [dg.star_polygons(rng, [n], [[side // 2, side // 2]], [frac * side / 2]).xy for n in (3, 40, 300, 1500)]
    sliver = [np.array([[0, 0], [side - 1, int(side * frac)], [side - 1, int(side * frac) + w]]) for w in (9, 900, 90_000)]
    D = pm.to_device(dg.from_list(star + sliver))
    box = (0, 0, side - 1, side - 1)
    walk = pm.sign(D, box, 3, k, 1 << 18)
    for bits in (3, 5, 6):
        got = pm.sign_binned(D, box, 3, k, 1 << 18, horizon=1 << 18, bin_bits=bits, walk_ratio=0.0)
        assert torch.equal(got, walk), bits

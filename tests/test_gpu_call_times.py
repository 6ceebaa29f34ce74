"""Calls whose path a rule on sizes chooses, against the same work on the other
path: the rule may not cost a multiple (least of several runs each, and room
for noise)."""
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


def _us(f, reps=7):
    import torch
    f()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


def _rings(n, verts, side, lo, hi, seed):
    """n rings of `verts` vertices near circles."""
    rng = np.random.default_rng(seed)
    r = rng.uniform(lo, hi, n) * side
    c = rng.uniform(hi, 1 - hi, (n, 2)) * side
    t = np.arange(verts) * (2 * np.pi / verts)
    rad = r[:, None] * rng.uniform(0.9, 1.0, (n, verts))
    xy = np.stack([c[:, :1] + rad * np.cos(t), c[:, 1:] + rad * np.sin(t)], 2)
    return [np.rint(p).astype(np.int64) for p in xy]


def test_refinement_of_many_pairs_of_500_edges(pm):
    """30,000 of them: by the rule for small calls, and as part of a call with
    room for 2^18."""
    import torch
    side, nq, per = 1 << 24, 300, 100
    D = pm.to_device(dg.from_list(_rings(300, 500, side, 0.1, 0.2, 1)))
    Q = pm.to_device(dg.from_list(_rings(nq, 500, side, 0.1, 0.2, 2)))
    ids = torch.randint(0, 300, (nq * per,), generator=torch.Generator().manual_seed(3), dtype=torch.int32).cuda()
    off = torch.arange(nq + 1, dtype=torch.int64).cuda() * per
    ws = pm.refine_workspace()
    small = _us(lambda: pm.refine(D, Q, off, ids, ws=ws, n_cand=nq * per))
    large = _us(lambda: pm.refine(D, Q, off, ids, ws=ws, n_cand=1 << 18))
    assert small <= 1.6 * large, (small, large)
    a, b = (pm.refine(D, Q, off, ids, ws=ws, n_cand=n)[:nq * per] for n in (nq * per, 1 << 18))
    assert torch.equal(a, b)


def test_lookup_of_long_lists(pm):
    """3,000 queries of some 4,800 entries each over 300,000 polygons, more than
    run at once with their bitmaps on chip, against six calls of 500."""
    import torch
    n, b, nq = 300_000, 16, 3000
    g = torch.Generator(device="cuda").manual_seed(4)
    z = torch.randint(0, n // 300, (n, b), generator=g, device="cuda") * b + torch.arange(b, device="cuda")
    z = (z ^ (z >> 30)) * -4658895280553007687
    z = (z ^ (z >> 27)) * -7723592293110705685
    z = z ^ (z >> 31)
    sk, se = pm.index_build(z.contiguous())
    qk = z[torch.randint(0, n, (nq,), generator=g, device="cuda")].contiguous()

    def call(q):
        off = torch.empty(q + 1, dtype=torch.int64, device="cuda")
        ids = torch.empty(q * 6000, dtype=torch.int32, device="cuda")
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.empty(int(pm.lib().polymh_query_workspace_size(n, q)), dtype=torch.uint8, device="cuda")
        return _us(lambda: pm.query_capped(sk, se, n, qk[:q], off, ids, flag, ws))
    whole, part = call(nq), call(500)
    assert whole <= 1.5 * 6 * part, (whole, part)


def test_top_entry_of_equal_values(pm):
    """The best of 5,000 lists of 3,000 that hold eight different J, against the
    best ten: one pass over the lists, against the digits' counts."""
    import torch
    nq, n = 5000, 3000
    g = torch.Generator(device="cuda").manual_seed(5)
    js = torch.randint(0, 8, (nq * n,), generator=g, device="cuda").double() / 8
    ids = torch.arange(n, dtype=torch.int32, device="cuda").repeat(nq)
    off = torch.arange(nq + 1, dtype=torch.int64, device="cuda") * n
    one, ten = _us(lambda: pm.topk(off, ids, js, 1)), _us(lambda: pm.topk(off, ids, js, 10))
    assert one <= 0.5 * ten, (one, ten)


def test_topk_of_zeros(pm):
    """Lists whose J are all zero, against lists of random J."""
    import torch
    nq, n = 5000, 500
    ids = torch.arange(n, dtype=torch.int32, device="cuda").repeat(nq)
    off = torch.arange(nq + 1, dtype=torch.int64, device="cuda") * n
    js = torch.rand(nq * n, generator=torch.Generator(device="cuda").manual_seed(6), dtype=torch.float64, device="cuda")
    zero = _us(lambda: pm.topk(off, ids, js * 0, 100)) - _us(lambda: js * 0)
    rand = _us(lambda: pm.topk(off, ids, js + 0, 100)) - _us(lambda: js + 0)
    assert zero <= 1.7 * rand, (zero, rand)


@pytest.mark.parametrize("values", [1, 8])
def test_topk_of_few_values(pm, values):
    """The best ten of 5,000 lists of 3,000 whose J take few values, against
    lists of random J."""
    import torch
    nq, n = 5000, 3000
    g = torch.Generator(device="cuda").manual_seed(12)
    ids = torch.arange(n, dtype=torch.int32, device="cuda").repeat(nq)
    off = torch.arange(nq + 1, dtype=torch.int64, device="cuda") * n
    few = torch.randint(0, values, (nq * n,), generator=g, device="cuda").double() / values
    rand = torch.rand(nq * n, generator=g, dtype=torch.float64, device="cuda")
    a, b = (_us(lambda: pm.topk(off, ids, js, 10)) for js in (few, rand))
    assert a <= 2.1 * b, (a, b)


def test_join_of_a_large_ring(pm):
    """One ring of 300,000 vertices: copying it takes no longer than staging it,
    which reads as much and computes besides."""
    xy = _rings(1, 300_000, 1 << 24, 0.1, 0.2, 7)[0]
    R, D = pm.rings_to_device(dg.from_rings([[xy]])), pm.to_device(dg.from_list([xy]))
    join, prepare = _us(lambda: pm.join_rings(R)), _us(lambda: pm.prepare(D))
    assert join <= prepare, (join, prepare)


def test_prepare_of_a_few_large_rings(pm):
    """Four rings of 300,000 vertices against one."""
    rings = _rings(4, 300_000, 1 << 24, 0.1, 0.2, 8)
    four, one = (_us(lambda: pm.prepare(D)) for D in (pm.to_device(dg.from_list(r)) for r in (rings, rings[:1])))
    assert four <= 2 * one, (four, one)


def test_binning_of_samples(pm):
    """Drawing 456,704 samples a hash, 256 hashes, and grouping them by cell,
    against twelve bytes a sample written once."""
    import torch
    side, k, h = 1 << 24, 256, 456_704
    rng = np.random.default_rng(9)
    D = pm.to_device(dg.star_polygons(rng, [20] * 16, rng.integers(1 << 22, 3 << 22, (16, 2)), [2e6] * 16))
    box = (0, 0, side - 1, side - 1)
    ws = torch.empty(pm.sign_binned_workspace_size(16, k, 1 << 26, h, 6), dtype=torch.uint8, device="cuda")
    first, again = (_us(lambda: pm.sign_binned(D, box, 0, k, 1 << 26, horizon=h, bin_bits=6, walk_ratio=0.0, ws=ws,
                                               rebin=r)) for r in (True, False))
    fill = _us(lambda: ws[:12 * k * h].fill_(1))
    assert first - again <= 5.5 * fill, (first, again, fill)


def test_lookup_of_few_hashes(pm):
    """100 large polygons' lookups of 16 hashes against 256, which read many
    samples at a time and so have fewer tested past their first hits."""
    import torch
    rng = np.random.default_rng(10)
    box = (0, 0, (1 << 24) - 1, (1 << 24) - 1)
    D = pm.to_device(dg.star_polygons(rng, rng.integers(40, 110, 100), rng.integers(3 << 20, 13 << 20, (100, 2)),
                                      rng.uniform(0.02, 0.15, 100) * (1 << 24)))

    def call(k):
        h, b = pm.binned_params(D, box, k, 1 << 22, 0.0)
        ws = torch.empty(pm.sign_binned_workspace_size(100, k, 1 << 22, h, b), dtype=torch.uint8, device="cuda")
        sign = lambda r: pm.sign_binned(D, box, 0, k, 1 << 22, horizon=h, bin_bits=b, walk_ratio=0.0, ws=ws, rebin=r)
        sign(True)
        return _us(lambda: sign(False))
    few, many = call(16), call(256)
    assert few <= 0.95 * many, (few, many)


def test_signing_by_even_items(pm):
    """3,000 polygons of 128 hashes in workgroups of 512: the library's choice of
    hashes a work item against halves."""
    rng = np.random.default_rng(11)
    box = (0, 0, (1 << 24) - 1, (1 << 24) - 1)
    D = pm.to_device(dg.star_polygons(rng, rng.integers(40, 110, 3000), rng.integers(3 << 20, 13 << 20, (3000, 2)),
                                      rng.uniform(0.02, 0.15, 3000) * (1 << 24)))
    auto, even = (_us(lambda: pm.sign(D, box, 0, 128, 1 << 22, config=pm.sign_config(block_threads=512, hash_block=h)))
                  for h in (0, 64))
    assert auto <= 1.2 * even, (auto, even)

"""The lookup against the brute-force candidates where it changes from the
bitmap on chip to gathered lists: row lengths about the short-row limit and
the on-chip limit, few and many queries, several chunks of bands, and keys
that recur in other bands or in most polygons."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_16576_amd import polymh
    polymh.check_device()
    return polymh


@pytest.mark.parametrize("nd, nq, b, vals", [
    (32 * 5120, 40, 8, 4000), (32 * 5120 + 1, 40, 8, 4000), (32 * 5120 + 1, 2100, 4, 4000),
    (32 * 32768, 12, 5, 20000), (32 * 32768 + 1, 12, 5, 20000), (3000, 30, 300, 700), (70, 9, 257, 3),
    (20000, 60, 64, 2)])
def test_lookup_at_its_limits(pm, orc, nd, nq, b, vals):
    import torch
    rng = np.random.default_rng([nd, nq, b])
    dk = rng.integers(0, vals, (nd, b)).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    dk[rng.choice(nd, nd // 3, replace=False), 0] = 7          # a bucket of a third of the polygons
    qk = dk[rng.integers(0, nd, nq)].copy()
    qk[0, :] = 5                                               # no candidate
    if b > 1:
        qk[1] = np.roll(qk[1], 1)                              # its keys are others' in other bands
    t = lambda a: torch.from_numpy(a.view(np.int64)).cuda()
    sk, si = pm.index_build(t(dk))
    pick = np.sort(rng.choice(nq, min(nq, 24), replace=False))
    pick[:2] = [0, 1]
    ooff, oids = orc.candidates(dk, qk[pick])
    off, ids = pm.query(sk, si, nd, t(qk))
    o, i = off.cpu().numpy(), ids.cpu().numpy()
    for n, q in enumerate(pick):
        assert np.array_equal(i[o[q]:o[q + 1]], oids[ooff[n]:ooff[n + 1]]), q
    ws = torch.full((int(pm.lib().polymh_query_workspace_size(nd, nq)),), 0x5A, dtype=torch.uint8, device="cuda")
    coff = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    flag = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    cids = torch.full((max(ids.numel(), 1),), -7, dtype=torch.int32, device="cuda")
    pm.query_capped(sk, si, nd, t(qk), coff, cids, flag, ws)
    assert int(flag.item()) == 0 and torch.equal(coff, off) and torch.equal(cids[:ids.numel()], ids)
    short = cids[:ids.numel() - 1].fill_(-7)
    pm.query_capped(sk, si, nd, t(qk), coff, short, flag, ws)
    assert int(flag.item()) == 1 and not coff.any() and bool((short == -7).all())


@pytest.mark.parametrize("nq", [1, 7, 256, 257])
@pytest.mark.parametrize("nd, b", [(1, 1), (2, 3), (5, 3), (17, 1), (33, 2), (4000, 16), (4000, 65)])
def test_searches(pm, orc, nd, b, nq):
    """Searches by one thread a band and by 16 (up to 256 queries on 256 CUs):
    tables shorter and longer than a round's 16 keys, uniform keys, crowded
    ones at either end of the range, keys below and above all others."""
    rng = np.random.default_rng([nd, b, nq])
    top = np.uint64(2 ** 64 - 1)
    for spread in ("uniform", "low", "high", "few"):
        dk = rng.integers(0, 2 ** 64 - 1, (nd, b), dtype=np.uint64, endpoint=True)
        if spread == "low":
            dk >>= np.uint64(40)
        elif spread == "high":
            dk |= top << np.uint64(30)
        elif spread == "few":
            dk = dk % np.uint64(3) * (top // np.uint64(2))
        qk = dk[rng.integers(0, nd, nq)].copy()
        qk[rng.random(qk.shape) < 0.2] = 0
        qk[rng.random(qk.shape) < 0.2] = top
        qk[rng.random(qk.shape) < 0.2] += np.uint64(1)
        t = lambda a: torch.from_numpy(a.view(np.int64)).cuda()
        import torch
        sk, si = pm.index_build(t(dk))
        off, ids = pm.query(sk, si, nd, t(qk))
        ooff, oids = orc.candidates(dk, qk)
        assert np.array_equal(off.cpu().numpy(), ooff) and np.array_equal(ids.cpu().numpy(), oids), spread

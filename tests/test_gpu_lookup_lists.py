"""Lists about the caps that send a query from one pass to another, in data sets
whose bitmap rows are built on chip at once, in turn, and in memory."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# entries of the buckets of band 0; of band 1 each holds a third of them again
SIZES = [1, 63, 64, 65, 2048, 4095, 4096, 4097, 6000, 16383, 16384, 16385, 20000]


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_16576_amd import polymh
    polymh.check_device()
    return polymh


def _keys(x):
    """Spread keys, so that numbers are apart as band keys are."""
    x = np.asarray(x, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    x ^= x >> np.uint64(29)
    return (x * np.uint64(0xBF58476D1CE4E5B9)).view(np.int64)


@pytest.mark.parametrize("nq", [3, 300, 2100])
@pytest.mark.parametrize("n", [163_840, 163_841, 400_000, 1_048_576, 1_048_577])
def test_lists_at_the_caps(pm, n, nq):
    import torch
    rng = np.random.default_rng(n + nq)
    perm = rng.permutation(n)
    band = np.stack([np.arange(n) + 1000, np.arange(n) + 1000 + n], 1)      # alone in their buckets
    members, at = [], 0
    for i, c in enumerate(SIZES):
        ids = np.sort(perm[at:at + c])
        at += c
        band[ids, 0] = i
        other = ids[::3]                                  # in band 1 too, with as many others
        extra = perm[at:at + other.size]
        at += other.size
        band[other, 1] = 100 + i
        band[extra, 1] = 100 + i
        members.append((ids, np.unique(np.concatenate([other, extra]))))
    keys = torch.from_numpy(_keys(band)).cuda()
    sk, se = pm.index_build(keys)
    pick = rng.integers(0, len(SIZES), (nq, 2))
    pick[:min(nq, len(SIZES))] = np.arange(min(nq, len(SIZES)))[:, None]
    pick[::7, 1] = -1                                     # no bucket in band 1
    qk = torch.from_numpy(_keys(np.stack([pick[:, 0], np.where(pick[:, 1] < 0, 99, 100 + pick[:, 1])], 1))).cuda()
    off, ids = pm.query(sk, se, n, qk)
    off, ids = off.cpu().numpy(), ids.cpu().numpy()
    cache = {}
    for q, (i, j) in enumerate(pick):
        if (i, j) not in cache:
            cache[i, j] = np.union1d(members[i][0], members[j][1]) if j >= 0 else members[i][0]
        assert np.array_equal(ids[off[q]:off[q + 1]], cache[i, j]), (q, i, j)
    # the same lists in one call with a capacity
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    o2, i2 = torch.empty(nq + 1, dtype=torch.int64, device="cuda"), torch.empty(int(off[-1]), dtype=torch.int32, device="cuda")
    ws = torch.empty(int(pm.lib().polymh_query_workspace_size(n, nq)), dtype=torch.uint8, device="cuda")
    pm.query_capped(sk, se, n, qk, o2, i2, flag, ws)
    assert int(flag.item()) == 0
    assert np.array_equal(o2.cpu().numpy(), off) and np.array_equal(i2.cpu().numpy(), ids)

"""The top-k selection where it changes from one pass an entry to counting
digits (4 and 5 entries), and where counting skips the bits in which no entry
differs, against the oracle."""
import numpy as np
import pytest

from oracle import core

pytestmark = pytest.mark.gpu

LENS = [0, 2, 3, 4, 5, 63, 256, 257, 511, 512, 513, 1025, 3000]


@pytest.mark.parametrize("many", [False, True])         # 1,024 and 256 threads a list
@pytest.mark.parametrize("values", [0, 1, 3, 1 << 40])  # how many a J may take: all zero, ..., nearly all different
@pytest.mark.parametrize("k", [2, 3, 4, 5])
def test_topk_of_a_few(k, values, many):
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    rng = np.random.default_rng([k, values, many])
    lens = LENS + ([7] * 1100 if many else [])
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ids = np.concatenate([np.sort(rng.choice(4 * n + 4, n, replace=False)) for n in lens]).astype(np.int32)
    js = rng.integers(0, values + 1, ids.size) / max(values, 1)
    top, val = (t.cpu().numpy() for t in pm.topk(*(torch.from_numpy(a).cuda() for a in (off, ids, js)), k))
    want, wval = core.topk(off, ids, js, k)
    assert np.array_equal(top, want) and np.array_equal(val, wval)


@pytest.mark.parametrize("ids_from", ["0", "spread", "top"])
@pytest.mark.parametrize("k", [5, 63, 64, 65, 200])
def test_lists_of_few_values(k, ids_from):
    """Lists with one J, two that differ in one bit, or some whose bits end
    early or late; their ids consecutive, spread over 31 bits or at their top."""
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    rng = np.random.default_rng([k, len(ids_from)])
    one = np.float64(0.7)
    kinds = [[0.0], [one], [1.0], [one, np.nextafter(one, 1)], [0.0, 5e-324], [0.5, 0.5 + 2.0 ** -30], [0.0, one, 1.0],
             [-1.5, -1.5 - 2.0 ** -40], list(0.5 + np.arange(7) * 2.0 ** -45), list(0.5 + np.arange(300) / 1024)]
    lists = []
    for values in kinds:
        for n in (127, 128, 129, 200, 257, 401, 3000):
            ids = {"0": np.arange(n), "spread": np.sort(rng.choice(2 ** 31 - 1, n, replace=False)),
                   "top": 2 ** 31 - n + np.arange(n)}[ids_from]
            lists.append((ids, rng.choice(values, n)))
    off = np.concatenate([[0], np.cumsum([len(i) for i, _ in lists])]).astype(np.int64)
    ids = np.concatenate([i for i, _ in lists]).astype(np.int32)
    js = np.concatenate([j for _, j in lists])
    top, val = (t.cpu().numpy() for t in pm.topk(*(torch.from_numpy(a).cuda() for a in (off, ids, js)), k))
    want, wval = core.topk(off, ids, js, k)
    assert np.array_equal(top, want) and np.array_equal(val, wval)

"""The top-k selection where it changes from one pass an entry to counting
digits (3 to 5 entries; 512 entries a list at 4), against the oracle."""
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

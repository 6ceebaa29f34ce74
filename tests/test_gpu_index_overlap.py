"""The bucket table where the keys share memory with either output: the passes
read the keys before they write there."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [4, 12, 20, 28, 64])       # of a key that vary: one pass to eight
@pytest.mark.parametrize("at", [-70_000, 0, 140_000, 279_996])  # where the entries start, in bytes from the keys
def test_entries_in_the_keys_memory(at, bits):
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    m = 70_001
    keys = np.random.default_rng(bits).integers(0, 2 ** bits, m, dtype=np.uint64)
    order = np.argsort(keys, kind="stable")
    buf = torch.zeros(4 * m + 8 * m + 4 * m + 1024, dtype=torch.uint8, device="cuda")
    k0 = 4 * m + 252 & ~255
    kv = buf[k0:k0 + 8 * m].view(torch.int64)
    kv.copy_(torch.from_numpy(keys.view(np.int64)))
    si = buf[k0 + at:k0 + at + 4 * m].view(torch.int32)
    sk = torch.empty(m, dtype=torch.int64, device="cuda")
    ws = torch.empty(int(pm.lib().polymh_index_workspace_size(m, 1)), dtype=torch.uint8, device="cuda")
    pm._check(pm.lib().polymh_index_build(pm._ptr(kv), m, 1, pm._ptr(ws), ws.numel(), pm._ptr(sk), pm._ptr(si),
                                          pm._stream(None)))
    assert np.array_equal(sk.cpu().numpy().view(np.uint64), keys[order])
    assert np.array_equal(si.cpu().numpy(), order.astype(np.int32))

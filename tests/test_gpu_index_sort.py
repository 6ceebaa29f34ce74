"""The bucket table's sort against numpy's stable argsort, at the sizes and
key sets where its parts take over from each other: tile edges, the two tile
sizes, digits with one value, keys that need all eight digits, runs of equal
prefixes of every length class whose keys are out of order, and keys that
share memory with the output."""
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


def _spread(rng, m):
    return rng.integers(0, 2**64, m, dtype=np.uint64)


def _keys(kind, m, rng):
    if kind == "spread":
        return _spread(rng, m)
    if kind == "few":                       # three keys, one of them most entries
        return _spread(rng, 3)[rng.choice(3, m, p=[0.9, 0.07, 0.03])]
    if kind == "one":
        return np.full(m, 0x123456789ABCDEF0, dtype=np.uint64)
    if kind == "small":                     # only the low digits vary
        return rng.integers(0, 1 << 20, m, dtype=np.uint64)
    # few prefixes of equal upper halves, lower halves spread: runs of every
    # length class out of order (about 3, 30, 300 entries, and thousands)
    per = {"runs3": 3, "runs30": 30, "runs300": 300, "runs9000": 9000}[kind]
    top = _spread(rng, max(m // per, 1)) & np.uint64(0xFFFFFFFF00000000)
    return top[rng.integers(0, top.size, m)] | rng.integers(0, 1 << 12, m, dtype=np.uint64)


@pytest.mark.parametrize("kind", ["spread", "few", "one", "small", "runs3", "runs30", "runs300", "runs9000"])
@pytest.mark.parametrize("m", [1, 2, 63, 4095, 4096, 4097, 70_001, (3 << 19) - 1, (3 << 19) + 8193])
def test_sort_equals_stable_argsort(pm, kind, m):
    import torch
    keys = _keys(kind, m, np.random.default_rng([m, len(kind)]))
    order = np.argsort(keys, kind="stable")
    k = torch.from_numpy(keys.view(np.int64)).cuda().reshape(m, 1)
    ws = torch.full((int(pm.lib().polymh_index_workspace_size(m, 1)),), 0xA5, dtype=torch.uint8, device="cuda")
    for _ in range(2):                      # the second on the first one's scratch
        sk, si = pm.index_build(k, ws=ws)
        assert np.array_equal(sk.cpu().numpy().view(np.uint64), keys[order])
        assert np.array_equal(si.cpu().numpy(), order.astype(np.int32))


@pytest.mark.parametrize("kind", ["spread", "small", "one"])
def test_sort_of_keys_in_the_output_array(pm, kind):
    import torch
    m = 70_001
    keys = _keys(kind, m, np.random.default_rng(5))
    order = np.argsort(keys, kind="stable")
    buf = torch.from_numpy(keys.view(np.int64)).cuda()
    ids = torch.empty(m, dtype=torch.int32, device="cuda")
    ws = torch.empty(int(pm.lib().polymh_index_workspace_size(m, 1)), dtype=torch.uint8, device="cuda")
    pm._check(pm.lib().polymh_index_build(buf.data_ptr(), m, 1, ws.data_ptr(), ws.numel(), buf.data_ptr(),
                                          ids.data_ptr(), pm._stream()))
    assert np.array_equal(buf.cpu().numpy().view(np.uint64), keys[order])
    assert np.array_equal(ids.cpu().numpy(), order.astype(np.int32))

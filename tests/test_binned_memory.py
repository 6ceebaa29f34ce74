"""Memory of the binned samples: what one hash more than a group costs, and the
horizon that a given memory allows (host code, no GPU needed)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_16576_amd", "libpolymh.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libpolymh.so not built")


@pytest.mark.parametrize("bits", [0, 4, 5, 6])
@pytest.mark.parametrize("k", [257, 513, 1025])
def test_one_hash_more_than_groups(k, bits):
    from paper_2511_16576_amd import polymh as pm
    size, full = (pm.sign_binned_workspace_size(1, j, 1 << 26, 1 << 18, bits) for j in (k, k - 1))
    # at most what rounding each group up to 32 hashes and its tables add
    groups = -(-k // 256)
    assert size <= full * (k + 32 * groups) / (k - 1) * 1.06


@pytest.mark.parametrize("k", [1, 4, 64, 128, 256, 257, 512])
@pytest.mark.parametrize("max_bytes", [1 << 20, 1 << 28, 1 << 31])
def test_horizon_within_memory(k, max_bytes):
    from paper_2511_16576_amd import polymh as pm
    cap, size = 1 << 26, lambda h, b: pm.sign_binned_workspace_size(1, k, 1 << 26, h, b)
    for bits in (0, 3, 6):
        h = pm._binned_horizon(k, cap, bits, cap, max_bytes)
        assert h % 256 == 0 and (h == 256 or size(h, bits) <= max_bytes + (1 << 16))
        # no more than a tenth, or a chunk of each hash, is given away
        if h < cap and h > 256:
            assert size(h + h // 10 + (1 << 15), bits) > max_bytes
        # room for all: the horizon as it was asked for, a step of 256 above
        assert pm._binned_horizon(k, 1000, bits, 1000, max_bytes) in (1000, 256, 512, 768)
        if size(1000, bits) <= max_bytes:
            assert pm._binned_horizon(k, 1000, bits, 1000, max_bytes) == 1000
            assert pm._binned_horizon(k, cap, bits, 700, max_bytes) == 768

"""Memory of the binned samples: what one hash more than a group costs (host
code, no GPU needed)."""
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

"""The weight gradients' split over the rows where its rule changes, against the
oracle, and the memory that its partial sums need."""
import os

import numpy as np
import pytest

from oracle import mlp as om

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_16576_amd", "libpolymh.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="libpolymh.so not built")
def test_partial_sums_of_256_rows():
    """16,384 rows in 64 partial sums of both weight gradients; fewer rows need
    no more memory than the most, whatever their split."""
    from paper_2511_16576_amd import polymh as pm
    partials = (om.OFF_B1 - om.OFF_W1 + om.OFF_B2 - om.OFF_W2) * 4
    size = [int(pm.lib().polymh_mlp_scratch_size(B)) for B in range(0, 40_000, 32)]
    assert size == sorted(size)
    assert size[16_384 // 32] >= 64 * partials + 2 * 16_384 * 256 * 2
    assert size[8192 // 32] < 33 * partials + 2 * 8192 * 256 * 2 + (3 << 20)


def _bits(x):
    return (om.bf16_round(np.asarray(x, np.float32)).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)


@pytest.mark.gpu
@pytest.mark.parametrize("B", [4096, 4128, 16_352, 16_384, 16_416, 20_000])
def test_gradients(B):
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    rng = np.random.default_rng(B)
    p = rng.normal(0, 0.05, om.N_PARAMS).astype(np.float32)
    p[om.OFF_W1:om.OFF_B1] = om.bf16_round(p[om.OFF_W1:om.OFF_B1])
    p[om.OFF_W2:om.OFF_B2] = om.bf16_round(p[om.OFF_W2:om.OFF_B2])
    X = om.bf16_round(rng.normal(0, 1, (B, om.N_IN)).astype(np.float32))
    lab = rng.random(B).astype(np.float32)
    params, Xg, labg = torch.from_numpy(p).cuda(), torch.from_numpy(_bits(X)).cuda(), torch.from_numpy(lab).cuda()
    wbf16 = torch.empty(pm.mlp_bf16_count(), dtype=torch.int16, device="cuda")
    pm.mlp_sync_bf16(params, wbf16)
    acts, scratch = pm.mlp_buffers(B)
    pm.mlp_forward(Xg, params, wbf16, acts)
    grad, loss = torch.empty_like(params), torch.zeros(1, dtype=torch.float32, device="cuda")
    pm.mlp_backward(Xg, params, wbf16, acts, labg, grad, loss, scratch)
    want, S = om.backward_mixed(X.astype(np.float64), p.astype(np.float64), lab.astype(np.float64), terms=True)
    assert np.all(np.abs(grad.cpu().numpy().astype(np.float64) - want) <= 2 ** -7 * S + 1e-9)

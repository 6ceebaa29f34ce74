"""The scorer's forward and backward passes where their 32-row tiles and the
splits of the weight gradients change: one tile, fewer tiles than CUs, one
more than a round of the CUs, and rows that the splits leave a remainder of.
Against the oracle's mixed-precision network: FP32 sums and a BF16 rounding
that falls the other way move an entry by at most a BF16 rounding (2^-7) of the
sum of the absolute values of its terms."""
import numpy as np
import pytest

from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_16576_amd import polymh
    polymh.check_device()
    return polymh


def _bits(x):
    return (om.bf16_round(np.asarray(x, np.float32)).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)


@pytest.mark.parametrize("B", [32, 64, 288, 2080, 8160, 8192, 8224])
def test_forward_and_backward(pm, B):
    import torch
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
    y = pm.mlp_forward(Xg, params, wbf16, acts).cpu().numpy()
    p64, X64 = p.astype(np.float64), X.astype(np.float64)
    a = om.forward_mixed(X64, p64)
    S3 = np.abs(a["h2"]) @ np.abs(p64[om.OFF_W3:om.OFF_B3])
    assert np.all(np.abs(y - a["y"]) <= 0.25 * 2 ** -7 * S3 + 1e-6)
    grad, loss = torch.empty_like(params), torch.zeros(1, dtype=torch.float32, device="cuda")
    pm.mlp_backward(Xg, params, wbf16, acts, labg, grad, loss, scratch)
    want, S = om.backward_mixed(X64, p64, lab.astype(np.float64), terms=True)
    err = np.abs(grad.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= 2 ** -7 * S + 1e-9)
    assert abs(float(loss.item()) - float(np.mean((a["y"] - lab) ** 2))) < 1e-5

"""Predictions of a list of pairs in one launch: fewer rows than a tile, whole
and ragged tiles, more tiles than workgroups, rows without a pair, and
signatures that are not 16-byte aligned, against the feature rows and the
forward pass.  Both round the same BF16 activations; the output layer's 256
FP32 products are added in another order, so the sums differ by at most 2 x 256
x 2^-24 of the sum of their absolute values and the predictions by a quarter."""
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


@pytest.mark.parametrize("R,aligned", [(1, True), (31, True), (33, True), (1000, True), (8192, True), (8225, True),
                                       (9000, False)])
def test_predict_pairs(pm, R, aligned):
    import torch
    from paper_2511_16576_amd import scorer
    rng = np.random.default_rng(R)
    n = 300
    buf = torch.from_numpy(rng.integers(1, 4, n * 256 + 1).astype(np.int32)).cuda()
    sig = (buf[:-1] if aligned else buf[1:]).view(n, 256)
    f = rng.uniform(-1, 1, (n, 12)).astype(np.float32)
    f[:, 6] = rng.uniform(1, 1e6, n)
    f[:, 8:10] = rng.uniform(0, 100, (n, 2))
    f[:, 10:12] = f[:, 8:10] + rng.uniform(1, 200, (n, 2))
    feats = torch.from_numpy(f).cuda()
    li = rng.integers(0, n, R).astype(np.int32)
    ri = rng.integers(0, n, R).astype(np.int32)
    li[2::11] = -1
    ri[3::13] = -1
    L, Rr = torch.from_numpy(li).cuda(), torch.from_numpy(ri).cuda()
    sc = scorer.init_scorer(3)
    y = scorer.predict_pairs(sc, sig, feats, sig, feats, L, Rr)
    assert y.shape == (R,)
    pad = (R + 31) // 32 * 32
    X = pm.pair_features(sig, feats, sig, feats, L, Rr, R_pad=pad)
    acts, _ = pm.mlp_buffers(pad)
    want = pm.mlp_forward(X, sc.params, sc.wbf16, acts)[:R]
    w3 = sc.params[om.OFF_W3:om.OFF_W3 + 256].double()
    h2 = om.forward(om.bf16_round(np.asarray((X.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32),
                                             np.float32)).astype(np.float64),
                    sc.params.cpu().numpy().astype(np.float64))["h2"]
    terms = np.abs(h2[:R] * w3.cpu().numpy()).sum(1) * (1 + 2 ** -6)
    bound = 2 * 256 * 2 ** -24 * terms / 4 + 2 ** -23
    assert (np.abs(y.cpu().numpy().astype(np.float64) - want.cpu().numpy()) <= bound).all()


def test_predict_pairs_of_nothing(pm):
    import torch
    from paper_2511_16576_amd import scorer
    sig = torch.ones((2, 256), dtype=torch.int32, device="cuda")
    feats = torch.ones((2, 12), device="cuda")
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    assert scorer.predict_pairs(scorer.init_scorer(0), sig, feats, sig, feats, none, none).shape == (0,)

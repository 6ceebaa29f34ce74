"""Staging and joining where a set's size decides how many polygons share a
wavefront (16 a CU), and a ring's size who copies it, against their
definitions."""
import numpy as np
import pytest

from paper_2511_16576_amd import datagen as dg

pytestmark = pytest.mark.gpu

# rings of a shape: both sides of 128 vertices and of 64 a ring
SHAPES = [[3], [64], [127], [128], [129], [700], [3, 3], [100, 28], [100, 30], [3] * 50, [64, 64, 65], [64, 64, 64],
          [1000, 3, 3], [511, 512, 513, 1], [3, 0, 200]]


def _sets():
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return [1, 2, 5, 16 * cus - 1, 16 * cus, 16 * cus + 1]


@pytest.mark.parametrize("which", range(6))
def test_join_of_sizes(which):
    import torch
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    n = _sets()[which]
    rng = np.random.default_rng(which)
    shapes = [SHAPES[i] for i in rng.integers(0, len(SHAPES), n)] if n > 5 else SHAPES[3 * which:3 * which + n]
    rings = [m for s in shapes for m in s]
    roff = np.concatenate([[0], np.cumsum(rings)]).astype(np.int64)
    prings = np.concatenate([[0], np.cumsum([len(s) for s in shapes])]).astype(np.int64)
    xy = rng.integers(-2**31, 2**31, (roff[-1], 2)).astype(np.int32)
    want, off = [], [0]
    for p in range(n):
        rs = [xy[roff[r]:roff[r + 1]] for r in range(prings[p], prings[p + 1])]
        v0 = rs[0][:1]
        seq = [rs[0]] + ([v0] if len(rs) > 1 else [])
        for i, r in enumerate(rs[1:]):
            seq += [r, r[:1] if len(r) else v0] + ([v0] if i + 2 < len(rs) else [])
        want.append(np.concatenate(seq))
        off.append(off[-1] + want[-1].shape[0])
    out = torch.empty((off[-1], 2), dtype=torch.int32, device="cuda")
    out_off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    t = [torch.from_numpy(a).cuda() for a in (xy, roff, prings)]
    pm._check(pm.lib().polymh_join_rings(pm._ptr(t[0]), len(xy), pm._ptr(t[1]), len(rings), pm._ptr(t[2]), n,
                                         pm._ptr(out), off[-1], pm._ptr(out_off), pm._ptr(bad), pm._stream(None)))
    torch.cuda.synchronize()
    assert np.array_equal(out_off.cpu().numpy(), off) and np.array_equal(out.cpu().numpy(), np.concatenate(want))
    assert int(bad) == int(any(m < 3 for m in rings))


@pytest.mark.parametrize("which", range(6))
def test_prepare_of_sizes(which):
    from paper_2511_16576_amd import polymh as pm
    pm.check_device()
    n = _sets()[which]
    rng = np.random.default_rng(which)
    sizes = rng.choice([3, 16, 17, 127, 128, 129, 700], n)
    polys = [rng.integers(-2**24, 2**24, (m, 2)) for m in sizes]
    mbr, area2, flags = (t.cpu().numpy() for t in pm.prepare(pm.to_device(dg.from_list(polys))))
    for p, q in enumerate(polys):
        assert mbr[p].tolist() == [*q.min(0), *q.max(0)], p
        x, y = q.T
        assert area2[p] == int((x * np.roll(y, -1) - np.roll(x, -1) * y).sum()), p
        assert flags[p] == 0, p

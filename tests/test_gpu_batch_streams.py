"""A captured batch launched on the caller's own stream: its result is the
run's, and an overflow of its candidates is reported, not the flag of a run
before it."""
import numpy as np
import pytest

from paper_2511_16576_amd import datagen as dg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_16576_amd import polymh
    polymh.check_device()
    return polymh


@pytest.mark.parametrize("own", [False, True])
def test_overflow_of_a_graph_on_another_stream(pm, own):
    import torch
    from paper_2511_16576_amd import pipeline
    w = dg.workload(1, n=400, n_queries=60)
    D = pm.to_device(w.data)
    sk, se = pm.index_build(pm.band(pm.sign(D, w.box, w.seed, w.k, w.cap), w.bands, w.rows, w.seed))
    sets = [w.queries.subset(np.arange(20 * i, 20 * i + 20)) for i in range(3)]
    total = [int(pm.query(sk, se, D.n, pm.band(pm.sign(pm.to_device(s), w.box, w.seed, w.k, w.cap), w.bands, w.rows,
                                               w.seed))[0][-1].item()) for s in sets]
    lo, hi = int(np.argmin(total)), int(np.argmax(total))
    assert total[lo] < total[hi]
    maxv = max(s.xy.shape[0] for s in sets)
    qb = pipeline.QueryBatch(D, sk, se, w.box, w.seed, w.k, w.cap, w.bands, w.rows, 20, maxv, cand_cap=total[lo])
    qb.load(sets[lo])
    graph = qb.capture()
    with torch.cuda.stream(torch.cuda.Stream() if own else torch.cuda.default_stream()):
        for i, fails in ((hi, True), (lo, False), (hi, True)):
            qb.load(sets[i])
            torch.cuda._sleep(200_000_000)      # the run starts late
            graph.launch(torch.cuda.current_stream())
            if fails:
                with pytest.raises(RuntimeError):
                    qb.result()
            else:
                ids, _ = (x.clone() for x in qb.result())
                qb.run_graph()
                assert torch.equal(ids, qb.result()[0])
            torch.cuda.synchronize()

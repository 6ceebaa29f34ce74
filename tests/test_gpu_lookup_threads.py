"""Lookups of host threads with data sets of different sizes at once: the rows
built on chip are of different sizes, and a thread's call depends on no
other's."""
import threading

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


def test_rows_of_different_sizes(pm):
    import torch
    b, nq, jobs = 4, 30, []
    g = torch.Generator(device="cuda").manual_seed(1)
    for n in (340_000, 600_000, 1_040_000, 1_048_576):
        keys = torch.randint(0, n // 3, (n, b), generator=g, device="cuda")
        keys = keys * 4 + torch.arange(b, device="cuda")
        sk, se = pm.index_build(keys)
        qk = keys[torch.randint(0, n, (nq,), generator=g, device="cuda")].contiguous()
        want = pm.query(sk, se, n, qk)
        jobs.append((n, sk, se, qk, want))
    torch.cuda.synchronize()
    errors, start = [], threading.Barrier(len(jobs))

    def work(n, sk, se, qk, want):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                off, ids = torch.empty_like(want[0]), torch.empty(want[1].numel(), dtype=torch.int32, device="cuda")
                flag = torch.zeros(1, dtype=torch.int32, device="cuda")
                ws = torch.empty(int(pm.lib().polymh_query_workspace_size(n, nq)), dtype=torch.uint8, device="cuda")
                start.wait()
                for _ in range(200):
                    pm.query_capped(sk, se, n, qk, off, ids, flag, ws, stream=stream)
                stream.synchronize()
                assert int(flag.item()) == 0 and torch.equal(off, want[0]) and torch.equal(ids, want[1]), n
        except Exception as e:      # reported by the test's own thread
            errors.append(e)
    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors

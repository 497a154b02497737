"""Results through host memory that kernels write: allocated with the handle, one per
handle, none with a caller arena."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def she():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_12157_amd import she as mod
    mod.load()
    return mod


def make(she, q=0, **kw):
    return she.Handle([she.Instance(n=(100,), r=0.1, eps=1e-2, init_sd=0.1, realisation=q),
                       she.Instance(n=(60,), bc=1, r=0.1, eps=1e-2, u_left=1.1, u_right=0.9, realisation=q)],
                      precision=1, sample_every=2, stats=she.STAT_MOMENTS | she.STAT_CORR, **kw)


def results(h):
    return [x for q in (0, 1) for x in (h.read_field(q), *(h.stats(q, corr=True, sk=True)[k]
                                                           for k in ("mean", "var", "corr", "sk")))]


def same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


def test_threads_with_their_own_handles(she):
    import torch
    want = []
    for q in range(6):
        with make(she, q) as h:
            h.run(40)
            want.append(results(h))
    got = [[] for _ in range(6)]

    def work(q):
        for _ in range(5):
            with make(she, q, stream=torch.cuda.Stream().cuda_stream) as h:
                h.run(40)
                for _ in range(10):
                    got[q].append(results(h))

    threads = [threading.Thread(target=work, args=(q,)) for q in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for q in range(6):
        assert len(got[q]) == 50
        for r in got[q]:
            same(r, want[q])


def test_results_with_an_arena(she):
    import torch
    with make(she) as h:
        h.run(30)
        want = results(h)
        insts = h.instances
    kw = dict(precision=1, sample_every=2, stats=she.STAT_MOMENTS | she.STAT_CORR)
    arena = torch.empty(she.Handle.arena_bytes(insts, **kw), dtype=torch.uint8, device="cuda")
    with make(she, arena=arena) as h:
        h.run(30)
        same(results(h), want)

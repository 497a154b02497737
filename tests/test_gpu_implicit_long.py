"""Rods above 512 cells in batches with implicit ones: the kernel with one barrier per
stage, with statistics, in every shape, beside short rods of the same batch."""
import numpy as np
import pytest

import oracle
from helpers import gpu_instance, max_rel, oracle_desc
from paper_2406_12157_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 1e-12}        # states, relative
STAT_TOL = {0: 1e-3, 1: 1e-9}    # statistics, relative


@pytest.fixture(scope="module")
def she():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_12157_amd import she as mod
    mod.load()
    return mod


def rod(n, scheme, bc, q, **kw):
    return W.instance((n,), bc=bc, scheme=scheme, r=2.0 if scheme >= W.BE else 0.1, eps=1e-3, u0=1.0,
                      u_left=1.0 + 0.1 * bc, u_right=1.0 - 0.1 * bc, init_sd=0.1, seed=6, realisation=q, **kw)


# 256 threads with one and two blocks each, 512 with one, two (and FP32) four;
# explicit, composite and short rods beside them
@pytest.mark.parametrize("precision,n,block_threads", [(0, 513, 0), (1, 513, 0), (0, 1000, 0), (1, 1000, 0), (1, 1000, 512),
                                                       (0, 1500, 256), (0, 2000, 512), (0, 2000, 0), (0, 2400, 0),
                                                       (1, 1300, 0)])
def test_statistics_against_the_oracle(she, n, block_threads, precision):
    rng = np.random.default_rng(n)
    coef = dict(cond=list(0.5 + rng.random(n)), cap=list(0.7 + 0.6 * rng.random(n)))
    insts = [rod(n, W.CN, 0, 0), rod(n, W.BE, 1, 1), rod(n, W.CN, 1, 2, **coef), rod(n, W.HEUN, 1, 3), rod(100, W.BE, 0, 4),
             rod(300, W.CN, 1, 5)]
    corr, lags = n == 513, 4 if n == 513 else 0
    mask = she.STAT_MOMENTS | (she.STAT_CORR | she.STAT_TCORR if corr else 0)
    steps = 290 if corr else 60
    with she.Handle([gpu_instance(she, i) for i in insts], precision=precision, burn_in=10, sample_every=1, stats=mask,
                    tcorr_lags=lags, block_threads=block_threads) as h:
        init = [h.read_field(q) for q in range(len(insts))]
        for k in (1, 33, steps - 34):
            h.run(k)
        fields = [h.read_field(q) for q in range(len(insts))]
        got = [h.stats(q, corr=corr, sk=corr, tcorr=corr) for q in range(len(insts))]
    for q, inst in enumerate(insts):
        d = oracle_desc(inst, precision)
        st = oracle.Stats(d, burn_in=10, every=1, corr=corr, sk=corr, tcorr_lags=lags)
        u = init[q].copy()
        oracle.advance(d, u, 0, steps, st)
        g = got[q]
        assert max_rel(fields[q], u) <= TOL[precision], q
        assert g["n_samples"] == st.n_samples == steps - 10
        assert max_rel(g["mean"], st.mean()) < STAT_TOL[precision]
        assert max_rel(g["var"], st.var()) < STAT_TOL[precision]
        assert abs(g["spatial_var"] / st.spatial()[2] - 1) < STAT_TOL[precision]
        if corr:
            assert np.max(np.abs(g["corr"] - st.cov())) < STAT_TOL[precision] * np.max(np.abs(st.cov()))
            assert max_rel(g["sk"], st.structure_factor()) < STAT_TOL[precision]
            want = st.time_corr()
            assert np.max(np.abs(g["tcorr"] - want)) < STAT_TOL[precision] * np.max(np.abs(want))


def test_freeze(she):
    """An explicit rod that diverges beside an implicit one: the state of the sample
    that is not finite, the statistics before it; the others go on."""
    bad = she.Instance(n=(600,), r=0.2, eps=100.0, init_sd=0.1, realisation=1)
    other = [she.Instance(n=(m,), bc=1, scheme=she.BE, r=2.0, eps=1e-3, u_left=1.1, u_right=0.9) for m in (600, 90)]
    kw = dict(precision=1, sample_every=5, stats=she.STAT_MOMENTS, flags=she.ALLOW_UNSTABLE)
    with she.Handle([bad] + other, **kw) as h:
        h.run(20000)
        first, frozen = h.stats(0, raise_nonfinite=False), h.read_field(0)
        assert h.stats(1)["n_samples"] == h.stats(2)["n_samples"] == 4000
    t = 5 * (first["n_samples"] + 1)
    assert first["nonfinite"] and t <= 20000 and not np.all(np.isfinite(frozen))
    with she.Handle([bad] + other, **kw) as h:
        h.run(t - 1)
        before = h.stats(0)
        h.step(1)
        np.testing.assert_array_equal(h.read_field(0), frozen)
    for key in ("n_samples", "mean", "var"):
        np.testing.assert_array_equal(first[key], before[key])

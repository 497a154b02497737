"""Explicit 1D step kernels at the edges of their work split: cells per lane,
lanes per wave, waves per instance, halo exchanges, launch chunks and samples."""
import numpy as np
import pytest

import oracle
from helpers import gpu_instance, max_rel, oracle_desc
from paper_2406_12157_amd import workloads as W

pytestmark = pytest.mark.gpu

# bars of the state parity tests: FP32 1e-5, FP64 1e-12, relative
TOL = {0: 1e-5, 1: 1e-12}


@pytest.fixture(scope="module")
def she():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_12157_amd import she as mod
    mod.load()
    return mod


def batch(n, eq=W.HEAT, noise=0):
    u0, eps, gap, sd = {W.HEAT: (1.0, 1e-2, 0.1, 0.1), W.SPECIES: (100.0, 1.0, 20.0, 10.0),
                        W.BURGERS: (0.3, 1e-4, 0.0, 4e-3)}[eq]
    return [W.instance((n,), eq=eq, bc=bc, scheme=scheme, noise=noise, r=0.1, eps=eps, u0=u0, u_left=u0 + gap * bc,
                       u_right=u0 - gap * bc, init_sd=sd, seed=9, realisation=2 * bc + scheme,
                       nu=0.3 if eq == W.BURGERS else 0.0)
            for bc in (0, 1) for scheme in (0, 1) if n > 1 or bc]


def check(she, insts, precision, steps, **kw):
    with she.Handle([gpu_instance(she, i) for i in insts], precision=precision, **kw) as h:
        init = [h.read_field(q) for q in range(len(insts))]
        h.step(steps)
        got = [h.read_field(q) for q in range(len(insts))]
    for q, inst in enumerate(insts):
        want = init[q].copy()
        oracle.advance(oracle_desc(inst, precision), want, 0, steps)
        err = max_rel(got[q], want)
        assert err <= TOL[precision], (inst["n"], inst["bc"], inst["scheme"], err)
    return got


# one wave with 1, 2, 4 cells per lane, full and not; two waves from 257 cells
# on; full waves of 62 units; 16 waves; 8 cells per lane in the middle waves
# (and FP32: 16 in all)
SIZES = [1, 2, 3, 63, 64, 65, 127, 128, 129, 253, 255, 256, 257, 495, 497, 503, 505, 992, 993, 2001, 3903, 3904, 3968,
         3969, 3975, 3976, 4005, 4096, 4223, 4473, 5400]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_rod_sizes(she, n, precision):
    insts = batch(n)
    got = check(she, insts, precision, 23)
    if n <= 512:  # every wave its own numbers: the same bits
        with she.Handle([gpu_instance(she, i) for i in insts], precision=precision, block_threads=64) as h:
            h.step(23)
            for q in range(len(insts)):
                np.testing.assert_array_equal(h.read_field(q), got[q])


@pytest.mark.parametrize("n", [7800, 8001, 8191])
def test_rod_sizes_16_cells_per_lane(she, n):
    check(she, batch(n), 0, 19)


@pytest.mark.parametrize("eq,noise", [(W.SPECIES, 0), (W.BURGERS, 0), (W.HEAT, 1), (W.HEAT, 2)])
@pytest.mark.parametrize("n", [62, 128, 251, 500, 4100])
def test_rod_face_kinds(she, n, eq, noise):
    check(she, batch(n, eq, noise), 0, 21)


@pytest.mark.parametrize("n", [61, 128, 254, 700])
def test_samples_do_not_depend_on_the_launches(she, n):
    """Samples on every third step, over calls of all lengths (chunk ends,
    X blocks completed inside a call), against one call; FP64 sums of the same
    values in the same order per cell."""
    insts = batch(n)
    kw = dict(precision=0, sample_every=3, burn_in=4, stats=she.STAT_MOMENTS | she.STAT_CORR)
    with she.Handle([gpu_instance(she, i) for i in insts], **kw) as a, \
            she.Handle([gpu_instance(she, i) for i in insts], **kw) as b:
        a.run(900)
        for k in (1, 2, 31, 32, 33, 64, 1, 300, 436):
            b.run(k)
        for q in range(len(insts)):
            np.testing.assert_array_equal(a.read_field(q), b.read_field(q))
            x, y = a.stats(q, corr=True), b.stats(q, corr=True)
            assert x["n_samples"] == y["n_samples"] == 898 // 3
            for key in ("mean", "var", "corr"):
                np.testing.assert_array_equal(x[key], y[key])


def test_moments_in_registers_and_in_memory(she):
    """A batch that fills more than one workgroup per CU keeps its per-cell sums
    in memory, a small one in registers: the same FP64 sums of the same values
    in the same order, samples up to the last step of a call."""
    insts = [W.instance((n,), bc=bc, scheme=scheme, r=0.1, eps=1e-2, u0=1.0, u_left=1.0 + 0.1 * bc,
                        u_right=1.0 - 0.1 * bc, init_sd=0.1, seed=3, realisation=q)
             for q, (n, bc, scheme) in enumerate([(3967, 1, 0), (3967, 0, 1), (257, 1, 1), (4100, 0, 0)] * 129)]
    kw = dict(precision=0, sample_every=3, burn_in=0, stats=she.STAT_MOMENTS | she.STAT_SPATIAL)
    with she.Handle([gpu_instance(she, i) for i in insts], **kw) as a, \
            she.Handle([gpu_instance(she, i) for i in insts[:4]], **kw) as b:
        for h in (a, b):
            for k in (1, 2, 27, 33):
                h.run(k)
        for q in range(4):
            np.testing.assert_array_equal(a.read_field(q), b.read_field(q))
            x, y = a.stats(q), b.stats(q)
            assert x["n_samples"] == y["n_samples"] == 21
            for key in ("mean", "var"):
                np.testing.assert_array_equal(x[key], y[key])
            # the order over cells follows the work split: 2 x 4100 x 2^-53, doubled
            assert abs(x["spatial_var"] / y["spatial_var"] - 1) <= 2e-12


# one wave per rod up to 512 cells (1, 2, 4, 8 cells per lane, full and not);
# 513: the kernel of longer implicit rods.  r = 0.01: two levels of the
# reduction matter, r = 300: all of them
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 4, 63, 64, 65, 127, 128, 130, 255, 256, 257, 500, 512, 513])
def test_implicit_rod_sizes(she, n, precision):
    insts = [W.instance((n,), bc=bc, scheme=scheme, r=r, eps=1e-3, u0=1.0, u_left=1.0 + 0.1 * bc,
                        u_right=1.0 - 0.1 * bc, init_sd=0.05, seed=4, realisation=3 * bc + scheme)
             for bc in (0, 1) for scheme, r in ((W.BE, 0.01), (W.CN, 2.0), (W.BE, 300.0)) if bc or n >= 3]
    insts.append(W.instance((min(n, 40),), bc=1, scheme=W.HEUN, r=0.05, eps=1e-3, u0=1.0, u_left=1.1, u_right=0.9,
                            init_sd=0.05, seed=4, realisation=9))
    check(she, insts, precision, 25)


def test_samples_at_the_longest_interval(she):
    """One sample every 2^31 - 1 steps: a chunk of steps has room for it (the steps
    before are skipped by a checkpoint with a later step count)."""
    every = 2 ** 31 - 1
    kw = dict(precision=1, sample_every=every, stats=she.STAT_MOMENTS)
    inst = she.Instance(n=(100,), r=0.1, eps=1e-2, init_sd=0.1, seed=3)
    with she.Handle([inst], **kw) as h:
        blob = bytearray(h.get_state())
        assert int.from_bytes(blob[16:24], "little") == 0
        blob[16:24] = (every - 20).to_bytes(8, "little")
        h.set_state(bytes(blob))
        h.step(20)
        want = h.read_field(0)
    with she.Handle([inst], **kw) as h:
        h.set_state(bytes(blob))
        h.run(50)
        st = h.stats(0)
    assert st["steps"] == every + 30 and st["n_samples"] == 1
    np.testing.assert_array_equal(st["mean"], 1.0 + (want - 1.0))

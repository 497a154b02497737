"""Finalisation kernels at the edges of their splits: the sum of a 2D/3D field
(one block, or one per span of cells) and the 1D S_k from the circulant sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def she():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_12157_amd import she as mod
    mod.load()
    return mod


# one block; its largest field; two, three and many blocks with short last
# ones; more than 1024 spans of 8192 cells (wider spans)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [(8, 3), (64, 256), (8, 2049), (64, 385), (16, 12, 101), (1024, 1000), (256, 256, 136)])
def test_field_sum_over_block_splits(she, n, precision):
    insts = [she.Instance(n=n, r=0.05, eps=1e-2, init_sd=0.1, seed=3, realisation=q) for q in range(2)]
    with she.Handle(insts, precision=precision, stats=she.STAT_SPATIAL, sample_every=1) as h:
        h.run(1)
        u = h.read_field(1)
        got = h.stats(1)["sum_u"]
    # additions in one chain: at most 8 x 4 x 17 in a thread (spans of 16384),
    # 8 in the block tree, then at most 4 + 8 over 1024 partials; numpy's own
    # sum adds up to 128 + log2(n) roundings
    assert abs(got - u.sum()) <= (544 + 8 + 12 + 160) * EPS * np.abs(u).sum()


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 130, 257, 1024])
@pytest.mark.parametrize("bc", [0, 1])
def test_sk_from_the_covariance(she, n, bc):
    ul, ur = (1.1, 0.9) if bc else (1.0, 1.0)
    inst = she.Instance(n=(n,), bc=bc, r=0.1, eps=1e-2, u_left=ul, u_right=ur, init_sd=0.1, seed=11)
    with she.Handle([inst], precision=1, stats=she.STAT_MOMENTS | she.STAT_CORR, sample_every=3) as h:
        h.run(3 * 21)
        st = h.stats(0, corr=True, sk=True)
        only = h.stats(0, sk=True)
    want = np.abs(np.fft.fft(st["mean"])) ** 2 + np.real(np.diag(np.fft.fft(np.fft.ifft(st["corr"], axis=1) * n, axis=0)))
    # each of the ~3 N + N^2 terms is formed with a few roundings and summed in
    # chains of at most N / 64 + 6 and N / 64 + 6 + N additions
    scale = np.abs(st["mean"]).sum() ** 2 + np.abs(st["corr"]).sum()
    assert np.max(np.abs(st["sk"] - want)) <= (2 * n + 64) * EPS * scale
    np.testing.assert_array_equal(only["sk"], st["sk"])

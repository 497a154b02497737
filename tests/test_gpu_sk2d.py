"""Column transforms of the 2D structure factor: every height, few shells and
many, a wave per column group (few tiles) and several groups per wave."""
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


# one instance, and enough of them for more than 512 blocks of tiles
@pytest.mark.parametrize("nx,ny,count,precision",
                         [(nx, ny, count, p) for p, hs in ((0, (2, 4, 8, 16, 32, 64, 128, 256, 512, 1024)),
                                                           (1, (2, 16, 128, 512)))
                          for ny in hs for nx, many in ((64, 520), (1024, 260)) for count in (1, many)
                          if nx * ny * count * (1 + p) < 1 << 28])
def test_shells_of_one_sample(she, nx, ny, count, precision):
    insts = [she.Instance(n=(nx, ny), r=0.1, eps=1e-2, init_sd=0.1, seed=5, realisation=q) for q in range(count)]
    with she.Handle(insts, precision=precision, stats=she.STAT_SPATIAL | she.STAT_SK, sample_every=1) as h:
        h.run(1)
        got = [(h.read_field(q).reshape(ny, nx), h.stats(q, sk=True)) for q in {0, count - 1}]
    kx, ky = np.meshgrid(np.fft.fftfreq(nx, 1 / nx), np.fft.fftfreq(ny, 1 / ny))
    shell = np.floor(np.sqrt(kx * kx + ky * ky) + 0.5).astype(int).ravel()
    for u, st in got:
        assert st["n_samples"] == 1
        p = np.bincount(shell, (np.abs(np.fft.fft2(u - 1.0)) ** 2).ravel())
        modes = np.bincount(shell)
        np.testing.assert_array_equal(st["sk_modes"], modes)
        want = np.divide(p, modes, out=np.zeros(len(p)), where=modes > 0)
        # a few roundings of the state's precision per radix-2 stage, twice in
        # the power; the shell of k = 0 holds N u0 too and is left out
        eps = 2.0 ** (-23 if precision == 0 else -52)
        bar = 4 * (np.log2(nx * ny) + 4) * eps * want[1:].max()
        assert np.max(np.abs(st["sk"][1:] - want[1:])) <= bar

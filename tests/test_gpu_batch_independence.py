"""A rod's field does not depend on the batch it runs in or on the launch shape:
the same bits from every kernel that may serve it."""
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


def field(she, insts, precision, steps=9, **kw):
    """Field of the last instance."""
    with she.Handle(insts, precision=precision, **kw) as h:
        h.step(steps)
        return h.read_field(len(insts) - 1)


# up to 256 cells: numbers drawn ahead by other waves; above: by every wave;
# beside an implicit rod of 100 cells: with that kernel's solve compiled in, and of
# 600: the kernel with one barrier per stage
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("n", [40, 130, 301, 700])
def test_composite_rod(she, n, bc, scheme, precision):
    rng = np.random.default_rng(n)
    gap = 0.1 * bc
    rod = she.Instance(n=(n,), bc=bc, scheme=scheme, r=0.1, eps=1e-2, u_left=1.0 + gap, u_right=1.0 - gap, init_sd=0.1,
                       seed=5, cond=0.5 + rng.random(n), cap=0.7 + 0.6 * rng.random(n))
    want = field(she, [rod], precision)
    for other in (she.Instance(n=(300,)), she.Instance(n=(100,), scheme=she.BE), she.Instance(n=(600,), scheme=she.BE)):
        np.testing.assert_array_equal(field(she, [other, rod], precision), want)
    if n <= 512:
        np.testing.assert_array_equal(field(she, [rod], precision, block_threads=64), want)


# one wave with 1, 2, 4, 8 cells per lane (full and not), and one barrier per
# level above 512 cells; each alone, beside rods of every other kind, and with the
# smallest workgroups; with a composite rod among them every rod's coefficients come
# from a table.  FP64 shows the order of the elimination in the last bits.
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("scheme", [2, 3])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("n", [60, 64, 65, 128, 200, 257, 511, 600])
def test_implicit_rod(she, n, bc, scheme, precision):
    gap = 0.1 * bc
    rod = she.Instance(n=(n,), bc=bc, scheme=scheme, r=2.0, eps=1e-3, u_left=1.0 + gap, u_right=1.0 - gap, init_sd=0.1,
                       seed=5)
    others = [she.Instance(n=(m,), bc=1, scheme=s, r=r, eps=1e-3, u_left=1.1, u_right=0.9)
              for m, s, r in ((40, she.BE, 50.0), (100, she.HEUN, 0.1), (300, she.CN, 1.0), (700, she.BE, 5.0))]
    others.append(she.Instance(n=(50,), r=0.1, cond=np.linspace(0.5, 1.5, 50)))
    want = field(she, [rod], precision)
    for some in (others[:1], others[:2], others[:3], others[:4], others[4:], others):
        np.testing.assert_array_equal(field(she, some + [rod], precision), want)
    np.testing.assert_array_equal(field(she, [rod], precision, block_threads=512), want)
    if n <= 512:
        np.testing.assert_array_equal(field(she, [rod], precision, block_threads=64), want)

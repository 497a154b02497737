"""FP64 face normals against extended precision: the radius and angle functions
are written for the 2^23 arguments Box-Muller meets."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_fp64_normals_within_two_ulp():
    from paper_2406_12157_amd import she
    n = 1 << 20
    for seed, step in ((1, 0), (77, 12345)):
        z = she.debug_normals(seed, 3, 0, step, 0, n, she.F64)
        # the words of the blocks, then the definition in 64-bit significands
        blocks = np.arange(n // 4, dtype=np.uint32)
        ctr = np.stack([blocks, np.full_like(blocks, step), np.zeros_like(blocks), np.full_like(blocks, 3)], 1)
        w = she.debug_philox(seed, ctr).reshape(-1, 2, 2)
        assert np.array_equal(w[5].ravel(), oracle.philox(ctr[5], [seed, 0]))
        ua = ((w[..., 0] >> 9).astype(np.longdouble) + np.longdouble(0.5)) / np.longdouble(2 ** 23)
        m = (w[..., 1] >> 9).astype(np.int64)
        q = (m + (1 << 20)) >> 21
        pi4 = np.longdouble("0.785398163397448309615660845819875721")
        th = (m - (q << 21)).astype(np.longdouble) * (pi4 / np.longdouble(2 ** 20))
        c, s = np.cos(th), np.sin(th)
        q &= 3
        cc = np.choose(q, [c, -s, -c, s])
        ss = np.choose(q, [s, c, -s, -c])
        rho = np.sqrt(-2 * np.log(ua))
        want = np.stack([rho * cc, rho * ss], -1).ravel()
        # radius within 0.86 ulp, angle functions within 0.76 ulp (all arguments),
        # the product's rounding 0.5; an ulp is at most 2^-52 of the value
        err = np.abs(z.astype(np.longdouble) - want)
        assert np.all(err <= np.abs(want) * (0.86 + 0.76 + 0.51) * 2.0 ** -52)


def test_initial_normals_are_the_entry_points():
    from paper_2406_12157_amd import she
    n = 4096
    inst = she.Instance(n=(n,), u0=0.0, init_sd=1.0, seed=21, realisation=5)
    with she.Handle([inst], precision=she.F64) as h:
        np.testing.assert_array_equal(h.read_field(0), she.debug_normals(21, 5, 1, 0, 0, n, she.F64))

"""Direct DFT stages of the odd primes above 5 (axis lengths that are neither compiled nor dense).

Real transforms against numpy, prime factors alone, first, last and repeated, on the x, the y and the
outer axis, one and several sequences per tile.  Tolerance, relative 2-norm: a stage of radix R sums
(R - 1) / 2 <= 21 products in one chain, at worst half as many roundings of 1.1e-16, up to three stages
an axis and three axes: 3 x 3 x 11 x 1.1e-16 = 1.1e-14 if every one grew the same way; as random signs,
their root: 3 x 11 x 1.1e-16 = 4e-15.
"""

import numpy as np
import pytest

from helpers import ncomp

pytestmark = pytest.mark.gpu

TOL = 4e-15


@pytest.mark.parametrize("n", [7, 11, 13, 14, 259, 286, 299, 301, 343, 308])
@pytest.mark.parametrize("make_shape", [lambda n: (4, n), lambda n: (n, 6), lambda n: (3, n, 5), lambda n: (n, 2, 3)])
def test_prime_stages_match_numpy_and_invert(n, make_shape):
    from paper_2408_03804_amd.binding import FFTHomog
    shape = make_shape(n)
    h = FFTHomog(shape, "small", "linear_elastic", 2, tangent=True)
    x = np.random.default_rng(n).standard_normal((2, ncomp("small", len(shape))) + shape)
    spec = h.debug_rfft(x).cpu().numpy()
    ref = np.fft.rfftn(x, axes=tuple(range(2, 2 + len(shape))))
    assert np.linalg.norm(spec - ref) < TOL * np.linalg.norm(ref)
    back = h.debug_irfft(ref).cpu().numpy()
    assert np.linalg.norm(back - x) < 2 * TOL * np.linalg.norm(x)

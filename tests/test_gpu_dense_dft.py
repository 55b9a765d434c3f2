"""The folded dense DFT on the FP64 matrix cores (axis lengths without a compiled radix schedule).

Real transforms against numpy at the lengths where its tiles change: around multiples of 32 (row
tiles of 16 on half the length), the smallest and the largest length it takes, odd, even and prime
(130 and 255, without a large prime factor, are the direct stages' in 2D or in both),
on the x, the y and the outer axis, with tiles of one and of several sequences.  Tolerance, relative
2-norm: each axis sums n/2 <= 128 products in chains of 8, about (8 + n/32)/2 roundings of 1.1e-16
each way of growing, and the spectrum passes through three axes: 3 x 6 x 1.1e-16 = 2e-15.
"""

import numpy as np
import pytest

from helpers import ncomp

pytestmark = pytest.mark.gpu

TOL = 2e-15
LENGTHS = [17, 18, 31, 33, 34, 47, 63, 66, 97, 130, 199, 254, 255]


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("make_shape", [lambda n: (5, n), lambda n: (n, 6), lambda n: (3, n, 20), lambda n: (n, 4, 9)])
def test_dense_transform_matches_numpy_and_inverts(n, make_shape):
    from paper_2408_03804_amd.binding import FFTHomog
    shape = make_shape(n)
    h = FFTHomog(shape, "small", "linear_elastic", 2, tangent=True)
    x = np.random.default_rng(n).standard_normal((2, ncomp("small", len(shape))) + shape)
    spec = h.debug_rfft(x).cpu().numpy()
    ref = np.fft.rfftn(x, axes=tuple(range(2, 2 + len(shape))))
    assert np.linalg.norm(spec - ref) < TOL * np.linalg.norm(ref)
    back = h.debug_irfft(ref).cpu().numpy()
    assert np.linalg.norm(back - x) < 2 * TOL * np.linalg.norm(x)

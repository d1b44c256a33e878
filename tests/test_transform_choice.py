"""Which transforms a plan runs, on the host: BS_FFT_AUTO in float64 takes the
own ones on the documented sizes (powers of two from 64 to 512, 16, 32, and the
multiples of 8 from 40 to 504 with no prime factor above 7) and hipFFT's on every
other, 1024 among them, where BS_FFT_PRUNED is refused; mixed precision the own
ones on powers of two from 64; an explicit choice is kept."""
import math

import pytest

from paper_2406_07366_amd import binding as B

L = 2 * math.pi


def params(n, mode, precision):
    return B.make_params(L=L, a=1e-6, tol=1e-3, grid_n=n, w=4, alpha=30.0 / L, rcut=0.4 * L,
                         fft_mode=mode, precision=precision)


def smooth(n):
    for f in (2, 3, 5, 7):
        while n % f == 0:
            n //= f
    return n == 1


def pow2(n):
    return n & (n - 1) == 0


@pytest.mark.parametrize("n", range(16, 1025, 4))
def test_automatic_choice(n):
    own64 = n in (16, 32, 64, 128, 256, 512) or \
        (n % 8 == 0 and 40 <= n <= 504 and smooth(n))
    own32 = pow2(n) and 64 <= n <= 1024
    for precision, own in ((B.BS_FP64, own64), (B.BS_FP32_MIXED, own32)):
        want = B.BS_FFT_PRUNED if own else B.BS_FFT_LIBRARY
        assert B.params_transforms(params(n, B.BS_FFT_AUTO, precision)) == want
        assert B.params_transforms(params(n, B.BS_FFT_LIBRARY, precision)) == B.BS_FFT_LIBRARY
        if pow2(n) and n <= (512 if precision == B.BS_FP64 else 1024):
            assert B.params_transforms(params(n, B.BS_FFT_PRUNED, precision)) == B.BS_FFT_PRUNED
        else:
            with pytest.raises(B.BsError) as e:
                B.params_transforms(params(n, B.BS_FFT_PRUNED, precision))
            assert e.value.code == B.BS_EINVAL


def test_float64_1024_stays_on_hipfft():
    p = params(1024, B.BS_FFT_AUTO, B.BS_FP64)
    assert B.params_transforms(p) == B.BS_FFT_LIBRARY
    assert B.resolve_params(p).fft_mode == B.BS_FFT_LIBRARY

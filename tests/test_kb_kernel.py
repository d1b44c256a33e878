"""The float64 form of the backward Kaiser-Bessel kernel (bs_device.h, kb_phi64), as
written there, against its 80-bit value: relative error at rounding over the whole
support at every width, and up to the edge, where the form with one exponential alone
cancels (exp's own rounding is magnified by zeta |s - 1|; the bound is that of the
form with expm1 the kernel replaced, measured here beside it)."""
import math

import numpy as np
import pytest

LD = np.longdouble


def exact(z, zeta):
    s = np.sqrt((1 - z.astype(LD)) * (1 + z.astype(LD)))
    y = LD(zeta) * s
    with np.errstate(divide="ignore", invalid="ignore"):
        r = np.sinh(y) / y
    t = y * y
    series = 1 + t / 6 * (1 + t / 20 * (1 + t / 42 * (1 + t / 72)))
    return np.where(t < 1e-3, series, r) * LD(zeta) / np.sinh(LD(zeta))


def constants(zeta):
    c2 = math.exp(-2 * zeta)
    inv_den = 1 / (-math.expm1(-2 * zeta))
    return c2, inv_den, 2 * zeta * math.exp(-zeta) * inv_den


def one_exponential(z, zeta):
    c2, inv_den, edge = constants(zeta)
    s2 = 1 - z * z
    s = np.sqrt(np.where(s2 > 0, s2, 1))
    a = np.exp(zeta * (s - 1))
    return np.where(s2 <= 0, edge, (a - c2 / a) / s * inv_den)


def kb_phi64(z, zeta):
    _, _, edge = constants(zeta)
    s2 = 1 - z * z
    t = zeta * zeta * s2
    p = np.full_like(z, 1 / math.factorial(17))
    for k in range(7, -1, -1):
        p = p * t + 1 / math.factorial(2 * k + 1)
    return np.where(s2 <= 0, edge, np.where(t < 1, p * edge, one_exponential(z, zeta)))


def with_expm1(z, zeta):
    _, inv_den, edge = constants(zeta)
    s2 = 1 - z * z
    s = np.sqrt(np.where(s2 > 0, s2, 1))
    v = np.exp(zeta * (s - 1)) * (-np.expm1(-2 * zeta * s)) / s * inv_den
    return np.where(s2 <= 0, edge, v)


@pytest.mark.parametrize("sigma", [1.25, 1.5, 2.0, 4.0])
@pytest.mark.parametrize("w", range(4, 17))
def test_relative_error(w, sigma):
    zeta = 0.995 * w * math.pi * (1 - 1 / (2 * sigma))
    rng = np.random.default_rng(w)
    z = np.concatenate([rng.uniform(-1, 1, 20000), 1 - 10.0 ** rng.uniform(-16, -1, 20000),
                        [1.0, np.nextafter(1, 0), 1 - 2.0 ** -52, 0.0]])
    ref = exact(z, zeta)

    def err(v):
        return float((np.abs(v.astype(LD) - ref) / ref).max())

    new, old = err(kb_phi64(z, zeta)), err(with_expm1(z, zeta))
    # 1 - z^2 is rounded before any form: 2^-54 of it, doubled by z z's own
    # rounding, over s2 in the relative error of s; all forms share it
    assert new <= 1.2 * old
    near = np.abs(z) > 1 - 1e-9
    ref = ref[near]
    assert err(kb_phi64(z[near], zeta)) < 4e-15

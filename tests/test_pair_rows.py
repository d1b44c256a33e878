"""CPU model of the float64 short-range cell rows (no GPU).

Points are binned in ncx x ncy x ncy cells, x fastest, edges of at least r_c / 3
along x and r_c / 2 along y and z (with room for a float32 margin of 1e-4
cells).  A target scans 5 x 5 rows of cells along x, each cut to the cells that
meet the sphere of radius r_c, the part beyond the periodic boundary as a range
of its own.  With the kernel's float32 index arithmetic: every point within
r_c (minimum image) lies in the ranges, and the ranges never overlap.
"""
import math

import numpy as np
import pytest

L = 2 * math.pi
MARGIN = np.float32(1e-4)
F = np.float32


def cells(rc, nq):
    q = L / (rc * (1 + 2e-4))
    cap = np.cbrt(max(1024.0, min(float(nq), 1 << 21)) / 1.5)
    ny = math.floor(min(2 * q, cap, 340.0))
    if ny < 5:
        return 1, 1
    return math.floor(min(3 * q, 1.5 * ny)), ny


def ranges(w, rc, ncx, ncy):
    fx, fy = ncx / L, ncy / L
    cx, cy, cz = F(w[0] * fx), F(w[1] * fy), F(w[2] * fy)
    ry = F(F(rc * fy) + MARGIN)
    ratio = F(F(ncx) / F(ncy))
    out = []
    for lane in range(64):
        r = lane & 31
        iz = (r * 13) >> 6
        iy = r - 5 * iz
        jy, jz = int(np.floor(cy - ry)) + iy, int(np.floor(cz - ry)) + iz
        dy = max(F(jy) - cy, cy - F(jy + 1), F(0))
        dz = max(F(jz) - cz, cz - F(jz + 1), F(0))
        d2 = F(ry * ry - dy * dy - dz * dz)
        if r >= 25 or d2 <= 0:
            continue
        xr = F(F(np.sqrt(d2)) * ratio + MARGIN)
        x0, x1 = int(np.floor(cx - xr)), int(np.floor(cx + xr))
        a, b = max(x0, 0), min(x1, ncx - 1)
        if lane >= 32:
            a = x0 + ncx if x0 < 0 else 0
            b = ncx - 1 if x0 < 0 else x1 - ncx
        jy += ncy if jy < 0 else (-ncy if jy >= ncy else 0)
        jz += ncy if jz < 0 else (-ncy if jz >= ncy else 0)
        assert 0 <= jy < ncy and 0 <= jz < ncy
        if b >= a:
            assert 0 <= a and b < ncx
            out.append((a, b, jy, jz))
    return out


def test_division_by_five():
    assert [(r * 13) >> 6 for r in range(25)] == [r // 5 for r in range(25)]


@pytest.mark.parametrize("rc", [0.047, 0.144, 0.2917, 0.6, 1.225, 2.4, 2.5124, 3.1])
@pytest.mark.parametrize("nq", [100, 40000, 2000000])
def test_every_point_within_rc_is_in_one_range(rc, nq):
    ncx, ncy = cells(rc, nq)
    assert ncx * ncy * ncy <= 2048 * 2048
    if ncy == 1:
        return                          # one cell holds every point
    assert ncy >= 5 and ncx >= 7
    assert L / ncx >= rc / 3 and L / ncy >= rc / 2
    rng = np.random.default_rng(int(rc * 1000) + nq)
    edge = np.array([0.0, np.nextafter(L, 0), rc, L - rc, L / ncx, 3 * L / ncy])
    targets = np.concatenate([rng.uniform(0, L, (60, 3)), rng.choice(edge, (60, 3))])
    for w in targets:
        # points on and inside the sphere's surface, and at cell boundaries
        u = rng.standard_normal((400, 3))
        u *= (rc * rng.choice([1 - 1e-12, 0.999, 0.5], (400, 1))) / np.linalg.norm(u, axis=1, keepdims=True)
        p = w + u
        p -= L * np.floor(p / L)
        p[(p < 0) | (p >= L)] = 0.0
        nc = np.array([ncx, ncy, ncy])
        c = np.minimum((p / L * nc).astype(int), nc - 1)
        hit = np.zeros(len(p), int)
        for a, b, jy, jz in ranges(w, rc, ncx, ncy):
            hit += (c[:, 0] >= a) & (c[:, 0] <= b) & (c[:, 1] == jy) & (c[:, 2] == jz)
        d = p - w
        d -= L * np.rint(d / L)
        near = (d ** 2).sum(1) < rc * rc
        assert (hit[near] == 1).all()
        assert (hit <= 1).all()

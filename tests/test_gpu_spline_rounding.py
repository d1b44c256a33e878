"""Rounding of the spline solves against the same systems solved in 80 bits, on
unevenly spaced nodes, which magnify it.  The bounds are 1.2 times the errors of the
solve whose quotients are all correctly rounded divisions (cubic: second
derivatives 2.1e-14; quintic on the same curves 1.4e-13 in the slopes, on 200-node
curves, beyond the LDS, 3.2e-14); rows scaled by reciprocals gave 3.0e-14, 1.8e-13
and 1.1e-13.  On the grid of 64^3 the small input's kernel solves, on 68^3 the
general one, where they hold filaments of the length."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu
LD = np.longdouble


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def uneven(nfil, n, seed):
    """Closed curves with nodes at random angles."""
    rng = np.random.default_rng(seed)
    fs = W.ellipses(nfil, n, seed=seed)
    x = []
    for _ in range(nfil):
        th = np.sort(rng.uniform(0, 2 * np.pi, n)) + np.arange(n) * 1e-3
        a, b = rng.uniform(.3, 1.0, 2)
        c = rng.uniform(0, 6.28, 3)
        R = W.haar_rotations(rng, 1)[0]
        x.append(c + np.stack([a * np.cos(th), b * np.sin(th), 0.2 * np.cos(3 * th)], 1) @ R.T)
    fs.xyz = np.concatenate(x)
    return fs


def solve(A, b):
    A, b, n = A.copy(), b.copy(), len(A)
    for k in range(n):
        p = k + np.argmax(np.abs(A[k:, k]))
        if p != k:
            A[[k, p]], b[[k, p]] = A[[p, k]], b[[p, k]]
        f = A[k + 1:, k] / A[k, k]
        nz = np.nonzero(f)[0]
        A[k + 1 + nz, k:] -= f[nz, None] * A[k, k:]
        b[k + 1 + nz] -= f[nz, None] * b[k]
    x = np.zeros_like(b)
    for k in range(n - 1, -1, -1):
        x[k] = (b[k] - A[k, k + 1:] @ x[k + 1:]) / A[k, k]
    return x


def spline(x, order):
    """Slopes and second derivatives at the nodes of the periodic spline through x
    on chord-length knots: C2 cubic or C4 quintic Hermite segments."""
    n, x = len(x), x.astype(LD)
    d = np.roll(x, -1, 0) - x
    h = np.sqrt((d ** 2).sum(1))
    hm, dm = np.roll(h, 1), np.roll(d, 1, 0)
    k = np.arange(n)
    km, kp = (k - 1) % n, (k + 1) % n
    if order == 4:
        A = np.zeros((n, n), LD)
        A[k, km] += h
        A[k, k] += 2 * (h + hm)
        A[k, kp] += hm
        D = solve(A, 3 * (h[:, None] * dm / hm[:, None] + hm[:, None] * d / h[:, None]))
        hh = h[:, None]
        return D, 2 * (3 * d - 2 * hh * D - hh * np.roll(D, -1, 0)) / hh ** 2
    A, b = np.zeros((2 * n, 2 * n), LD), np.zeros((2 * n, 3), LD)
    for i in range(n):     # third and fourth derivatives match
        m, p, jm, jp = 1 / hm[i], 1 / h[i], km[i], kp[i]
        r = A[2 * i]
        r[2 * jm] += -8 * m * m
        r[2 * jm + 1] += -m
        r[2 * i] += 12 * (p * p - m * m)
        r[2 * i + 1] += 3 * (m + p)
        r[2 * jp] += 8 * p * p
        r[2 * jp + 1] += -p
        b[2 * i] = 20 * (d[i] * p ** 3 - dm[i] * m ** 3)
        r = A[2 * i + 1]
        r[2 * jm] += 14 * m ** 3
        r[2 * jm + 1] += 2 * m * m
        r[2 * i] += 16 * (m ** 3 + p ** 3)
        r[2 * i + 1] += -3 * (m * m - p * p)
        r[2 * jp] += 14 * p ** 3
        r[2 * jp + 1] += -2 * p * p
        b[2 * i + 1] = 30 * (dm[i] * m ** 4 + d[i] * p ** 4)
    s = np.abs(A).max(1)[:, None]
    X = solve(A / s, b / s)
    return X[0::2], X[1::2]


@pytest.mark.parametrize("grid", [64, 68])
@pytest.mark.parametrize("nfil,n,seed,order,what,bound", [
    (20, 60, 2, 4, "sddot", 1.2 * 2.1e-14),
    (20, 60, 2, 6, "sdot", 1.2 * 1.4e-13),
    (4, 200, 5, 6, "sdot", 1.2 * 3.2e-14),
])
def test_rounding(B, nfil, n, seed, order, what, bound, grid):
    fs = uneven(nfil, n, seed)
    print(f"\n[case] order {order}, {nfil} x {n} nodes, grid {grid}", flush=True)
    plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=grid, w=8, alpha=3.5 / (0.3 * fs.L),
                                rcut=0.3 * fs.L, spline_order=order))
    xyz, g = B.load_workload(fs)
    plan.set_filaments(fs.offsets, xyz, g)
    got = plan.geometry()[what].cpu().numpy()
    plan.status()
    plan.close()
    ref = np.concatenate([spline(fs.xyz[a:b], order)[0 if what == "sdot" else 1]
                          for a, b in zip(fs.offsets[:-1], fs.offsets[1:])])
    err = float(np.sqrt(((got - ref) ** 2).mean() / (ref ** 2).mean()))
    print(f"  {what} {err:.2e} (bound {bound:.2e})")
    assert err < bound

"""Filaments crowded into a small part of the box: a few spread tiles and cells
hold all points, so that the per-bin order, the spread and the pair sums meet
bins of thousands of entries.  Against the sums over the plan's own quadrature
points in float64 (1e-12, in mixed precision the float32 terms' 1e-5; points
formed again elsewhere differ by their rounding, 1e-12 of the distances here),
twice with equal bits (bins ordered by index), and no stage may take the time that work
quadratic in a bin's entries would (the binning of the densest of these took
1.5 s that way; 5 ms is 7 times what it takes)."""
import math

import numpy as np
import pytest

from scipy.special import erfc

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def cluster(nfil, n_per, R, seed=6):
    """Ellipses of half the radius R around centres within R / 2 of a point."""
    fs = W.ellipses(nfil=nfil, n_per=n_per, seed=seed)
    c = np.repeat(fs.xyz.reshape(nfil, n_per, 3).mean(1), n_per, 0)
    rng = np.random.default_rng(seed)
    cen = np.repeat(rng.uniform(-0.5, 0.5, (nfil, 3)) * R, n_per, 0)
    fs.xyz = (fs.xyz - c) * (0.5 * R / (math.pi / 3)) + cen + 0.37 * fs.L
    return fs


def short_range(fs, geo, alpha, rc, targets, Q):
    """eq:velocity_shortrange over the given points, the two segments next to
    each target left out."""
    qp, qc = geo["qpos"].cpu().numpy(), geo["qcharge"].cpu().numpy()
    seg = np.arange(len(qp)) // Q
    prev = np.arange(fs.n_nodes) - 1
    prev[fs.offsets[:-1]] = fs.offsets[1:] - 1
    out = np.zeros((len(targets), 3))
    for k, i in enumerate(targets):
        r = qp - fs.xyz[i]
        r -= fs.L * np.rint(r / fs.L)
        d = np.sqrt((r ** 2).sum(1))
        ok = (d < rc) & (seg != i) & (seg != prev[i])
        r, d, x = r[ok], d[ok], alpha * d[ok]
        w = (erfc(x) + 2 / math.sqrt(math.pi) * x * np.exp(-x * x)) / d ** 3
        out[k] = (w[:, None] * np.cross(r, qc[ok])).sum(0) / (4 * math.pi)
    return out


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("grid,R,nfil", [(128, 0.02, 200), (96, 0.02, 200), (128, 0.1, 200),
                                         (256, 0.05, 200), (60, 0.03, 40)])
def test_crowded_bins(B, grid, R, nfil, mixed):
    fs = cluster(nfil, 100, R * 2 * math.pi)
    print(f"\n[case] {fs.n_nodes} nodes in {R} L on {grid}^3, mixed {mixed}", flush=True)
    plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=grid,
                                precision=B.BS_FP32_MIXED if mixed else B.BS_FP64))
    xyz, g = B.load_workload(fs)
    p = plan.params()
    v = []
    for _ in range(2):
        plan.set_filaments(fs.offsets, xyz, g)
        v.append(plan.velocity().cpu().numpy())
    assert np.array_equal(v[0], v[1])
    t = {k: x.cpu().numpy() for k, x in plan.velocity_terms().items()}
    plan.set_profiling(True)
    ms = []
    for _ in range(3):
        plan.stage_times(reset=True)
        plan.set_filaments(fs.offsets, xyz, g)
        plan.velocity()
        ms.append(plan.stage_times(reset=True)["binning"][0])
    plan.status()
    geo = plan.geometry()
    plan.close()
    tg = np.arange(0, fs.n_nodes, fs.n_nodes // 150)
    ref = short_range(fs, geo, p.alpha, p.rcut, tg, p.Q)
    err = np.linalg.norm(t["short"][tg] - ref) / np.linalg.norm(ref)
    whole = np.linalg.norm(v[0] - (t["local"] + t["short"] + t["long"] - t["self"]))
    whole /= np.linalg.norm(v[0])
    print(f"  short {err:.2e}, sum of terms {whole:.2e}, binning {min(ms):.3f} ms")
    assert err < (1e-5 if mixed else 1e-12)
    assert whole < (1e-6 if mixed else 1e-12)
    assert min(ms) < 5.0

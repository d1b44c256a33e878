"""Near-singular integrals of nodes above the middle of a straight segment at a third
of its length (and at h / 9, h / 27), where the panels' triples meet the segment's
ends to rounding: the graded panels against the closed form of a straight segment's
velocity minus its Q-point sum.  The rule's error is 4e-12 of the integral: 1e-10."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def ladder(gap, n=16, h=0.375):
    """Two lines along x, the second's nodes above the middles of the first's
    segments."""
    x = np.arange(n) * h
    a = np.stack([x, np.full(n, 1.0), np.full(n, 2.0)], 1)
    b = np.stack([x + 0.5 * h, np.full(n, 1.0 + gap), np.full(n, 2.0)], 1)
    return W.FilamentSet("ladder", n * h, 1e-6, np.array([0, n, 2 * n], dtype=np.int64),
                         np.concatenate([a, b]), np.array([1.0, 0.7]), 32, 1e-6,
                         periods=np.array([[1, 0, 0], [1, 0, 0]]))


@pytest.mark.parametrize("triples", [1, 2, 3])
def test_triples_that_meet_the_ends(B, triples):
    h = 0.375
    gap = h / 3.0 ** triples
    fs = ladder(gap)
    print(f"\n[case] gap h / {3 ** triples}", flush=True)
    plan = B.Plan(B.params_for(fs, ns_mode=B.BS_NS_ADAPTIVE))
    plan.set_periods(fs.periods)
    xyz, g = B.load_workload(fs)
    plan.set_filaments(fs.offsets, xyz, g)
    got = plan.velocity_terms()["ns"].cpu().numpy()
    pairs = plan.ns_counts()[0]
    geo = {k: v.cpu().numpy() for k, v in plan.geometry().items()}
    plan.status()
    plan.close()
    Q, L, N = 2, fs.L, fs.n_nodes
    seg0 = fs.xyz                                   # segment j from node j, along x
    ref, count = np.zeros((N, 3)), 0
    gam = np.repeat(fs.gamma, 16)
    for i in range(N):
        for j in range(N):
            if j // 16 == i // 16:
                continue                            # a line does not act on itself
            a = seg0[j] - fs.xyz[i]
            a -= L * np.rint((a + [0.5 * h, 0, 0]) / L)
            b = a + [h, 0, 0]
            t = np.clip(-a[0] / h, 0, 1)
            if np.linalg.norm(a + t * (b - a)) >= h:    # eta = 1: closer than the segment's length
                continue
            count += 1
            # integral of r x ds / r^3 along the segment, less the quadrature's sum
            e = np.array([1.0, 0, 0])
            d = a - a[0] * e                        # from the node to the line
            full = np.cross(d, e) / (d @ d) * (b[0] / np.linalg.norm(b) - a[0] / np.linalg.norm(a))
            s = np.zeros(3)
            for q in range(Q):
                r = geo["qpos"][Q * j + q] - seg0[j] + a
                s += np.cross(r, geo["qcharge"][Q * j + q]) / np.linalg.norm(r) ** 3
            ref[i] += (gam[j] * full - s) / (4 * np.pi)
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  pairs {pairs} ({count}), error {err:.2e}")
    assert pairs >= count and err < 1e-10

"""The near-singular search for nodes a rounding error below the box's origin (a
ring through a coordinate plane has such nodes: R cos(3 pi / 2) = -1.8e-16 R).  Folded
into the box they are 0, not L: the flagged pairs and the correction are those of
the same filaments moved away from the plane, to the rounding of the moved positions
(1e-15 of coordinates, pairs 0.02 apart: 1e-11)."""
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


@pytest.mark.parametrize("tiny", [-1e-17, -1.8e-16, 0.0])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_nodes_just_below_the_origin(B, axis, tiny):
    n, R, gap = 64, 0.5, 0.02
    th = 2 * np.pi * np.arange(n) / n
    u, v = R * np.cos(th), R * np.sin(th)
    u[np.abs(u) < 1e-12] = tiny            # the nodes on the plane
    rings = []
    for z, s in ((2.0, 1), (2.0 + gap, -1)):
        p = np.zeros((n, 3))
        p[:, axis], p[:, (axis + 1) % 3], p[:, (axis + 2) % 3] = u, 2.0 + s * v, z
        rings.append(p)
    fs = W.FilamentSet("rings", 2 * np.pi, 1e-6, np.array([0, n, 2 * n], dtype=np.int64),
                       np.concatenate(rings), np.array([1.0, 1.0]), 64, 1e-6)
    out = []
    for shift in (0.0, 0.3):
        print(f"\n[case] axis {axis}, {tiny}, moved by {shift}", flush=True)
        plan = B.Plan(B.params_for(fs, ns_mode=B.BS_NS_ADAPTIVE))
        xyz, g = B.load_workload(fs)
        plan.set_filaments(fs.offsets, xyz + shift, g)
        out.append((plan.ns_counts()[0], plan.velocity_terms()["ns"].cpu().numpy()))
        plan.status()
        plan.close()
    (na, va), (nb, vb) = out
    err = np.abs(va - vb).max() / np.abs(vb).max()
    print(f"  pairs {na} {nb}, error {err:.2e}")
    assert na == nb > 0 and err < 1e-11

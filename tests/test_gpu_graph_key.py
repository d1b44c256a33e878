"""When a recorded bs_step graph may be replayed.  It holds the plan's buffers
in its kernel arguments, so a bs_set_filaments with other offsets (which may move
them) has to drop it; and a replay rewrites what a pair search left running on
the second stream by an earlier bs_set_filaments reads, so it waits for that."""
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


@pytest.mark.parametrize("ns", [False, True])
def test_other_filaments_drop_the_recorded_graph(B, ns):
    import torch
    a, b = W.ellipses(nfil=5, n_per=40, seed=1), W.ellipses(nfil=150, n_per=64, seed=2)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        print(f"\n[case] graph, other filaments in between, ns {ns}", flush=True)
        plan = B.Plan(B.params_for(a, ns_mode=B.BS_NS_ADAPTIVE if ns else B.BS_NS_OFF), stream=s)
        xa, ga = B.load_workload(a)
        xb, gb = B.load_workload(b)
        out = torch.empty_like(xa)
        plan.set_filaments(a.offsets, xa, ga)
        ref = plan.velocity().cpu().numpy()
        plan.set_graph(True)
        plan.step(a.offsets, xa, ga, out)
        plan.step(a.offsets, xa, ga, out)
        if not plan.graph_active():
            pytest.skip("no graph recorded")
        plan.set_filaments(b.offsets, xb, gb)       # more nodes: buffers grow
        assert not plan.graph_active()
        plan.set_filaments(a.offsets, xa, ga)
        assert not plan.graph_active()
        for k in range(4):
            out.fill_(float(k))
            plan.step(a.offsets, xa, ga, out)
            assert plan.graph_active()
            assert np.array_equal(out.cpu().numpy(), ref), k
        plan.status()
        plan.close()


def test_replay_after_a_pending_pair_search(B):
    import torch
    fs = W.ringpairs(npairs=400, nbg=20, seed=3)
    fs.grid_n, fs.tol = 64, 1e-6
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        print("\n[case] graph replay after an eager set_filaments", flush=True)
        plan = B.Plan(B.params_for(fs, ns_mode=B.BS_NS_ADAPTIVE), stream=s)
        xyz, g = B.load_workload(fs)
        moved = xyz + 0.25
        out = torch.empty_like(xyz)
        plan.set_filaments(fs.offsets, xyz, g)
        ref = plan.velocity().cpu().numpy()
        n = plan.ns_counts()
        plan.set_graph(True)
        for k in range(6):
            plan.set_filaments(fs.offsets, moved, g)   # its search is left pending
            plan.step(fs.offsets, xyz, g, out)
            assert np.array_equal(out.cpu().numpy(), ref), k
            assert plan.ns_counts() == n
        plan.status()
        plan.close()


def test_replay_follows_the_networks_precision(B):
    """bs_mlp_set_fp32 between two steps: the second is the eager result."""
    import torch
    fs = W.ringpairs(npairs=100, nbg=4, seed=4)
    fs.grid_n, fs.tol = 64, 1e-1      # a budget that lets the network take pairs
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        print("\n[case] graph and the network's precision", flush=True)
        plan = B.Plan(B.params_for(fs, ns_mode=B.BS_NS_MLP, precision=B.BS_FP32_MIXED), stream=s)
        mlp = B.MLP(B.mlp_init(5), stream=s)
        plan.set_mlp(mlp, np.full(B.ns_error_bins()[2], 1e-6, np.float32))
        xyz, g = B.load_workload(fs)
        out = torch.empty_like(xyz)
        eager = {}
        for fp32 in (False, True):
            mlp.set_fp32(fp32)
            plan.set_filaments(fs.offsets, xyz, g)
            eager[fp32] = plan.velocity().cpu().numpy()
        assert not np.array_equal(eager[False], eager[True])
        plan.set_graph(True)
        for k, fp32 in enumerate((False, False, True, True, False)):
            mlp.set_fp32(fp32)
            plan.step(fs.offsets, xyz, g, out)
            assert np.array_equal(out.cpu().numpy(), eager[fp32]), k
        plan.status()
        plan.close()

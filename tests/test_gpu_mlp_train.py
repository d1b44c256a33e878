"""The training pass at the edges of its batches: fewer samples than a
wavefront's 16, one tile of a workgroup (64 in BF16, 32 in FP32) cut short and
just exceeded, and more tiles than workgroups (each then loops).  Gradients against the FP64
oracle: in FP32 mode sums of at most ~500 sequential float32 additions (a random walk of 6e-8 steps:
5e-6), in BF16 the 8-bit mantissas of the activations (3e-2 at a single sample).
The fused Adam step against the same step from the gradient in numpy."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def data(B, n, seed):
    import torch
    P = B.mlp_init(seed)
    rng = np.random.default_rng(seed + 1)
    X = rng.standard_normal((n, 8)).astype(np.float32)
    T = rng.standard_normal((n, 3)).astype(np.float32)
    return P, X, T, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()


@pytest.mark.parametrize("n", [1, 17, 32, 33, 64, 65, 20011])
@pytest.mark.parametrize("fp32", [True, False])
def test_gradient_at_batch_edges(B, n, fp32):
    P, X, T, Xd, Td = data(B, n, n)
    print(f"\n[case] batch {n} fp32 {fp32}", flush=True)
    m = B.MLP(P)
    m.set_fp32(fp32)
    loss, g = m.loss_grad(Xd, Td)
    P64 = P.astype(np.float64)
    if not fp32:
        o = 0
        for din, dout in ((8, 64), (64, 64), (64, 64), (64, 3)):
            P64[o:o + din * dout] = B.bf16_round(P[o:o + din * dout])
            o += din * dout + dout
    lr, gr = O.mlp_loss_grad(P64, X.astype(np.float64), T.astype(np.float64))
    e = np.linalg.norm(g.cpu().numpy() - gr) / np.linalg.norm(gr)
    print(f"  loss {abs(loss.item() / lr - 1):.2e} gradient {e:.2e}")
    assert e < (5e-6 if fp32 else 3e-2)
    assert abs(loss.item() / lr - 1) < (5e-6 if fp32 else 3e-2)


@pytest.mark.parametrize("fp32", [True, False])
def test_adam_step_is_the_gradient_step(B, fp32):
    import torch
    P, X, T, Xd, Td = data(B, 1000, 5)
    m = B.MLP(P)
    m.set_fp32(fp32)
    lr, b1, b2, eps = 1e-2, 0.9, 0.999, 1e-8
    p, mm, vv = (P.astype(np.float64), np.zeros(len(P)), np.zeros(len(P)))
    for k in (1, 2, 3):
        loss, g = m.loss_grad(Xd, Td)
        ls = torch.zeros(1, device="cuda")
        m.adam_step(Xd, Td, lr, b1, b2, eps, loss=ls)
        assert ls.item() == loss.item()
        g = g.cpu().numpy().astype(np.float64)
        mm = b1 * mm + (1 - b1) * g
        vv = b2 * vv + (1 - b2) * g * g
        p = p - lr * (mm / (1 - b1 ** k)) / (np.sqrt(vv / (1 - b2 ** k)) + eps)
        q = m.params().astype(np.float64)
        # float32 moments and parameters: a few ulp of the parameters per step,
        # 1e-5 of the step (the moments' and corrections' rounding)
        d = np.abs(q - p).max()
        print(f"  step {k}: {d:.2e}")
        assert d < 1e-6 + 1e-5 * lr * k
    # the kernels' weight images follow the parameters: a network made from
    # them gives the same values
    m2 = B.MLP(m.params())
    m2.set_fp32(fp32)
    assert torch.equal(m.forward(Xd), m2.forward(Xd))

"""The network's row kernels at the edges of their tiles: one row, a full and a just begun tile of 16,
and more tiles than workgroups (512), so that a workgroup takes several. Forward, loss and gradient
against FP64 (FP32 sums of at most 256 products in a row of four quarters, 2050 rows in a quarter of a
gradient: the bounds of the smaller batches' tests hold, 2e-5 and 1e-4 normwise); what has to be the
same bits: a row in any batch, a training step and its two halves, an output that overlaps its
input."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nfm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2011_08560_amd import nfm as m
    m.lib()
    return m


def _normwise(a, b):
    return np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)


@pytest.mark.parametrize("B", [1, 16, 17, 8200])
def test_rows(nfm, B):
    import torch
    from oracle import mlp as M
    print("rows", B, flush=True)
    rng = np.random.default_rng(B)
    net = nfm.Mlp(batch_max=B)
    net.init(3)
    theta, _ = net.get_params()
    P = M.unflatten(np.arange(M.N_PARAM))
    for name in ("b0", "b1", "b2", "b3"):
        idx = P[name].astype(int).reshape(-1)
        theta[idx] = rng.normal(0, 0.1, len(idx))
    norm = np.stack([rng.normal(0, 1, M.D_IN), rng.uniform(0.5, 2.0, M.D_IN)]).astype(np.float32)
    net.set_params(theta, norm)
    net.to_bf16()
    X = rng.normal(0, 1, (B, M.D_IN)).astype(np.float32)
    T = rng.normal(0, 1, (B, M.D_OUT)).astype(np.float32)
    Mk = (rng.random((B, M.D_OUT)) < 0.6).astype(np.float32)
    x, t, m = (torch.tensor(v, device="cuda") for v in (X, T, Mk))
    y, yb = net.forward(x), net.infer_bf16(x)
    assert _normwise(y.cpu().numpy(), M.forward(theta.astype(np.float64), norm.astype(np.float64),
                                                X.astype(np.float64))) <= 2e-5
    # a row in another batch, and in place of its own input
    lo = max(0, B - 21)
    assert torch.equal(net.forward(x[lo:].contiguous()), y[lo:])
    assert torch.equal(net.infer_bf16(x[lo:].contiguous()), yb[lo:])
    for f, want in ((net.forward, y), (net.infer_bf16, yb)):
        both = torch.zeros(B * 256 + 64, dtype=torch.float32, device="cuda")
        xin = both[64:64 + B * 81].view(B, 81)
        xin.copy_(x)
        out = both[:B * 256].view(B, 256)
        f(xin, out=out)
        assert torch.equal(out, want)
    loss = net.loss_grad(x, t, m)
    g = net.get_grads()
    L64, g64 = M.loss_and_grad(theta.astype(np.float64), norm.astype(np.float64), X.astype(np.float64),
                               T.astype(np.float64), Mk.astype(np.float64))
    assert abs(loss - L64) <= 2e-5 * L64
    G, G64 = M.unflatten(g.astype(np.float64)), M.unflatten(g64)
    for name in G64:
        assert _normwise(G[name], G64[name]) <= 1e-4, name
    # two steps in one call each, and in two
    net.adam(lr=1e-3)
    net.loss_grad(x, t, m)
    net.adam(lr=1e-3)
    p_halves, _ = net.get_params()
    net.set_params(theta, norm)
    for _ in range(2):
        net.train_step(x, t, m, lr=1e-3)
    p_steps, _ = net.get_params()
    assert np.array_equal(p_steps.view(np.uint32), p_halves.view(np.uint32))
    net.close()

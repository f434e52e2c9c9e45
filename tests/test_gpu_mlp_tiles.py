"""GPU: the network's products at the edges of their tiles (16 and 64 results a
side, steps of 32 along k) and on both sides of the choice between them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# omega (in = omega (omega + 3) / 2, out = omega), batch, hidden
SHAPES = [(2, 1, 16), (3, 17, 33), (13, 64, 31), (24, 256, 256), (6, 520, 1040)]


@pytest.mark.parametrize("omega,batch,hidden", SHAPES)
def test_gradients(oracle_mod, omega, batch, hidden):
    """Against the FP64 oracle.  A product rounds both operands to 8 bits (2^-8
    together) and six of them follow one another on the longest way to a
    gradient, so every element lies within 3e-2 of its block's largest."""
    import torch
    from paper_2001_01978_amd import warm
    net = warm.WarmNet(omega, hidden=hidden, seed=3)
    rng = np.random.default_rng(omega)
    X = rng.normal(size=(batch, warm.n_features(omega))).astype(np.float32)
    T = rng.uniform(0, 1, (batch, omega)).astype(np.float32)
    g, loss = net.gradients(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
    params = net.param_arrays()
    out, cache = oracle_mod.mlp_forward(params, X.astype(np.float64))
    l64, dout = oracle_mod.mlp_loss(out, T)
    want = np.concatenate([a.reshape(-1) for a in oracle_mod.mlp_backward(params, cache, dout)])
    got = g.cpu().numpy().astype(np.float64)
    assert abs(float(loss.item()) - l64) <= 3e-2 * abs(l64)
    o = 0
    for name, a in zip(["W1", "b1", "W2", "b2", "W3", "b3"], params):
        w = want[o:o + a.size]
        assert np.abs(got[o:o + a.size] - w).max() <= 3e-2 * np.abs(w).max(), name
        o += a.size


def test_tile_sizes_agree():
    """A row's logits do not depend on the batch: with 520 rows of 1040 hidden
    units the first layers use tiles of 64, with 50 rows tiles of 16, and
    both sum over k in the same order."""
    import torch
    from paper_2001_01978_amd import warm
    net = warm.WarmNet(6, hidden=1040, seed=1)
    X = torch.tensor(np.random.default_rng(0).normal(size=(520, warm.n_features(6))).astype(np.float32), device="cuda")
    all_rows = net.forward(X)
    for at in (0, 257, 470):
        assert torch.equal(net.forward(X[at:at + 50].contiguous()), all_rows[at:at + 50])

"""GPU: products of large full spaces, which go by orbit windows (window_impl.h),
and of the spaces below them, which take a row per lane (sigma_small_kernel).

The spaces cover every window width, one, two and three windows, half-filled,
sparse and mirrored fillings, and both sides of the rules that choose the
product's kernels.  Inputs are dyadic (every product and partial sum exact),
so results are compared with the oracle bit for bit.
"""
import math

import numpy as np
import pytest

from paper_2001_01978_amd import inputs

pytestmark = pytest.mark.gpu

SPACES = [
    (17, 1), (17, 16),   # a row per lane: one tile and a remainder
    (21, 10), (20, 14),  # a row per lane
    (40, 4), (36, 33),   # the same with 64-bit state words
    (23, 10),            # just below the smallest space of windows
    (23, 11), (23, 12),  # one window of 7
    (24, 10), (24, 14),  # two windows of 4
    (24, 12),            # one window of 8
    (25, 9), (25, 16),   # windows of 5 and 4
    (26, 9), (26, 17),   # two windows of 5
    (27, 8), (27, 19),   # windows of 6 and 5, the fewest pairs
    (28, 8),             # two windows of 6
    (29, 8),             # windows of 7 and 6
    (31, 8), (31, 24),   # windows of 8 and 7; 7 pairs: a row per lane
    (33, 7),             # three windows (6, 6, 5), short segments in groups
]


@pytest.fixture(scope="module")
def pdg():
    import torch
    from paper_2001_01978_amd import pairdiag
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pairdiag.load()
    return pairdiag


@pytest.mark.parametrize("om,n", SPACES)
def test_product_exact(pdg, oracle_mod, om, n):
    import torch
    _, _, eps, V = inputs.dyadic_instance(om, n, seed=om + n)
    x = inputs.dyadic_vector(om, math.comb(om, n), bits=6)
    want = oracle_mod.sigma(om, n, eps, V, oracle_mod.basis_alg1(om, n), x)
    b = pdg.Basis(om, n, store_states=True)    # the states lie behind the plan in the handle's buffer
    for dt in (torch.float64, torch.float32):
        xt = torch.tensor(x, dtype=dt, device="cuda")
        for _ in range(2):
            y = torch.full_like(xt, float("nan"))
            b.sigma(eps, V, xt, y)
            assert np.array_equal(y.cpu().numpy().astype(np.float64), want), (dt, om, n)
    got = b.states().cpu().numpy().view(np.uint64)
    assert np.array_equal(got, oracle_mod.basis_alg1(om, n))


def test_product_rounding(pdg, oracle_mod):
    """Random inputs, an x that starts on any 8-byte (4-byte) boundary: within
    the summation bound (hops + 2) u sum |H_ij x_j| of the oracle, every row."""
    import torch
    om, n = 23, 11
    _, _, eps, V = inputs.c5_instance(om, n, seed=3)
    d = math.comb(om, n)
    x = inputs.random_vector(5, d)
    basis = oracle_mod.basis_alg1(om, n)
    b = pdg.Basis(om, n, store_states=False)
    for dt, u in ((torch.float64, 2.0 ** -53), (torch.float32, 2.0 ** -24)):
        xt = torch.empty(d + 1, dtype=dt, device="cuda")[1:]
        xt.copy_(torch.tensor(x))
        xd = xt.cpu().numpy().astype(np.float64)
        want = oracle_mod.sigma(om, n, eps, V, basis, xd)
        scale = oracle_mod.sigma(om, n, np.abs(eps), np.abs(V), basis, np.abs(xd))
        y = b.sigma(eps, V, xt).cpu().numpy().astype(np.float64)
        # (FP32 also rounds the couplings: one more u per term)
        assert np.all(np.abs(y - want) <= (n * (om - n) + 4) * u * scale), dt


@pytest.mark.parametrize("om,n", [(34, 17), (35, 17)])
def test_every_row_of_a_far_space(pdg, om, n):
    """Above 2^32 bytes the 64 lanes of a wave can lie further apart than a 32-bit offset
    reaches (at 34 orbits in FP64 only, at 35 in FP32 too, at other places).  All terms of a
    row are positive, so every row of the FP32 product is within (hops + 4) 2^-24 of the FP64 one."""
    import gc
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    rng = np.random.default_rng(om)
    eps = rng.uniform(1.0, 3.0, om)
    V = rng.uniform(0.1, 0.3, (om, om))
    V = (V + V.T) / 2
    b = pdg.Basis(om, n, store_states=False)
    print(f"omega={om} n={n} dim={b.dim}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(om)
    x = torch.rand(b.dim, dtype=torch.float32, device="cuda", generator=g).add_(0.5)
    y32 = b.sigma(eps, V, x)
    x = x.double()
    y = b.sigma(eps, V, x)
    del x
    worst = 0.0
    for i in range(0, b.dim, 1 << 27):
        w = y[i:i + (1 << 27)]
        worst = max(worst, float(((y32[i:i + (1 << 27)].double() - w).abs_() / w).max()))
    print(f"worst relative difference {worst:.2e}", flush=True)
    del y, y32, w
    torch.cuda.empty_cache()
    assert worst <= (n * (om - n) + 4) * 2.0 ** -24

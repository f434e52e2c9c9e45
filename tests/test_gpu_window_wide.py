"""GPU: the windowed product with three windows of 6 to 8 orbits and up to 32
orbits below the top one (the 32-bit words of a lane's low state full)."""
import math

import numpy as np
import pytest

from paper_2001_01978_amd import inputs

pytestmark = pytest.mark.gpu

SPACES = [(36, 7), (37, 7), (37, 30), (38, 8), (39, 7), (39, 32), (40, 7), (40, 8), (40, 33)]


@pytest.mark.parametrize("om,n", SPACES)
def test_three_windows_exact(oracle_mod, om, n):
    """Dyadic inputs: sampled rows equal the oracle's, and every row of the FP32
    product the FP64 one's."""
    import torch
    assert torch.cuda.is_available()
    from paper_2001_01978_amd import pairdiag as pdg
    _, _, eps, V = inputs.dyadic_instance(om, n, seed=om + n)
    d = math.comb(om, n)
    b = pdg.Basis(om, n, store_states=False)
    g = torch.Generator(device="cuda").manual_seed(om * n)
    x = torch.randint(-63, 64, (d,), dtype=torch.float64, device="cuda", generator=g)
    y = b.sigma(eps, V, x, torch.full_like(x, float("nan")))
    y32 = b.sigma(eps, V, x.float(), torch.full_like(x, float("nan"), dtype=torch.float32))
    assert torch.equal(y32.double(), y)
    rng = np.random.default_rng(n)
    rows = np.unique(np.concatenate([rng.integers(0, d, 4000), np.arange(300), np.arange(d - 300, d)]))
    diag, tg, cf = oracle_mod.row_terms(om, n, eps, V, rows)
    at = lambda v, i: v[torch.tensor(i.reshape(-1), device="cuda")].cpu().numpy().reshape(i.shape)
    assert np.array_equal(at(y, rows), diag * at(x, rows) + (cf * at(x, tg)).sum(axis=1))

"""GPU: more streams than a handle has coefficient blocks, the first of them
alone on it for a while (its block then has no event to wait for)."""
import math

import numpy as np
import pytest

from paper_2001_01978_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("om,n", [(16, 8), (20, 9), (24, 11)])
def test_seven_streams_one_handle(oracle_mod, om, n):
    import torch
    from paper_2001_01978_amd import pairdiag as pdg
    basis = oracle_mod.basis_alg1(om, n)
    cases = []
    for s in range(7):
        _, _, eps, V = inputs.dyadic_instance(om, n, seed=90 + s)
        x = inputs.dyadic_vector(s, math.comb(om, n), bits=6)
        cases.append((eps, V, torch.tensor(x, device="cuda"), oracle_mod.sigma(om, n, eps, V, basis, x)))
    b = pdg.Basis(om, n, store_states=False)
    streams = [torch.cuda.Stream() for _ in cases]
    torch.cuda.synchronize()
    ys = []

    def issue(j):
        eps, V, x, _ = cases[j]
        with torch.cuda.stream(streams[j]):
            y = torch.full_like(x, float("nan"))
            b.sigma(eps, V, x, y, stream=streams[j])
            ys.append((j, y))

    for _ in range(4):
        issue(0)
    for _ in range(3):
        for j in (1, 2, 3, 4, 5, 6):     # the first stream stays away: its block is not taken
            issue(j)
    for _ in range(3):
        for j in range(7):
            issue(j)
    torch.cuda.synchronize()
    for j, y in ys:
        assert np.array_equal(y.cpu().numpy(), cases[j][3]), j

"""GPU: the three levels of the batched schedule (large teams, teams of 8 and
single workgroups), alone and together, against the oracle."""
import math

import numpy as np
import pytest

from paper_2001_01978_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pdg():
    import torch
    from paper_2001_01978_amd import pairdiag
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pairdiag.load()
    return pairdiag


# (spaces, teams reported): one workgroup per instance; teams of 8 only; large teams
# first, then teams of 8 and single workgroups
CASES = [
    ([(10, 5)] * 40 + [(9, 2)] * 8, 0),
    ([(14, 7)] * 40, 32),
    ([(20, 10)] * 9 + [(14, 7)] * 30 + [(10, 4)] * 20, 8),
]


@pytest.mark.parametrize("spaces,teams", CASES)
@pytest.mark.parametrize("block,krylov", [(128, 9), (256, 17), (512, 32)])
def test_levels(pdg, oracle_mod, spaces, teams, block, krylov):
    """krylov 9, 17, 32: the projection's bounds of 8, 16, 24 and 32 columns and one
    beyond each.  E0 within 1e-10 relative, occupations within 1e-8 (residuals of
    1e-11) of the oracle's dense solution, or of the single-instance solver beyond it."""
    insts = [inputs.family3_instance(500 + i, omega=om, n=n) for i, (om, n) in enumerate(spaces)]
    r = pdg.lanczos_ground_batched(insts, krylov=krylov, tol=1e-11, seed=3, block=block)
    assert r.status == pdg.PD_OK and r.converged.all()
    if r.info["grid"] >= 64 and r.info["grid"] % 64 == 0:
        assert r.info["teams"] == teams, r.info
    assert np.allclose([o.sum() for o in r.occ], [2.0 * n for _, n in spaces], atol=1e-9)
    seen = {}
    for q, (om, n, eps, V) in enumerate(insts):
        seen.setdefault((om, n), []).append(q)
    for (om, n), qs in seen.items():
        for q in qs[:1] + qs[-1:]:
            _, _, eps, V = insts[q]
            if math.comb(om, n) < 2000:
                e0, _, occ, _ = oracle_mod.dense_ground(om, n, eps, V)
            else:
                b = pdg.Basis(om, n, store_states=False)
                s = pdg.lanczos_ground(b, eps, V, krylov=20, tol=1e-11, start="random", seed=2, want_psi=False)
                e0, occ = s.E0, s.occ
            assert abs(r.E0[q] - e0) <= 1e-10 * abs(e0), (q, om, n)
            assert np.allclose(r.occ[q], occ, atol=1e-8), (q, om, n)


@pytest.mark.parametrize("m", [1, 2, 3, 20, 32])
def test_krylov_sizes_up_to_the_space(pdg, oracle_mod, m):
    """Spaces of m states (one pair on m orbits): the whole space is spanned, so
    the wave's tridiagonal solver sees every size and an invariant subspace."""
    insts = [inputs.family3_instance(70 + s, omega=m, n=1) for s in range(3)]
    r = pdg.lanczos_ground_batched(insts, krylov=32, tol=1e-10, seed=1, block=128)
    assert r.status == pdg.PD_OK and r.converged.all()
    for q, (om, n, eps, V) in enumerate(insts):
        e0, _, occ, _ = oracle_mod.dense_ground(om, n, eps, V)
        assert abs(r.E0[q] - e0) <= 1e-10 * max(abs(e0), 1.0)
        assert np.allclose(r.occ[q], occ, atol=1e-8)

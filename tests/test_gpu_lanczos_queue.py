"""Lanczos cycles whose steps are queued ahead of the host.

Only the orbits below r are coupled, so that with one pair and the start vector
on orbit 0 the Krylov space has exactly r vectors: the cycle ends there, inside a
run of steps that were already queued for every r but 1, 2, 4, 8 and 16.  The
products behind the end are not counted, the energy is the r x r block's
(tolerance 1e-10: FP64 rounding of a problem of norm 60 is 1e-14 of it), and one
more product confirms it.  Krylov sizes on either side of the instantiated column
counts run one restart each."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pdg():
    from paper_2001_01978_amd import pairdiag
    pairdiag.load()
    return pairdiag


@pytest.mark.parametrize("krylov", [6, 20])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 7, 9, 12, 17])
def test_invariant_subspace(pdg, oracle_mod, r, krylov):
    if r > krylov:
        pytest.skip("the space does not fit one cycle")
    om = 30
    rng = np.random.default_rng(r)
    eps = np.arange(om) + rng.uniform(0.0, 0.3, om)
    V = np.zeros((om, om))
    g = rng.uniform(1.0, 2.0, (r, r))
    V[:r, :r] = -(g + g.T) / 2
    E0, _, occ0, _ = oracle_mod.dense_ground(r, 1, eps[:r], V[:r, :r])
    b = pdg.Basis(om, 1, store_states=False)
    got = pdg.lanczos_ground(b, eps, V, krylov=krylov, tol=1e-11, start="e1")
    assert got.converged and abs(got.E0 - E0) <= 1e-10 * max(abs(E0), 1.0)
    assert np.allclose(got.occ[:r], occ0, atol=1e-8) and np.allclose(got.occ[r:], 0.0, atol=1e-12)
    assert got.iterations == (r + 1 if r > 1 else 1) and got.iterations_f32 == 0


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("krylov", [2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 21, 24, 25, 32, 33, 64])
def test_krylov_sizes(pdg, oracle_mod, krylov, precision):
    om, n = 12, 6
    rng = np.random.default_rng(7)
    eps = np.sort(rng.uniform(0.0, 4.0, om))
    g = rng.uniform(0.1, 0.6, (om, om))
    V = -(g + g.T) / 2
    E0, _, occ0, _ = oracle_mod.dense_ground(om, n, eps, V)
    b = pdg.Basis(om, n, store_states=False)
    got = pdg.lanczos_ground(b, eps, V, krylov=krylov, tol=1e-9, max_restarts=400, precision=precision)
    assert got.converged and abs(got.E0 - E0) <= 1e-9 * abs(E0)
    assert np.allclose(got.occ, occ0, atol=1e-7)

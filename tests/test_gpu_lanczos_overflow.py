"""GPU: a ground-state solve whose products overflow ends with PD_EDEVICE (its
tridiagonal matrix is not finite), neither converged nor after all restarts."""
import numpy as np
import pytest

from paper_2001_01978_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("om,n,start", [(8, 4, "random"), (8, 4, "e1"), (16, 8, "random"), (24, 12, "random")])
def test_overflowing_product(om, n, start, precision):
    import torch
    assert torch.cuda.is_available()
    from paper_2001_01978_amd import pairdiag as pdg
    _, _, _, V = inputs.c5_instance(om, n, seed=1)
    # every pair energy is finite, and every sum of n of them is not
    eps = np.linspace(3e307, 4e307, om)
    b = pdg.Basis(om, n, store_states=False)
    with pytest.raises(pdg.PairDiagError) as e:
        pdg.lanczos_ground(b, eps, V, krylov=20, tol=1e-10, max_restarts=50, start=start, seed=1,
                           precision=precision, want_psi=False)
    assert e.value.status == pdg.PD_EDEVICE, e.value

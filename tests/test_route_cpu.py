"""Host-only: which full spaces have the plan of the windowed product."""
import math

from paper_2001_01978_amd import pairdiag as pdg


def test_spaces_without_a_row_kernel_have_a_plan():
    """Below 2^32 states a row per lane is built for at most 11 pairs (or holes);
    every space with more carries the windowed product's plan in its buffer."""
    L = pdg.load()
    bare = L.pd_basis_bytes(2, 1, 0)
    seen = 0
    for om in range(1, 63):
        for n in range(om + 1):
            if 12 <= min(n, om - n) <= 20 and math.comb(om, n) < 2 ** 32:
                assert L.pd_basis_bytes(om, n, 0) > bare, (om, n)
                seen += 1
    assert seen

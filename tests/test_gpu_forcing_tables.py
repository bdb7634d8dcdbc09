"""Body-force tables formed on the device against the FP64 oracle's own: rows
that do not fill a workgroup, more columns than rows, wave numbers of either
sign and beyond the box's edge, and an edge beyond 65536, where the phase index
needs a 64-bit product.

From rest the velocity after two steps is the force itself, so the velocity
bars of the parity comparison bound the tables' error.
"""
import numpy as np
import pytest

import oracle as O
from parity import check
from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 8, 8), (9, 31, 13), (8, 8, 1100), (65544, 8, 8)])
def test_forced_from_rest(shape):
    from paper_2505_01126_amd import lbm

    rng = np.random.default_rng(shape[0])
    ks = [(0, 3, 1), (1, -2, 5), (-1, 1024, -3), (2, 0, -1024), (-2, 7, 9)]
    own = np.array([[*k, *(rng.standard_normal(6) * 1e-5)] for k in ks])
    modes = np.concatenate([I.forcing_modes(1e-5, seed=3), own])
    g = lbm.Lattice(shape, 0.8, two_phase=False, u0=np.zeros((3, *shape)), modes=modes, p0=1.0)
    o = O.Oracle(shape, 0.8, u0=np.zeros((3, *shape)), modes=modes, p0=1.0)
    g.step(2)
    o.step(2)
    m, mo = g.moments(), o.moments()
    check({"u": m["u"].cpu().numpy().astype(np.float64)}, {"u": mo["u"]}, label=str(shape))

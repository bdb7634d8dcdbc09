"""Harvested training rows against the FP64 oracle where the row writer's split
can go wrong: ranges shorter than, and not a multiple of, the 1024 sites listed
at a time, more ranges than one thread sums, more spheres than a launch carries
(32), both phase-field storages, and a capacity of nothing, of one row and of
all rows but one.

Inputs sit on the 2^-30 grid of the fixed-point storage, so both storages hold
them exactly: the stencil rows are the same 16-bit numbers, and the labels are
FP64 values rounded once to FP32 (half an ulp, 6e-8, taken as 1e-6 with the
cancellation in x - c).
"""
import numpy as np
import pytest

import oracle as O
from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,spheres,phi_storage", [
    ((9, 8, 11), 1, "f64"), ((31, 17, 29), 32, "fix32"), ((40, 44, 66), 33, "f64"), ((96, 110, 130), 40, "fix32"),
])
def test_rows_match_oracle(shape, spheres, phi_storage):
    from paper_2505_01126_amd import lbm

    rng = np.random.default_rng(spheres)
    c = rng.random((spheres, 3)) * np.array(shape[::-1])
    r = rng.uniform(2.0, 5.0, spheres) * rng.choice([-1.0, 1.0], spheres)
    phi = rng.random(shape) * 1.5 - 0.25  # a third of the cells outside the interface
    phi[shape[0] // 2] = 1.0              # and stretches without any
    phi = np.rint(phi * 2.0**30) / 2.0**30
    g = lbm.Lattice(shape, 0.8, phi0=phi, rho_l=1.0, rho_g=0.1, sigma=0.01, mobility=0.05, width=4.0, p0=0.0,
                    phi_storage=phi_storage)
    Xo, Yo, no = O.harvest(phi, c, r, cap=phi.size)
    for cap in (phi.size, no - 1, 1, 0):
        X, Y, n = g.harvest(c, r, cap=cap)
        m = min(cap, no)
        assert n == no and X.shape[0] == Y.shape[0] == m
        x16 = X.cpu().numpy().view(np.float16).astype(np.float64)
        np.testing.assert_array_equal(x16[:, :27], Xo[:m].astype(np.float16).astype(np.float64))
        assert (x16[:, 27:] == 0).all()
        np.testing.assert_allclose(Y.cpu().numpy(), Yo[:m], rtol=1e-6, atol=1e-6)

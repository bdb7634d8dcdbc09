"""Initial state, field read-out and reduction at the edges of their marches
(256 sites of a plane in small and ragged boxes; rows of 64 sites per wave, one,
two or four waves side by side, in chunks of planes, from 1.18 M sites on): every
field and statistic against the FP64 oracle's initial state."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from parity import check
from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 8), (9, 10, 63), (11, 9, 65), (40, 17, 128), (150, 127, 64), (81, 119, 126), (70, 71, 250),
          (71, 70, 257)]


def both(shape, two, storage, **kw):
    from paper_2505_01126_amd import lbm

    phi, _ = I.droplet(shape, 0.25 * min(shape), 4.0, seed=7, inside=0.0)
    u = I.random_u(shape, 0.02, seed=8)
    args = dict(rho_l=1.0, rho_g=0.2, sigma=0.005, mobility=0.05, width=4.0, p0=0.0) if two else dict(p0=1.0)
    args["modes"] = I.forcing_modes(1e-4, seed=9)
    phi = phi if two else None
    return (lbm.Lattice(shape, 0.7, phi0=phi, u0=u, storage=storage, **args, **kw),
            O.Oracle(shape, 0.7, phi0=phi, u0=u, **args))


@pytest.mark.parametrize("two,phs", [(True, "f64"), (True, "fix32"), (False, "f64")])
@pytest.mark.parametrize("shape", SHAPES)
def test_initial_fields_and_statistics(shape, two, phs):
    g, o = both(shape, two, "f32", phi_storage=phs)
    mg, mo = g.moments(), o.moments()
    u = mg["u"].double().cpu().numpy()
    # FP32 populations and arithmetic: the bar of the parity tests
    assert np.linalg.norm(u - mo["u"]) < 1e-5 * np.linalg.norm(mo["u"])
    # rho: four FP32 roundings of values up to 1
    assert np.abs(mg["rho"].double().cpu().numpy() - mo["rho"]).max() < 4 * 2.0 ** -24
    if two:
        assert np.abs(mg["phi"].cpu().numpy() - mo["phi"]).max() <= (2.0 ** -31 if phs == "fix32" else 0.0)
    rg, ro = g.reduce(), o.reduce()
    n = float(np.prod(shape))
    # sums of n values of relative error 1e-5 (u) or 1e-6 (rho, p*), each of size <= 1
    assert np.abs(rg[:7] - ro[:7]).max() < 1e-5 * n
    assert rg[7] == pytest.approx(ro[7], rel=1e-5) and rg[9] == 0
    f = mg["phi"].cpu().numpy()
    assert rg[0] == pytest.approx(f.sum(), rel=1e-13)
    uf = mg["u"].double().cpu().numpy()
    assert rg[7] == pytest.approx(np.sqrt((uf ** 2).sum(0)).max(), rel=1e-14)
    g.close()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_missing_outputs_are_left_alone(storage):
    import torch

    from paper_2505_01126_amd import lbm

    g, _ = both((9, 10, 70), True, storage)
    m = g.moments()
    u = torch.full_like(m["u"], float("nan"))
    lbm.lbm_moments(g.h, None, None, C.c_void_p(u.data_ptr()), None)
    assert torch.equal(u, m["u"])
    g.close()

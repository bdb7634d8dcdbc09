"""The step's options give the same bits for every work decomposition: the body
force (scalar rows and LDS twiddles in 64-wide tiles, vector rows in 32-wide
ones), the fixed-point phase field, the Runge-Kutta stages, the network pass with
its flags and plane ranges, buoyancy with two relaxation times, and the 16-bit
storages, at row lengths one past a tile or half a tile."""
import numpy as np
import pytest

from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


def fields_after(shape, tiling, steps, storage="f32", curv="fd", force=False, **kw):
    import torch

    from paper_2505_01126_amd import lbm

    phi = I.droplet(shape, 3.0, 4.0, seed=7)[0]
    if force:
        kw["modes"] = I.forcing_modes(1e-4, seed=9)
    g = lbm.Lattice(shape, 0.7, phi0=phi, u0=I.random_u(shape, 0.01, seed=8), storage=storage, rho_l=1.0, rho_g=0.2,
                    sigma=0.01, mobility=0.05, width=4.0, p0=0.0, curv_mode=curv, **kw)
    if curv == "mlp":
        w = (np.random.default_rng(3).standard_normal(6212) * 0.25).astype(np.float16)
        w[-3:] = [0.6, 0.5, 0.4]
        g.set_mlp(torch.tensor(w.view(np.int16), device="cuda"))
    if tiling is None:
        g.step(steps)
    else:
        b = lbm.Batch([g])
        b.set_tiling(*tiling)
        b.step(steps)
        b.close()
    m = {k: v.cpu().numpy() for k, v in g.moments().items()}
    g.close()
    return m


@pytest.mark.parametrize("opt", [
    dict(force=True), dict(phi_storage="fix32", force=True), dict(ac_rk3=True), dict(curv="mlp"),
    dict(curv="mlp", ac_rk3=True, force=True), dict(curv="mlp", phi_storage="fix32", storage="f16"),
    dict(gravity=(0.0, 1e-5, -1e-5), tau_g=0.6, storage="bf16", force=True),
    dict(gravity=(1e-5, 0.0, 0.0), tau_g=0.9, curv="mlp", storage="f16"),
], ids=lambda o: "-".join(k if v is True else str(v) for k, v in o.items()))
@pytest.mark.parametrize("shape", [(13, 19, 33), (9, 10, 65), (16, 12, 64)])
def test_same_bits_for_every_decomposition(shape, opt):
    ref = fields_after(shape, (64, shape[0]), 4, **opt)
    for tiling in (None, (64, 1), (32, 5), (32, 1), (64, 6)):
        m = fields_after(shape, tiling, 4, **opt)
        for k in ref:
            assert np.array_equal(ref[k], m[k]), (k, tiling)
    # the options act: the fields are not those of the plain step
    plain = fields_after(shape, None, 4, storage=opt.get("storage", "f32"))
    assert not np.array_equal(plain["u"], ref["u"]) and np.isfinite(ref["u"]).all()


@pytest.mark.parametrize("storage", ["f16", "f32"])
@pytest.mark.parametrize("shape", [(31, 51, 84), (44, 49, 82), (90, 30, 66), (30, 30, 96)])
def test_same_bits_for_small_ragged_boxes(shape, storage):
    # by default one round of 32-wide items for some of these, 64-wide ones for others
    ref = fields_after(shape, (64, 2), 2, storage=storage)
    for tiling in (None, (32, 1)):
        m = fields_after(shape, tiling, 2, storage=storage)
        for k in ref:
            assert np.array_equal(ref[k], m[k]), (k, tiling)

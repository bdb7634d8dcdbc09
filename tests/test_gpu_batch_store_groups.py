"""Batches whose boxes want different store policies: populations beyond 256 MB,
and boxes with nx a multiple of 64 (whole 128-byte lines) next to others.  By the
share of the former the step is one launch with cached stores, one with
non-temporal stores, or, beyond 3.3 GB, two launches; either way every box gives the bits that it
gives alone, in any order of the members, over graph replays and single steps."""
import functools

import numpy as np
import pytest

from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu

RAGGED, WHOLE, SMALL = (60, 101, 100), (49, 100, 128), (9, 8, 11)
RAGGED_L, WHOLE_L = (200, 190, 150), (200, 200, 256)


@functools.lru_cache(maxsize=8)
def fields(shape):
    phi = I.droplet(shape, 0.25 * min(shape), 4.0, seed=shape[2], inside=0.0)[0]
    return phi, I.random_u(shape, 0.01, seed=shape[1])


def make(shape, storage, two, curv="fd", **kw):
    import torch

    from paper_2505_01126_amd import lbm

    if storage != "f32":
        shape = (2 * shape[0],) + shape[1:]
    phi, u0 = fields(shape)
    args = dict(rho_l=1.0, rho_g=0.2, sigma=0.005, mobility=0.05, width=4.0, p0=0.0, curv_mode=curv) if two else {}
    g = lbm.Lattice(shape, 0.7, phi0=phi if two else None, u0=u0, storage=storage, **args, **kw)
    if curv == "mlp":
        w = (np.random.default_rng(3).standard_normal(6212) * 0.25).astype(np.float16)
        w[-3:] = [0.6, 0.5, 0.4]
        g.set_mlp(torch.tensor(w.view(np.int16), device="cuda"))
    return g


@pytest.mark.parametrize("storage,two,kw,tiling", [
    ("f32", True, {}, None), ("f32", True, {}, (32, 7)), ("f32", False, {}, (64, 5)), ("f16", True, {}, None),
    ("f16", True, {}, (32, 16)), ("f32", True, dict(ac_rk3=True), None), ("bf16", True, dict(phi_storage="fix32"), None),
    ("f32", True, dict(curv="mlp"), None)])
@pytest.mark.parametrize("shapes", [
    (RAGGED_L, WHOLE_L, SMALL),                # two thirds of the sites: two launches
    (RAGGED, WHOLE, SMALL),                    # half of them, too small for two: cached
    (SMALL, WHOLE, WHOLE),                     # nearly all: non-temporal
    (RAGGED, RAGGED, (20, 40, 64)),            # few: cached
])
def test_every_box_as_alone(shapes, storage, two, kw, tiling):
    import torch

    from paper_2505_01126_amd import lbm

    alone = [make(s, storage, two, **kw) for s in shapes]
    boxes = [make(s, storage, two, **kw) for s in shapes]
    b = lbm.Batch(boxes)
    if tiling:
        b.set_tiling(*tiling)
    b.step(3)
    boxes[0].step(1)  # on its own: the tables are made again
    b.step(2)
    for k, (g, a) in enumerate(zip(boxes, alone)):
        a.step(6 if k == 0 else 5)
        assert g.steps == a.steps
        m, ref = g.moments(), a.moments()
        for name in ref:
            assert torch.equal(m[name], ref[name]), (shapes[k], name)
    b.close()
    for g in alone + boxes:
        g.close()

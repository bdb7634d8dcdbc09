"""The step gives the same bits for every work decomposition and store policy:
tile width, planes per work item, workgroups against work items, cached or
non-temporal stores, at the sizes where tiles and items end."""
import numpy as np
import pytest

from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


def fields(shape, seed):
    r = 0.25 * min(shape)
    phi, _ = I.droplet(shape, r, 4.0, seed=seed, inside=0.0)
    return phi, I.random_u(shape, 0.01, seed=seed + 1)


def run(shape, two, storage, steps=3, tiling=None, others=(), **kw):
    """Fields after `steps`, the box advanced alone (tiling None) or in a batch."""
    from paper_2505_01126_amd import lbm

    def make(sh):
        phi, u = fields(sh, 5)
        args = dict(rho_l=1.0, rho_g=0.2, sigma=0.005, mobility=0.05, width=4.0, p0=0.0) if two else dict(p0=1.0)
        return lbm.Lattice(sh, 0.7, phi0=phi if two else None, u0=u, storage=storage, **args, **kw)

    boxes = [make(s) for s in (shape,) + tuple(others)]
    if tiling is None and not others:
        boxes[0].step(steps)
    else:
        b = lbm.Batch(boxes)
        if tiling:
            b.set_tiling(*tiling)
        b.step(steps)
        b.close()
    m = {k: v.cpu().numpy() for k, v in boxes[0].moments().items()}
    for g in boxes:
        g.close()
    return m


@pytest.mark.parametrize("two", [True, False])
@pytest.mark.parametrize("shape", [(8, 8, 8), (9, 11, 33), (17, 5 * 4 + 1, 65), (40, 30, 96), (13, 24, 64)])
def test_default_decomposition_is_exact(shape, two):
    ref = run(shape, two, "f32", tiling=(64, shape[0]))
    for tiling in (None, (64, 1), (32, 5)):
        m = run(shape, two, "f32", tiling=tiling)
        for k in ref:
            assert np.array_equal(ref[k], m[k]), (k, tiling)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_store_policy_is_exact(storage):
    # 256 MB of populations and rows of whole 128-byte lines: non-temporal
    # stores; together with a box of nx = 8, cached ones
    shape = (152, 128, 128) if storage == "bf16" else (80, 128, 128)
    ref = run(shape, True, storage)
    m = run(shape, True, storage, others=((8, 8, 8),))
    for k in ref:
        assert np.array_equal(ref[k], m[k]), k


@pytest.mark.parametrize("shape", [(64, 64, 64), (400, 20, 96)])
def test_items_beyond_the_grid(shape):
    """More work items than resident workgroups: the queue hands out the rest."""
    ref = run(shape, True, "f16", tiling=(64, shape[0]))
    m = run(shape, True, "f16", tiling=(64, 1))  # 1024 and 4000 items on 768 workgroups
    for k in ref:
        assert np.array_equal(ref[k], m[k]), k

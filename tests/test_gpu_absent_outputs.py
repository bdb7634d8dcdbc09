"""Read-out and set-up with outputs that are not asked for, in boxes large enough
for the marches by rows (one, two and four waves side by side, rows past the
first): what is asked for comes out as in the full call, bit for bit, whichever
of the four outputs are absent; a single-phase set-up has no phi and no u to
write."""
import ctypes as C
import itertools

import pytest

from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,two,storage", [((66, 73, 256), False, "f16"), ((80, 127, 128), False, "f32"),
                                               ((150, 127, 64), True, "bf16"), ((66, 73, 256), True, "f32")])
def test_each_output_alone(shape, two, storage):
    import torch

    from paper_2505_01126_amd import lbm

    phi = I.droplet(shape, 0.25 * min(shape), 4.0, seed=3)[0] if two else None
    args = dict(rho_l=1.0, rho_g=0.2, sigma=0.005, mobility=0.05, width=4.0, p0=0.0) if two else dict(p0=1.0)
    g = lbm.Lattice(shape, 0.7, phi0=phi, u0=I.random_u(shape, 0.02, seed=4), storage=storage, **args)
    full = g.moments()
    names = ("rho", "p", "u", "phi")
    for take in itertools.product((False, True), repeat=4):
        out = {k: torch.full_like(full[k], float("nan")) if t else None for k, t in zip(names, take)}
        lbm.lbm_moments(g.h, *(None if out[k] is None else C.c_void_p(out[k].data_ptr()) for k in names))
        for k in names:
            assert out[k] is None or torch.equal(out[k], full[k]), (k, take)
    g.close()

"""Set-up, read-out and reduction give the same fields and statistics whichever
way they go through a box: by sites (single phase, thin planes), by marches over
256 sites of a plane, or by rows of 64 (nx a multiple of 64, from 1.18 M sites on;
one, two or four waves side by side, rows and columns past the box's edge).

Two independent checks.  A periodic box repeated in x and y is the same flow, so
its fields equal those of the single period bit for bit.  And the ten statistics
are sums and maxima of the fields that are read out (rho and u are the very FP32
numbers that the reduction adds up in FP64), so they follow from those fields in
FP64 on the host: each sum to 1e-12 of the sum of its terms' magnitudes, a bound
on any order of the additions of up to 2^22 FP64 terms (2^22 x 2^-53 is 5e-10 in
the worst order; pairs and blocks as here stay below 1e-13), p* = 3 p / rho to four
FP32 roundings of its terms, maxima to one FP64 rounding."""
import numpy as np
import pytest

from paper_2505_01126_amd import inputs as I

pytestmark = pytest.mark.gpu


def smooth(shape, rng):
    """A field of a few waves, |values| up to 1, periodic in the box."""
    z, y, x = np.meshgrid(*(np.arange(n) / n for n in shape), indexing="ij")
    out = np.zeros(shape)
    for _ in range(4):
        k = rng.integers(-2, 3, 3)
        out += np.cos(2 * np.pi * (k[0] * z + k[1] * y + k[2] * x) + rng.uniform(0, 6.28)) / 4
    return out


def start(shape, seed):
    """phi with cells outside [0, 1], a velocity with a mean, a pressure that varies."""
    rng = np.random.default_rng(seed)
    z, _, x = np.meshgrid(*(np.arange(n) / n for n in shape), indexing="ij")
    phi = 0.5 + 0.6 * np.cos(2 * np.pi * (x + z))
    u = np.stack([0.01 * (a + 1) + 0.01 * smooth(shape, rng) for a in range(3)])
    return phi, u, 0.01 * smooth(shape, rng) + 0.02


def box(fields, two, storage, **kw):
    from paper_2505_01126_amd import lbm

    phi, u, ps = fields
    args = dict(rho_l=1.0, rho_g=0.2, sigma=0.005, mobility=0.05, width=4.0, p0=0.0) if two else dict(p0=1.0)
    g = lbm.Lattice(phi.shape, 0.7, phi0=phi if two else None, u0=u, pstar0=ps + (0.0 if two else 1.0),
                    storage=storage, **args, **kw)
    return g


@pytest.mark.parametrize("two,storage,phs", [(True, "f32", "f64"), (True, "bf16", "fix32"), (False, "f16", "f64")])
@pytest.mark.parametrize("period,repeats", [
    ((300, 8, 8), [(1, 2), (3, 3), (8, 8), (9, 16)]),  # thin; full planes; rows: one wave, and two side by side
    ((24, 13, 17), [(2, 3), (5, 4)]),                  # 221 sites: thin; ragged planes
    ((90, 11, 64), [(5, 4)]),                          # rows: four waves side by side
])
def test_a_repeated_period_is_the_same_flow(period, repeats, two, storage, phs):
    import torch

    f = start(period, 3)
    kw = dict(phi_storage=phs) if two else {}
    one = box(f, two, storage, **kw)
    fields = [one.moments()]
    one.step(2)
    fields.append(one.moments())
    for ry, rx in repeats:
        g = box(tuple(np.tile(a, (1,) * (a.ndim - 2) + (ry, rx)) for a in f), two, storage, **kw)
        for k, ref in enumerate(fields):
            m = g.moments()
            for name, v in ref.items():
                assert torch.equal(m[name], v.tile((1,) * (v.ndim - 2) + (ry, rx))), (ry, rx, k, name)
            if k == 0:
                g.step(2)
        g.close()
    one.close()


SHAPES = [(8, 8, 8), (33, 9, 8), (31, 13, 13), (20, 17, 17), (9, 10, 63), (40, 17, 128), (300, 63, 65),
          (290, 65, 64), (150, 127, 64), (80, 119, 128), (70, 71, 256), (17, 100, 704), (66, 141, 150)]


def check_statistics(g, two):
    m = {k: v.cpu().numpy().astype(np.float64) for k, v in g.moments().items()}
    r = g.reduce()
    rho, u, phi = m["rho"], m["u"], m["phi"]
    ps = 3.0 * m["p"] / rho
    e = 0.5 * rho * (u ** 2).sum(0)
    near = lambda v, t, tol: abs(v - t.sum()) <= tol * np.abs(t).sum()
    assert near(r[0], phi, 1e-12) and near(r[1], rho, 1e-12)
    assert near(r[2], ps, 4 * 2.0 ** -24)
    for a in range(3):
        assert near(r[3 + a], rho * u[a], 1e-12), a
        assert np.abs(rho * u[a]).sum() < 20 * abs((rho * u[a]).sum())  # the mean flow shows
    assert near(r[6], e, 1e-12)
    assert r[7] == pytest.approx(np.sqrt((u ** 2).sum(0)).max(), rel=2.0 ** -50)
    over = max((phi - 1.0).max(), (-phi).max()) if two else 0.0
    assert r[8] == pytest.approx(over, rel=2.0 ** -50) and (over > 1e-3) == two
    assert r[9] == 0


@pytest.mark.parametrize("two,storage,phs", [(True, "f32", "f64"), (True, "f16", "f64"), (True, "bf16", "fix32"),
                                             (False, "f32", "f64"), (False, "f16", "f64")])
@pytest.mark.parametrize("shape", SHAPES)
def test_statistics_of_the_fields(shape, two, storage, phs):
    kw = dict(modes=I.forcing_modes(1e-4, seed=9))
    g = box(start(shape, 5), two, storage, **kw, **(dict(phi_storage=phs) if two else {}))
    check_statistics(g, two)
    g.step(1)
    check_statistics(g, two)
    g.close()


@pytest.mark.parametrize("shape", [(8, 8, 8), (40, 20, 20), (48, 48, 48), (60, 141, 150), (72, 130, 128), (80, 66, 256)])
def test_statistics_with_the_network(shape):
    """The reduction and the read-out may take different ways here, whose u differ by an
    FP32 rounding at a few sites: taken as four of them at every site."""
    import torch

    w = (np.random.default_rng(3).standard_normal(6212) * 0.25).astype(np.float16)
    w[-3:] = [0.6, 0.5, 0.4]
    rng = np.random.default_rng(1)
    n = max(1, int(np.prod(shape)) // 20000)
    z, y, x = np.meshgrid(*(np.arange(k) for k in shape), indexing="ij")
    phi = np.ones(shape)
    for c in rng.uniform(0, 1, (n, 3)) * shape:
        d = [a - b for a, b in zip((z, y, x), c)]
        d = [a - k * np.rint(a / k) for a, k in zip(d, shape)]
        phi = np.minimum(phi, 0.5 + 0.55 * np.tanh((np.sqrt(sum(a * a for a in d)) - 3.0) / 2.0))
    _, u, ps = start(shape, 6)
    g = box((phi, u, ps), True, "f16", curv_mode="mlp")
    g.set_mlp(torch.tensor(w.view(np.int16), device="cuda"))
    m = {k: v.cpu().numpy().astype(np.float64) for k, v in g.moments().items()}
    r = g.reduce()
    for a in range(3):
        t = m["rho"] * m["u"][a]
        assert abs(r[3 + a] - t.sum()) <= 2.0 ** -22 * np.abs(t).sum()
    assert abs(r[0] - m["phi"].sum()) <= 1e-12 * np.abs(m["phi"]).sum()
    assert r[7] == pytest.approx(np.sqrt((m["u"] ** 2).sum(0)).max(), rel=2.0 ** -21)
    assert r[8] == pytest.approx(max((m["phi"] - 1.0).max(), (-m["phi"]).max()), rel=2.0 ** -50) and r[9] == 0
    g.close()

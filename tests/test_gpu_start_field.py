"""The start field's kernels at the edges of their loops: x chunks of 256 and
y tables of 128 nodes in the Fourier sums, several slabs of planes, edges too
short for all modes, tiles of many rows and planes, each storage convention,
and nodes in every quadrature rule.  Against the FP64 reference.

Tolerance 1e-12 of the largest speed and 1e-10 of the largest pressure, the
bounds the whole start field is held to: sums over N <= 3e5 nodes in FP64 carry
sqrt(N) 1e-16 < 1e-13 relative on either side, and the quadratures agree
within ~2e-15."""
import numpy as np
import pytest

from oracle import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    from paper_2403_05443_amd import lbell
    lbell.load()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return lbell


def _check(lat, shape, parts):
    mu = (1.0 - 0.5) / 3.0
    lat.stokes_start()
    rho, u = lat.fields(0)
    own = lat.mask(0)
    ref = [dict(centre=p[0], axes=p[1], q=np.array(p[2]), F=p[3], T=p[4], U=(0, 0, 0), W=(0, 0, 0),
                M=4 / 3 * np.pi * np.prod(p[1])) for p in parts]
    rr, ur = S.start_state(shape, own, ref, mu)
    fl = own == 0
    eu = np.abs(u[fl] - ur[fl]).max() / np.abs(ur[fl]).max()
    er = np.abs(rho[fl] - rr[fl]).max() / np.abs(rr[fl] - 1).max()
    print(f"{shape}: velocity {eu:.1e}, density {er:.1e}")
    assert eu < 1e-12 and er < 1e-10


def _particle(rng, centre, axes, torque=True):
    q = rng.normal(size=4)
    q /= np.linalg.norm(q)
    F, T = rng.normal(size=3) * 1e-4, rng.normal(size=3) * 1e-3
    return tuple(centre), tuple(axes), tuple(q), tuple(F), tuple(T) if torque else (0.0, 0.0, 0.0)


@pytest.mark.parametrize("shape,axes,torque", [
    ((300, 9, 7), (2.4, 1.2, 1.2), True),     # two x chunks
    ((8, 140, 6), (1.9, 1.0, 1.0), False),    # two y tables
    ((520, 4, 4), (0.9, 0.5, 0.5), True),     # modes cut short along two axes, tiles across planes
    ((4, 5, 70), (0.9, 0.9, 0.9), True),      # a sphere; 65 rows and 17 planes to a tile
    ((33, 34, 71), (9.0, 2.0, 2.0), True),    # slabs; every rule of a slender body
    ((64, 40, 40), (1.9, 1.0, 1.0), False),   # the far rules
    ((31, 29, 37), (3.0, 2.9, 2.9), True),    # nearly a sphere
])
def test_shapes(lb, shape, axes, torque):
    rng = np.random.default_rng(sum(shape))
    p = _particle(rng, [n / 2 + 0.3 * rng.uniform() for n in shape], axes, torque)
    lat = lb.Lattice([shape], collision="trt", tau=1.0, storage="fp64", max_semi_axis=10.0)
    lat.add_ellipsoid(p[0], p[1], p[2])
    lat.set_external(0, p[3], p[4])
    _check(lat, shape, [p])


@pytest.mark.parametrize("steps", [0, 1])
def test_in_place_conventions(lb, monkeypatch, steps):
    """One buffer in place: the state after an even and after an odd step."""
    shape, rng = (27, 22, 25), np.random.default_rng(3 + steps)
    monkeypatch.setenv("LBELL_K1_VARIANT", "12")
    parts = [_particle(rng, (7.2, 11.0, 12.5), (4.0, 2.0, 2.0)), _particle(rng, (20.1, 10.2, 11.9), (3.0, 2.5, 2.0))]
    lat = lb.Lattice([shape], collision="trt", tau=1.0, storage="fp64", max_particles=3)
    for i, p in enumerate(parts):
        lat.add_ellipsoid(p[0], p[1], p[2])
    lat.add_ellipsoid((13.0, 3.0, 3.5), (1.5, 1.5, 1.5), (1, 0, 0, 0))  # carries no load
    lat.step(steps)  # at rest: nothing moves
    for i, p in enumerate(parts):
        lat.set_external(i, p[3], p[4])
    _check(lat, shape, parts + [((13.0, 3.0, 3.5), (1.5, 1.5, 1.5), (1, 0, 0, 0), (0, 0, 0), (0, 0, 0))])

"""Fat bodies, whose link rebuild takes windows of more than 512 words, shells
of more than 1024 nodes, and the moments from the written list over many window
segments: the list in its order (window index, direction), and bodies that move
over nodes, step by step against the oracle.

A body starts at a speed of several nodes a hundred steps, so that nodes change
side and the links are rebuilt inside the steps too.  The oracle sums full
populations over N < 60000 links, known to about N w 2^-53 sqrt(N) = 6e-11 a
component, against a momentum of M U > 500: 1e-9 of the speed (the FP64 bound of
the parity tests) is far above that and far below a link's part in the drag
matrix, 1 / N."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# shape, lattice, semi-axes, whether the window spans an axis (2 ceil(a) + 6 nodes at most)
CASES = [((58, 56, 60), 19, (25.0, 20.0, 18.0), False),
         ((52, 50, 54), 27, (22.0, 20.0, 19.0), False),
         ((61, 62, 60), 19, (27.0, 27.0, 27.0), False),
         ((42, 44, 43), 19, (20.0, 19.5, 19.8), True)]


@pytest.mark.parametrize("shape,q,axes,spans", CASES)
def test_list_order_and_steps(orc, shape, q, axes, spans):
    import torch
    from paper_2403_05443_amd import lbell
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lat = lbell.Lattice([shape], collision="trt", tau=0.9, storage="fp64", max_semi_axis=max(axes), lattice=q)
    ora = orc.OracleSim(shape, "trt", 0.9, **({"lattice": 27} if q == 27 else {}))
    c, quat = [n / 2 - 0.3 for n in shape], np.array([0.9, 0.2, -0.3, 0.1]) / np.sqrt(0.95)
    U, W, F, T = (0.02, -0.03, 0.025), (4e-4, -3e-4, 5e-4), (1e-2, -2e-2, 1e-2), (1e-1, 2e-1, -1e-1)
    for s in (lat, ora):
        s.add_ellipsoid(c, axes, quat)
        s.set_velocity(0, U, W)
        s.set_external(0, F, T)

    def compare():
        site, way = (np.asarray(v).astype(np.int64) for v in lat.links(0))
        so, wo = (np.asarray(v).astype(np.int64) for v in ora.links(0))
        assert np.array_equal(np.sort(32 * site + way), np.sort(32 * so + wo))
        if not spans:  # window coordinates from any corner below the body
            lo = np.round(lat.particle(0)["x"]).astype(int) - int(max(axes)) - 3
            at = [site % shape[0], site // shape[0] % shape[1], site // (shape[0] * shape[1])]
            x, y, z = ((a - l) % n for a, l, n in zip(at, lo, shape))
            assert (np.diff(((z * 64 + y) * 64 + x) * 32 + way) > 0).all()
        return len(site)

    assert np.array_equal(lat.mask(0), ora.mask())
    n = compare()
    assert 10000 < n < 60000
    for step in range(4):
        lat.step(1)
        ora.step(1)
        g, o = lat.particle(0), ora.particle(0)
        speed = np.abs(o["U"]).max()
        assert np.abs(g["U"] - o["U"]).max() < 1e-9 * speed
        assert np.abs(g["W"] - o["W"]).max() < 1e-9 * max(np.abs(o["W"]).max(), speed / max(axes))
        assert np.array_equal(lat.mask(0), ora.mask())
        assert compare() > 0
    assert (np.asarray(lat.mask(0)) != 0).sum() > 0

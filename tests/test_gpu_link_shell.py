"""Boundary links from the shell of the solid mask, where its listing can go
wrong: windows that span an axis (no shell, every fluid node listed), windows
across the periodic edge, more nodes than one listing round and more links
than one staging round, bodies thinner than a node, two bodies in touch.
Link lists equal the oracle's (as sets, exactly), and the step that follows,
which takes its drag matrices from the links' moments, agrees to 1e-9 (the FP64
bound of the parity tests).  That bound holds for bodies of up to some 2000
links: the oracle sums full populations (w_b each) over the links, and with
N links its force is only known to about N w 2^-53 sqrt(N), 3e-12 at N = 15000,
which the largest bodies here, under loads of 1e-4, would show as 1e-7."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = {
    # shape, max_semi_axis, lattice, [(centre, axes, quaternion)]
    "whole_axes": ((13, 14, 12), 8.0, 19, [((6.2, 7.1, 5.9), (5.0, 4.0, 3.0), (0.9, 0.1, -0.3, 0.3))]),
    "one_whole_axis": ((13, 40, 42), 8.0, 19, [((6.2, 20.1, 20.9), (5.5, 3.0, 2.0), (1.0, 0.02, 0.0, 0.0))]),
    "across_the_edge": ((30, 28, 26), 8.0, 19, [((0.3, 27.6, 0.1), (6.0, 2.5, 2.5), (0.6, 0.5, -0.4, 0.2))]),
    "two_rounds": ((58, 56, 60), 25.0, 19, [((28.3, 27.2, 30.4), (25.0, 20.0, 18.0), (0.8, 0.2, 0.4, -0.1))]),
    "two_rounds_d3q27": ((52, 50, 54), 22.0, 27, [((25.3, 24.2, 26.4), (22.0, 20.0, 19.0), (0.8, 0.2, 0.4, -0.1))]),
    "sphere_27": ((58, 57, 58), 27.0, 19, [((28.3, 28.2, 28.4), (27.0, 27.0, 27.0), (1.0, 0.0, 0.0, 0.0))]),
    "thin": ((20, 22, 24), 8.0, 19, [((9.7, 10.4, 11.6), (7.0, 0.4, 0.4), (0.7, 0.1, 0.6, 0.2))]),
    "one_node": ((12, 12, 12), 8.0, 19, [((5.0, 6.0, 7.0), (0.5, 0.5, 0.5), (1.0, 0.0, 0.0, 0.0))]),
    "touching": ((40, 30, 30), 8.0, 19, [((12.2, 15.1, 14.9), (6.0, 3.0, 3.0), (0.98, 0.0, 0.1, 0.15)),
                                         ((24.6, 15.3, 15.2), (6.0, 3.0, 3.0), (0.99, 0.1, 0.0, -0.1))]),
}


@pytest.fixture(scope="module")
def lb():
    import torch
    from paper_2403_05443_amd import lbell
    lbell.load()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return lbell


@pytest.mark.parametrize("name", sorted(CASES))
def test_links_and_step(lb, orc, name):
    shape, amax, q, parts = CASES[name]
    lat = lb.Lattice([shape], collision="trt", tau=0.9, storage="fp64", max_particles=len(parts),
                     max_semi_axis=amax, lattice=q)
    ora = orc.OracleSim(shape, "trt", 0.9, **({"lattice": 27} if q == 27 else {}))
    rng = np.random.default_rng(7)
    for c, ax, quat in parts:
        quat = np.array(quat) / np.linalg.norm(quat)
        F, T = rng.normal(size=3) * 1e-4, rng.normal(size=3) * 1e-3
        i, j = lat.add_ellipsoid(c, ax, quat), ora.add_ellipsoid(c, ax, quat)
        lat.set_external(i, F, T)
        ora.set_external(j, F, T)
    assert np.array_equal(lat.mask(0), ora.mask())
    for i in range(len(parts)):
        g, o = lat.links(i), ora.links(i)
        code = lambda v: np.sort(v[0].astype(np.int64) * 32 + v[1])  # noqa: E731
        assert np.array_equal(code(g), code(o))
    if len(lat.links(0)[0]) > 2000:
        return
    lat.step(3)
    ora.step(3)
    for i in range(len(parts)):
        g, o = lat.particle(i), ora.particle(i)
        assert np.abs(g["U"] - o["U"]).max() < 1e-9 * np.abs(o["U"]).max()
        assert np.abs(g["W"] - o["W"]).max() < 1e-9 * max(np.abs(o["W"]).max(), np.abs(o["U"]).max() / max(parts[i][1]))

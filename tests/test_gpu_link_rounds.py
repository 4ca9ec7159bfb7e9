"""Link rebuild of windows of at most 512 words (a word to a thread) whose
shell holds more nodes than one listing round (1024) takes.  Link lists equal
the oracle's exactly; the step that follows agrees to 1e-7: the oracle sums
full populations over N < 14000 links, which leaves its force uncertain by
about N w 2^-53 sqrt(N) = 3e-12, 3e-8 of the loads' 1e-4."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,axes", [
    (19, (11.3, 11.1, 11.2)),
    (27, (11.3, 10.2, 10.9)),
    (19, (8.1, 7.4, 7.7)),
])
def test_listing_rounds(orc, q, axes):
    import torch
    from paper_2403_05443_amd import lbell
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    shape, c = (34, 33, 35), (16.8, 16.2, 17.4)
    lat = lbell.Lattice([shape], collision="trt", tau=0.9, storage="fp64", max_semi_axis=12.0, lattice=q)
    ora = orc.OracleSim(shape, "trt", 0.9, **({"lattice": 27} if q == 27 else {}))
    quat = np.array([0.9, 0.2, -0.3, 0.1]) / np.sqrt(0.95)
    lat.add_ellipsoid(c, axes, quat)
    ora.add_ellipsoid(c, axes, quat)
    F, T = (3e-5, -8e-5, 5e-5), (4e-4, 6e-4, -2e-4)
    lat.set_external(0, F, T)
    ora.set_external(0, F, T)
    g, o = lat.links(0), ora.links(0)
    code = lambda v: np.sort(v[0].astype(np.int64) * 32 + v[1])  # noqa: E731
    assert np.array_equal(code(g), code(o))
    nodes = len(np.unique(np.asarray(g[0])))
    assert nodes > 1024 and len(g[0]) < 14000
    lat.step(2)
    ora.step(2)
    g, o = lat.particle(0), ora.particle(0)
    assert np.abs(g["U"] - o["U"]).max() < 1e-7 * np.abs(o["U"]).max()
    assert np.abs(g["W"] - o["W"]).max() < 1e-7 * np.abs(o["U"]).max() / max(axes)

"""A box alone in its context (its description comes with the launch) against
the same box beside another: the same bits, through plain steps, graph replays
and a change of the external load between the replays of one captured graph (the
counter-force must not be frozen in it)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(shapes, storage, lattice, graph, collision, variant, monkeypatch):
    from paper_2403_05443_amd import Lattice
    if variant is not None:
        monkeypatch.setenv("LBELL_K1_VARIANT", variant)
    lat = Lattice(shapes, collision=collision, tau=0.8, storage=storage, lattice=lattice, counterforce=True,
                  max_particles=2)
    for b, n in enumerate(shapes):
        lat.add_ellipsoid([v / 2 + 0.2 for v in n], (5.0, 2.5, 2.0), (0.8, 0.36, 0.48, 0.0), box=b)
        lat.set_external(b, (2e-4, -1e-4, 3e-4), (1e-3, 0, -1e-3))
    lat.set_graph(graph)
    out = []
    for load in (1.0, -2.0, 0.5):
        lat.set_external(0, (load * 2e-4, 1e-4, 0.0), (0, load * 1e-3, 0))
        lat.step(4)
        out += [lat.momentum(0), *lat.force_torque(0), *lat.particle(0).values(), *lat.fields(0)]
    lat.close()
    return out


@pytest.mark.parametrize("storage,lattice,graph,collision,variant", [
    ("fp64", 19, 0, "bgk", None), ("fp32", 19, 2, "reg", None), ("fp16", 19, 4, "trt", None),
    ("fp32", 27, 2, "trt", "12"), ("bf16", 19, 2, "trt", "12"), ("fp64", 27, 1, "bgk", None)])
def test_one_box_equals_one_of_two(monkeypatch, storage, lattice, graph, collision, variant):
    a = _run([(23, 19, 21)], storage, lattice, graph, collision, variant, monkeypatch)
    b = _run([(23, 19, 21), (17, 18, 16)], storage, lattice, graph, collision, variant, monkeypatch)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)

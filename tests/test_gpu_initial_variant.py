"""The collide-stream variant a context starts with: every choice gives the
bits of the plain two-buffer kernel (variant 0), on either side of the lines of
the rule and from the first field on (an in-place context is initialised
straight into its one buffer)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# shape, storage, lattice, walls; populations of one buffer in MB (the rule's lines: 128, then 200 or 400)
CASES = [((30, 25, 21), "fp64", 19, False),     # 2
         ((118, 118, 118), "fp32", 19, False),  # 125: two buffers just fit
         ((120, 120, 120), "fp32", 19, False),  # 131: one does
         ((121, 119, 118), "fp32", 19, True),   # 129, between moving walls
         ((172, 173, 174), "fp16", 19, False),  # 197: one, half format
         ((174, 174, 175), "bf16", 19, False),  # 201: neither
         ((156, 155, 153), "fp32", 27, False),  # 400
         ((157, 155, 153), "fp32", 27, False)]  # 402


@pytest.mark.parametrize("shape,storage,lattice,walls", CASES)
def test_default_equals_plain(monkeypatch, shape, storage, lattice, walls):
    from paper_2403_05443_amd import Lattice, make_box
    seen = []
    for variant in (None, "0"):
        if variant is None:
            monkeypatch.delenv("LBELL_K1_VARIANT", raising=False)
        else:
            monkeypatch.setenv("LBELL_K1_VARIANT", variant)
        box = make_box(*shape, walls=walls, wall_lo=(-0.01, 0, 0), wall_hi=(0.01, 0, 0),
                       init="couette" if walls else "rest")
        lat = Lattice([box], collision="trt", tau=0.8, storage=storage, velocity_scale=0.01, lattice=lattice)
        lat.add_ellipsoid([n / 2 + 0.3 for n in shape], (6.0, 3.0, 2.5), (0.8, 0.36, 0.48, 0.0))
        lat.set_external(0, (2e-4, -1e-4, 3e-4), (1e-3, 0, -1e-3))
        out = [lat.momentum(0)]
        for n in (1, 2):
            lat.step(n)
            out += [lat.momentum(0), *lat.force_torque(0), lat.particle(0)["U"], lat.particle(0)["W"]]
        if lat.shapes[0][0] <= 121:
            out += list(lat.fields(0))
        seen.append(out)
        lat.close()
        del lat
    for a, b in zip(*seen):
        assert np.array_equal(a, b)

"""The variant a context starts with, where the rule's lines lie: whether it is
an in-place one (a checkpoint says so), and the same bits as a kernel of the
other layout."""
import struct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# shape, storage, lattice, walls, in place, the variant to compare with; MB of one buffer
CASES = [((119, 119, 118), "fp32", 19, False, False, "12"),   # 127
         ((121, 120, 118), "fp32", 19, False, True, "15"),    # 130
         ((162, 163, 164), "fp32", 19, False, True, "15"),    # 329.1, below 330
         ((164, 163, 163), "fp32", 19, False, False, "12"),   # 331.2
         ((172, 173, 174), "fp16", 19, False, True, "3"),     # 197
         ((174, 174, 175), "bf16", 19, False, False, "12"),   # 201
         ((144, 145, 146), "fp32", 27, False, True, "3"),     # 329.2
         ((157, 155, 153), "fp32", 27, False, False, "12"),   # 402
         ((152, 151, 153), "fp16", 19, True, False, "12"),    # 133, half format between walls
         ((153, 154, 156), "fp16", 19, True, True, "3"),      # 140
         ((128, 96, 96), "bf16", 19, True, False, "12"),      # rows of 128 sites between walls
         ((64, 20, 20), "fp16", 19, True, False, "12")]


@pytest.mark.parametrize("shape,storage,lattice,walls,in_place,other", CASES)
def test_layout_and_bits(monkeypatch, tmp_path, shape, storage, lattice, walls, in_place, other):
    from paper_2403_05443_amd import Lattice, make_box
    seen = []
    for variant in (None, other):
        if variant is None:
            monkeypatch.delenv("LBELL_K1_VARIANT", raising=False)
        else:
            monkeypatch.setenv("LBELL_K1_VARIANT", variant)
        box = make_box(*shape, walls=walls, wall_lo=(-0.01, 0, 0), wall_hi=(0.01, 0, 0),
                       init="couette" if walls else "rest")
        lat = Lattice([box], collision="trt", tau=0.8, storage=storage, velocity_scale=0.01, lattice=lattice)
        lat.add_ellipsoid([n / 2 + 0.3 for n in shape], (6.0, 3.0, 2.5), (0.8, 0.36, 0.48, 0.0))
        lat.set_external(0, (2e-4, -1e-4, 3e-4), (1e-3, 0, -1e-3))
        if variant is None:
            lat.save(tmp_path / "ck")
            with open(tmp_path / "ck", "rb") as f:  # magic, version, nboxes, storage, np, cur, in place
                head = struct.unpack("8s6i", f.read(32))
            assert head[0] == b"LBELLCK1" and head[6] == int(in_place)
            (tmp_path / "ck").unlink()
        out = []
        for n in (1, 2):
            lat.step(n)
            out += [lat.momentum(0), *lat.force_torque(0), lat.particle(0)["U"], lat.particle(0)["W"]]
        out += list(lat.fields(0))
        seen.append(out)
        lat.close()
        del lat
    for a, b in zip(*seen):
        assert np.array_equal(a, b)

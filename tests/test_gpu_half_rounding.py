"""FP64 values stored to FP16 populations round to the nearest half, ties to
even, through every range of the format: checked bit for bit against numpy's
conversion, which rounds the double once.

The density of a lone population v in a box at rest is rho0 + v; the stored
values are spaced by at least 2^-24 / 1024 = 6e-11, so the rounding of the sum
(1e-16, 1e-14 from 64 up) leaves no doubt which half was stored."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SCALE = 1024.0  # 2^floor(log2(0.25 / (1e-3 / 6))), the scale of velocity_scale 1e-3


def _values():
    h = np.array([0x0001, 0x0002, 0x0003, 0x01ff, 0x03ff, 0x0400, 0x0401, 0x3bff, 0x3c00, 0x3c01, 0x57ff, 0x7bfe],
                 np.uint16)
    lo, hi = h.view(np.float16).astype(np.float64), (h + np.uint16(1)).view(np.float16).astype(np.float64)
    mid = 0.5 * (lo + hi)
    tiny = np.array([2.0 ** -25, np.nextafter(2.0 ** -25, 1), np.nextafter(2.0 ** -25, 0), 1e-30, 1e-45, 1e-300])
    near = [mid * (1 + k * 2.0 ** -p) for k in (-1, 1) for p in (52, 30, 25, 24, 23)]
    r = np.random.default_rng(4)
    rand = np.ldexp(r.uniform(1, 2, 60), r.integers(-27, 15, 60))
    v = np.concatenate([lo, hi, mid, tiny, rand] + near)
    return np.concatenate([v, -v])


def test_nearest_half():
    import torch
    from paper_2403_05443_amd import lbell
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    v = _values()
    lat = lbell.Lattice([(24, 24, 24)], collision="trt", tau=1.0, storage="fp16")
    lat.add_ellipsoid((0.4, 0.3, 0.2), (1.0, 1.0, 1.0), (1.0, 0.0, 0.0, 0.0))
    sites = [x + 24 * (y + 24 * z) for z in range(6, 18) for y in range(4, 20) for x in range(4, 20)][:len(v)]
    for k, s in enumerate(sites):
        lat.poke(0, s, k % 19, v[k] / SCALE)
    rho = np.asarray(lat.fields(0)[0]).reshape(-1)
    want = 1.0 + v.astype(np.float16).astype(np.float64) / SCALE
    assert np.array_equal(rho[sites], want)

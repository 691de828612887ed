"""Distance raster and edge lists of aperture polygons, made on the GPU.

Full physics: a square whose sides are split at binary fractions of their length
is the same opening, and every edge's ray arithmetic scales by a power of two,
so the doses of 4, 64, 256 and 1024 vertices are equal bit for bit (fewer, as
many and more vertices than a wavefront has lanes; splits add edges to every
list).  Straight mode: polygons with few vertices, with one more than a
wavefront, and a concave one against the oracle."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I
from test_gpu_parity import eng, gpu_q, straight_check  # noqa: F401

pytestmark = pytest.mark.gpu


def square(n):
    """16 mm square with n vertices (a multiple of 4, powers of two per side)"""
    c = np.array([(-8.0, -8.0), (8.0, -8.0), (8.0, 8.0), (-8.0, 8.0)])
    m = n // 4
    return np.concatenate([c[i] + (c[(i + 1) % 4] - c[i]) * (np.arange(m) / m)[:, None] for i in range(4)]).astype(np.float32)


def with_polygon(poly, physics, hist=60_000):
    c = I.config2(20.0, True, histories_per_case=hist, physics=physics, shape=(64, 64, 150))
    c.fields[0].polygon = np.ascontiguousarray(poly, np.float32)
    return c


def test_split_sides_same_bits(eng):  # noqa: F811
    want = gpu_q(eng, with_polygon(square(4), I.PHYS_ALL), k=34)
    for n in (64, 256, 1024):
        got = gpu_q(eng, with_polygon(square(n), I.PHYS_ALL), k=34)
        np.testing.assert_array_equal(got[0], want[0])
        np.testing.assert_array_equal(got[4], want[4])


def star(n=5, r0=10.0, r1=4.0):
    t = np.pi * np.arange(2 * n) / n + 0.1
    r = np.where(np.arange(2 * n) % 2 == 0, r0, r1)
    return np.stack([r * np.cos(t), r * np.sin(t)], 1)


@pytest.mark.parametrize("poly", [np.array([(-9.0, -7.0), (11.0, -3.0), (1.0, 10.0)]), star(),
                                  I.circle_polygon(19.0, 65)[::-1]], ids=["triangle", "star", "65-gon reversed"])
def test_straight_parity_polygons(eng, orc, poly):  # noqa: F811
    c = with_polygon(poly, 0, hist=30_000)
    qg, kg, _, _, _ = gpu_q(eng, c)
    qo, _, ko = orc.run_tally(c)
    straight_check(orc, c, qg, kg, qo, ko)

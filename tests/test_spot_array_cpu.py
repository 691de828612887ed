"""The spots handed to the library: every field of every spot as the conversion
of that one value, for the dtypes, strides and values a caller may have."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I
from paper_2307_01416_amd import vpmc as V

FIELDS = ("x_mm", "y_mm", "energy_mev", "sigma_mm", "energy_sigma_mev", "weight")


def by_hand(spots):
    arr = (V.vpmc_spot * max(1, len(spots)))()
    for i in range(len(spots)):
        for f in FIELDS:
            setattr(arr[i], f, float(spots[f][i]))
        arr[i].n_histories = int(spots["n_histories"][i])
    return bytes(arr)


@pytest.mark.parametrize("n", [0, 1, 7, 950])
@pytest.mark.parametrize("hist", [np.uint32, np.int64, np.float64])
def test_spot_array(n, hist):
    rng = np.random.default_rng(n)
    base = I.make_spots(rng.normal(size=(2 * n, 2)) * 1e3, 150.0, 3.0, 10)
    dt = [(f, np.float64) for f in FIELDS] + [("n_histories", hist)]
    spots = np.zeros(2 * n, dt)
    for f in FIELDS:
        spots[f] = base[f] + rng.normal(size=2 * n)
    spots["n_histories"] = rng.integers(0, 1 << 31, 2 * n)
    if n > 1:
        spots["x_mm"][2], spots["weight"][0], spots["y_mm"][0] = 1e300, np.nan, -0.0
        if hist is np.int64:
            spots["n_histories"][0], spots["n_histories"][2] = -1, (1 << 32) + 5
    for s in (spots, spots[::2], spots[::-1]):
        assert bytes(V.spot_array(s)) == by_hand(s)
    assert bytes(V.spot_array(base)) == by_hand(base)

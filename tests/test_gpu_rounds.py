"""Staged influence-matrix transport at the sizes where it can go wrong,
against the dense run of the same spots (integer tallies: equality, no
tolerance): staging buffers of one refill of a single workgroup (an epoch in
many rounds, rows split between them), rows without histories and of a lane
more or less than a wavefull, and fixed-point exponents at which a deposit
overflows the 32-bit entries of the row tile (carries and high halves)."""
import ctypes as C

import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    e = V.Engine(0)
    yield e
    e.close()


def case(hists, physics, divergent=False):
    c = I.config2(20.0, True, shape=(60, 60, 120), physics=physics, seed=11)
    f = c.fields[0]
    f.spots = f.spots[: len(hists)].copy()
    f.spots["n_histories"] = np.asarray(hists, np.uint32)
    if divergent:
        f.vsad_mm = 2000.0
        f.block.focus_mm = 2000.0
    c.scenarios = [I.Scenario(), I.Scenario((2.0, -1.0, 0.0), 1.035)]
    return c


def rows(eng, c, k, max_bytes=0, blocks=0, threads=0, hpl=0):
    from paper_2307_01416_amd import vpmc as V
    eng.load_case(c)
    spots = c.fields[0].spots
    n_rows = len(spots) * len(c.scenarios)
    rp = np.zeros(n_rows + 1, np.int64)
    o = V.make_opts(seed=c.seed, physics=c.physics, output=V.OUT_CSR, fixed_point_bits=k, max_device_bytes=max_bytes,
                    grid_blocks=blocks, block_threads=threads, hist_per_lane=hpl)
    led = np.zeros((len(c.scenarios), V.NLEDGER))
    V.vpmc_run_batched(eng.ctx, [0], [V.spot_array(spots)], V.scenario_array(c.scenarios), len(c.scenarios), o, None,
                       led, rp)
    col, q = np.zeros(rp[-1], np.int32), np.zeros(rp[-1], np.int64)
    V.vpmc_copy_csr(eng.ctx, col, None, q)
    return rp, col, q, led


HISTS = [0, 1, 63, 64, 65, 0, 700, 2049, 128]


@pytest.mark.parametrize("physics,divergent", [(I.PHYS_ALL, False), (0, False), (I.PHYS_ALL, True), (I.MCS, False)])
def test_rounds_equal_dense(eng, physics, divergent):
    from paper_2307_01416_amd import vpmc as V
    c = case(HISTS, physics, divergent)
    whole = rows(eng, c, 36)
    # one refill of one workgroup of four waves: 256 records per round
    capped = V.Engine(0)
    try:
        few = rows(capped, c, 36, max_bytes=1 << 31, blocks=1, threads=256, hpl=1)
    finally:
        capped.close()
    for a, b in zip(whole, few):
        np.testing.assert_array_equal(a, b)
    n = len(HISTS)
    eng.run_dose(c, 0, n_batches=0, sigma=False, fixed_point_bits=36)
    for s in range(2):
        q, _ = eng.last_tally(s)
        dense = np.zeros(c.geometry.nvox, np.int64)
        b, e = whole[0][s * n], whole[0][(s + 1) * n]
        np.add.at(dense, whole[1][b:e], whole[2][b:e])
        np.testing.assert_array_equal(q.cpu().numpy().ravel(), dense)


@pytest.mark.parametrize("k", [20, 44, 50])
def test_tile_carries(eng, k):
    c = case([3000, 500, 8], I.PHYS_ALL)
    c.scenarios = c.scenarios[:1]
    rp, col, q, _ = rows(eng, c, k)
    if k >= 44:
        assert q.max() > 1 << 33   # entries overflow 32 bits
    eng.run_dose(c, 0, n_batches=0, sigma=False, fixed_point_bits=k)
    want, _ = eng.last_tally(0)
    dense = np.zeros(c.geometry.nvox, np.int64)
    np.add.at(dense, col, q)
    np.testing.assert_array_equal(want.cpu().numpy().ravel(), dense)

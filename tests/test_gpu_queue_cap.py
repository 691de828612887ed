"""Iterations that queue_cap counts: a draw of the default size costs a quarter
of one, so a wavefront's share of a row in chunks of 256 histories fits in a cap
that counts those (131 072 histories over the four waves of one workgroup: 128
chunks a wave; a cap of 300 leaves room for uneven shares, row picks and waits,
and not for the 512 draws a wave)."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics", [I.PHYS_ALL, 0])
def test_cap_of_chunks(physics):
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    c = I.config1(n_histories=1 << 17, physics=physics)
    e = V.Engine(0)
    try:
        shape = dict(fixed_point_bits=34, grid_blocks=1, block_threads=256)
        want = e.run_csr(c, **shape)
        got = e.run_csr(c, queue_cap=300, **shape)
        for a, b in zip(want[:4], got[:4]):
            np.testing.assert_array_equal(a, b)
        with pytest.raises(V.VpmcError) as ei:   # below the chunks of a wave
            e.run_csr(c, queue_cap=60, **shape)
        assert ei.value.code == V.E_ABORTED
        with pytest.raises(V.VpmcError) as ei:   # draws of one wavefull asked for: one iteration each
            e.run_csr(c, queue_cap=300, hist_per_lane=1, **shape)
        assert ei.value.code == V.E_ABORTED
    finally:
        e.close()

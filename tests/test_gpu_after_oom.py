"""A dense run whose tallies exceed the device's memory is VPMC_E_OOM, and the
same context's next run gives a fresh context's bits."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_next_run_after_a_refused_one():
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    c = I.config1(n_histories=5_000)
    big = I.config1(n_histories=10)
    big.geometry = I.water_geometry((1000, 1000, 1000), (1.0, 1.0, 1.0))
    big.scenarios = [I.Scenario()] * 64   # 64 tallies of 8 GB
    assert 64 * 8e9 > torch.cuda.get_device_properties(0).total_memory
    spots = big.fields[0].spots
    used, fresh = V.Engine(0), V.Engine(0)
    try:
        used.load_case(big)
        with pytest.raises(V.VpmcError) as ei:
            V.vpmc_run_spots(used.ctx, 0, V.spot_array(spots), len(spots), V.scenario_array(big.scenarios), 64,
                             V.make_opts(fixed_point_bits=34, flags=V.DEVICE_PTRS), None, None, np.zeros((64, V.NLEDGER)))
        assert ei.value.code == V.E_OOM
        out = []
        for e in (used, fresh):
            e.load_case(c)
            dose, sig, led = e.run_dose(c, 0, n_batches=4, fixed_point_bits=34)
            out.append((dose.cpu().numpy(), sig.cpu().numpy(), led))
        assert out[0][0].max() > 0
        for a, b in zip(*out):
            np.testing.assert_array_equal(a, b)
    finally:
        used.close()
        fresh.close()

"""Influence-matrix rows handed to device arrays: every choice of outputs, entry
counts with each remainder of four, outputs aligned to 16 bytes or not, equal
the copies to host arrays bit for bit and write nothing past their end."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["water", "head"])
def test_device_outputs(kind):
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    c = I.config2(20.0, False, shape=(40, 40, 60))
    if kind == "head":
        c.geometry = I.head_ct(0, shape=(40, 40, 60), spacing=(4.0, 4.0, 3.0))
    few = c.fields[0].spots[:3].copy()
    scen = V.scenario_array(c.scenarios)
    eng = V.Engine(0)
    try:
        eng.load_case(c)
        seen = set()
        for hist in range(1, 40):
            few["n_histories"] = hist
            rp = np.zeros(4, np.int64)
            a = (eng.ctx, 0, V.spot_array(few), 3, scen, 1)
            V.vpmc_run_spots(*a, V.make_opts(seed=hist, output=V.OUT_CSR, fixed_point_bits=34), None, None, None, rp)
            n = int(rp[-1])
            if n % 4 in seen or n == 0:
                continue
            seen.add(n % 4)
            want = np.zeros(n, np.int32), np.zeros(n, np.float32), np.zeros(n, np.int64)
            V.vpmc_copy_csr(eng.ctx, *want)
            rpd = torch.zeros(4, dtype=torch.int64, device="cuda")
            V.vpmc_run_spots(*a, V.make_opts(seed=hist, output=V.OUT_CSR, fixed_point_bits=34, flags=V.DEVICE_PTRS),
                             None, None, None, rpd)
            assert int(rpd[-1]) == n
            for off in (0, 1, 2):
                for pick in (7, 1, 2, 4, 5, 6):
                    full = [torch.full((n + off + 5,), -77, dtype=d, device="cuda")
                            for d in (torch.int32, torch.float32, torch.int64)]
                    out = [f[off:off + n] if pick >> j & 1 else None for j, f in enumerate(full)]
                    V.vpmc_copy_csr(eng.ctx, *out)
                    for j, (f, w) in enumerate(zip(full, want)):
                        got = f.cpu().numpy()
                        if pick >> j & 1:
                            np.testing.assert_array_equal(got[off:off + n], w)
                            assert np.all(got[:off] == -77) and np.all(got[off + n:] == -77)
                        else:
                            assert np.all(got == -77)
        assert seen == {0, 1, 2, 3}
    finally:
        eng.close()

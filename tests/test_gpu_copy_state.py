"""Rows copied out after something else has happened on the context: another
grid loaded (columns and energies as before, values refused), the run's own
grid again, a dense run of another fixed-point exponent (everything as before)."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture()
def run():
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    c = I.config2(20.0, False, shape=(40, 40, 60))
    c.geometry = I.head_ct(0, shape=(40, 40, 60), spacing=(4.0, 4.0, 3.0))
    c.fields[0].spots = c.fields[0].spots[:3].copy()
    c.fields[0].spots["n_histories"] = 500
    e = V.Engine(0)
    rp, col, val, q, k = e.run_csr(c, fixed_point_bits=34)
    assert rp[-1] > 0
    yield V, e, c, (col, val, q)
    e.close()


def copy(V, e, n, val=True):
    out = np.zeros(n, np.int32), np.zeros(n, np.float32) if val else None, np.zeros(n, np.int64)
    V.vpmc_copy_csr(e.ctx, *out)
    return out


def test_another_grid(run):
    V, e, c, want = run
    n = len(want[0])
    V.vpmc_load_geometry(e.ctx, I.head_ct(0, shape=(8, 8, 8), spacing=(4.0, 4.0, 3.0)))
    with pytest.raises(V.VpmcError) as ei:
        copy(V, e, n)
    assert ei.value.code == V.E_STATE
    col, _, q = copy(V, e, n, val=False)
    np.testing.assert_array_equal(col, want[0])
    np.testing.assert_array_equal(q, want[2])
    V.vpmc_load_geometry(e.ctx, c.geometry)
    for a, b in zip(copy(V, e, n), want):
        np.testing.assert_array_equal(a, b)


def test_dense_run_of_another_exponent(run):
    V, e, c, want = run
    e.run_dose(c, 0, n_batches=0, sigma=False, fixed_point_bits=30)
    for a, b in zip(copy(V, e, len(want[0])), want):
        np.testing.assert_array_equal(a, b)

"""Dense runs with LET through the work queue: a voxel's dose and LET numerator
lie side by side and are added by pairs of lanes.  Integer tallies, so doses,
standard errors, tallies, LET numerators and ledgers equal those of the run
with a cap on device memory (one atomic per deposit) bit for bit: one batch,
several, more than fit at once; a few workgroups of few waves; a field whose
particles mostly miss any tile box."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I
from test_gpu_dense_queue import HISTS, case, eng, run, same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batches,hists,shape", [(0, HISTS, (60, 50, 110)), (1, [1], (40, 40, 40)),
                                                 (5, [64, 33, 31], (61, 47, 33)), (0, [40_000] * 9, (90, 90, 110)),
                                                 (600, [3000, 17], (100, 100, 110))])
def test_equals_capped_run(eng, batches, hists, shape):  # noqa: F811
    from paper_2307_01416_amd import vpmc as V
    c = case(hists, I.PHYS_ALL, shape=shape)
    if batches == 600:
        c.scenarios = c.scenarios[:1]
    other = V.Engine(0)
    try:
        want = run(other, c, batches, "run", let=True, max_bytes=1 << 30)
    finally:
        other.close()
    same(run(eng, c, batches, "run", let=True), want)
    same(run(eng, c, batches, "run", let=True, blocks=3, threads=256), want)
    plain = run(eng, c, batches, "run")                 # grids without LET, in the same memory
    same(plain[:2], want[:2])

"""Dense runs of one tally grid on either side of the sizes up to which they go
batch by batch (49 152 histories of an open field, 163 840 behind a block, 196 608
without processes; with a launch shape that is asked for, any go through the
queue): the allocation-free run's doses and ledgers, bit for bit, with LET those
of a run under a cap."""
import pytest

from paper_2307_01416_amd import inputs as I
from test_gpu_dense_queue import case, eng, run, same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics,block,most", [(I.PHYS_ALL, False, 49_152), (0, False, 49_152), (I.PHYS_ALL, True, 163_840),
                                                (I.MCS, True, 163_840), (0, True, 196_608)])
@pytest.mark.parametrize("rs", [False, True])
@pytest.mark.parametrize("n", ["one", "few", "most", "most + 1"])
def test_either_route(eng, physics, block, most, rs, n):  # noqa: F811
    from paper_2307_01416_amd import vpmc as V
    hists = {"one": [1], "few": [0, 63, 64, 65, 700], "most": [most - 5000, 0, 5000], "most + 1": [5000, most - 4999]}[n]
    c = case(hists, physics, shape=(40, 40, 60), rs=rs)
    if not block:
        c.fields[0].block = c.fields[0].polygon = None
    c.scenarios = c.scenarios[1:]
    want = run(eng, c, 0, "noalloc")
    same(run(eng, c, 0, "run")[:3], want[:3])
    same(run(eng, c, 0, "run", blocks=64, threads=512)[:3], want[:3])
    other = V.Engine(0)
    try:
        with_let = run(other, c, 0, "run", let=True, max_bytes=1 << 30)
    finally:
        other.close()
    same(run(eng, c, 0, "run", let=True), with_let)
    same(run(eng, c, 0, "run", let=True, blocks=64, threads=512), with_let)

"""Dense runs through the work queue against the batch-by-batch run of the same
arguments (the allocation-free entry, and a run with a cap on device memory,
both one history per lane at a time): integer tallies, so doses, standard
errors, LET numerators and ledgers are equal bit for bit.  Ragged history
counts, empty and missing spots, several scenarios, partial processes, a
divergent block, batch tallies that do not fit at once, and more histories than
one round stages."""
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


def run(eng, c, batches, entry, let=False, max_bytes=0, blocks=0, threads=0):
    """(dose, sigma, ledger, tallies, LET numerators) as numpy arrays"""
    import torch
    from paper_2307_01416_amd import vpmc as V
    eng.load_case(c)
    n, S = c.geometry.nvox, len(c.scenarios)
    dose = torch.empty((S, n), dtype=torch.float32, device="cuda")
    sig = torch.empty_like(dose) if batches >= 2 else None
    led = np.zeros((S, V.NLEDGER))
    spots = c.fields[0].spots
    o = V.make_opts(seed=c.seed, physics=c.physics, n_batches=batches, fixed_point_bits=34,
                    flags=V.DEVICE_PTRS | (V.LET if let else 0), max_device_bytes=max_bytes, grid_blocks=blocks,
                    block_threads=threads)
    a = (eng.ctx, 0, V.spot_array(spots), len(spots), V.scenario_array(c.scenarios), S, o, dose, sig, led)
    (V.vpmc_run_spots if entry == "run" else V.vpmc_run_spots_noalloc)(*a)
    torch.cuda.synchronize()
    out = [dose.cpu().numpy(), None if sig is None else sig.cpu().numpy(), led]
    if entry == "run":
        out += [[eng.last_tally(s)[0].cpu().numpy() for s in range(S)],
                [eng.last_let(s)[0].cpu().numpy() for s in range(S)] if let else None]
    return out


def same(a, b):
    for x, y in zip(a, b):
        if x is None or y is None:
            assert x is None and y is None
        else:
            np.testing.assert_array_equal(np.asarray(x), np.asarray(y))


def case(hists, physics, shape=(60, 50, 110), divergent=False, rs=True):
    c = I.config2(20.0, rs, shape=shape, physics=physics, seed=5)
    f = c.fields[0]
    f.spots = f.spots[: len(hists)].copy()
    f.spots["n_histories"] = np.asarray(hists, np.uint32)
    f.spots["energy_mev"][::2] -= 20.0
    if divergent:
        f.vsad_mm = 2000.0
        f.block.focus_mm = 2000.0
    c.scenarios = [I.Scenario(), I.Scenario((2.0, -1.0, 0.0), 1.035)]
    return c


HISTS = [0, 1, 63, 64, 65, 0, 700, 2049, 128, 5000]


@pytest.mark.parametrize("physics,batches,divergent", [(I.PHYS_ALL, 0, False), (I.PHYS_ALL, 16, False), (0, 3, False),
                                                       (I.PHYS_ALL, 7, True), (I.MCS | I.STRAGGLE, 2, False)])
def test_equals_batch_by_batch(eng, physics, batches, divergent):
    c = case(HISTS, physics, divergent=divergent)
    a, b = run(eng, c, batches, "run"), run(eng, c, batches, "noalloc")
    same(a[:3], b[:3])
    same(run(eng, c, batches, "run", blocks=3, threads=256)[:3], b[:3])   # few workgroups of few waves


@pytest.mark.parametrize("physics", [I.PHYS_ALL, 0])
def test_let_equals_capped_run(eng, physics):
    from paper_2307_01416_amd import vpmc as V
    c = case(HISTS, physics)
    other = V.Engine(0)
    try:
        same(run(eng, c, 4, "run", let=True), run(other, c, 4, "run", let=True, max_bytes=1 << 30))
    finally:
        other.close()


def test_batch_tallies_in_parts(eng):
    # 1024 batch tallies of 1.1e6 voxels exceed what is kept at once
    c = case([3000, 17, 1500], I.PHYS_ALL, shape=(100, 100, 110))
    c.scenarios = c.scenarios[:1]
    same(run(eng, c, 1024, "run")[:3], run(eng, c, 1024, "noalloc")[:3])
    same(run(eng, c, 16, "run")[:3], run(eng, c, 16, "noalloc")[:3])   # the tallies were left clear


def test_more_histories_than_a_round_stages(eng):
    c = case([36_000_000], I.PHYS_ALL, shape=(40, 40, 40), rs=False)
    c.scenarios = c.scenarios[:1]
    same(run(eng, c, 0, "run")[:3], run(eng, c, 0, "noalloc")[:3])


def test_no_histories(eng):
    c = case([0, 0], I.PHYS_ALL)
    a = run(eng, c, 4, "run")
    assert not a[0].any() and not a[1].any() and not a[2].any()

"""Cell merge of device arrays: the map is checked and the rows are cut and
summed on the GPU.  Rows of 0, 1, 63..65, 4095..4097 (a wavefront's share) and
all voxels, starting at a nonzero row_ptr[0], cells of 1 to 9000 voxels:
offsets, cells and int64 sums equal numpy's bit for bit, values equal the host
arrays' call bit for bit.  A bad map or row_ptr is E_ARG as from host arrays."""
import numpy as np
import pytest

from paper_2307_01416_amd import inputs as I

pytestmark = pytest.mark.gpu
SHAPE, K = (33, 31, 17), 30
NVOX = SHAPE[0] * SHAPE[1] * SHAPE[2]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_2307_01416_amd import vpmc as V
    g = I.head_ct(3, shape=SHAPE, spacing=(2.0, 2.0, 2.0))
    c = V.vpmc_create(0)
    V.vpmc_load_geometry(c, g)
    yield V, c
    V.vpmc_destroy(c)


def dev(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def rows(seed=0):
    rng = np.random.default_rng(seed)
    lens = [0, 1, 0, 63, 64, 65, 4095, 4096, 4097, 8191, 8193, NVOX, 1000, 0]
    cols = [np.sort(rng.choice(NVOX, n, replace=False)) for n in lens]
    first = 5   # entries before the first row are not part of the call
    col = np.concatenate([np.zeros(first, np.int64)] + cols).astype(np.int32)
    rp = (first + np.concatenate([[0], np.cumsum(lens)])).astype(np.int64)
    return rp, col, rng.integers(-(1 << 40), 1 << 40, len(col)).astype(np.int64)


def cell_map(width):
    rng = np.random.default_rng(width)
    step = np.zeros(NVOX, bool)
    v = 0
    while True:
        v += width if width in (1, 9000) else int(rng.integers(1, width + 1))
        if v >= NVOX:
            break
        step[v] = True
    m = np.cumsum(step).astype(np.int32)
    return m, int(m[-1]) + 1


@pytest.mark.parametrize("width", [1, 2, 4, 7, 64, 130, 9000])
def test_device_rows(ctx, width):
    V, c = ctx
    rp, col, q = rows()
    cmap, n = cell_map(width)
    got = [t.cpu().numpy() for t in V.vpmc_csr_cells(c, *dev(rp, col, q), K, *dev(cmap), n, V.DEVICE_PTRS)]
    host = V.vpmc_csr_cells(c, rp, col, q, K, cmap, n)
    off, cells, sums = [0], [], []
    for r in range(len(rp) - 1):
        u, inv = np.unique(cmap[col[rp[r]:rp[r + 1]]], return_inverse=True)
        s = np.zeros(len(u), np.int64)
        np.add.at(s, inv, q[rp[r]:rp[r + 1]])
        cells.append(u), sums.append(s), off.append(off[-1] + len(u))
    np.testing.assert_array_equal(got[0], off)
    np.testing.assert_array_equal(got[1], np.concatenate(cells))
    np.testing.assert_array_equal(got[2], np.concatenate(sums))
    for a, b in zip(got, host):
        np.testing.assert_array_equal(a, b)


def test_device_checks(ctx):
    V, c = ctx
    rp, col, q = rows()
    good, n = cell_map(4)

    def code(m=good, n_cells=n, rp_=rp):
        try:
            V.vpmc_csr_cells(c, *dev(rp_, col, q), K, *dev(m), n_cells, V.DEVICE_PTRS)
        except V.VpmcError as e:
            return e.code
        return 0

    assert code() == 0
    for v in (0, 1, NVOX // 2, NVOX - 2, NVOX - 1):
        for d in (-1, 2, -(1 << 31), (1 << 31) - 1):
            m = good.copy()
            m[v] = d if abs(d) > 2 else m[v] + d   # two steps up, one down, the type's ends
            if np.all(np.isin(np.diff(m.astype(np.int64)), (0, 1))) and m[0] == 0 and m[-1] == n - 1:
                continue
            assert code(m) == V.E_ARG, (v, d)
    assert code(n_cells=n + 1) == V.E_ARG and code(n_cells=n - 1) == V.E_ARG
    assert code(n_cells=NVOX + 1) == V.E_ARG
    down = rp.copy()
    down[5] = rp[4] - 1
    assert code(rp_=down) == V.E_ARG
    neg = rp.copy()
    neg[0] = -1
    assert code(rp_=neg) == V.E_ARG
    assert code() == 0

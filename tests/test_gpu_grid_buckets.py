"""The row pass and the leaf pass of the grid build (65 536 rows and more): pieces of every size, runs of one row and of a
whole piece, records of one word and of two side by side, rows outside all grids.  The set of voxels of every grid against
torch's distinct rows, and the indices of all rows against the position of their voxel."""
import numpy as np
import pytest
import torch

import paper_2407_01781_amd as fx

pytestmark = pytest.mark.gpu


def _check(g, rows, joffsets):
    jidx = torch.full((rows.shape[0],), -1, dtype=torch.int32, device="cuda")
    for b, (lo, hi) in enumerate(joffsets):
        jidx[lo:hi] = b
    inside = jidx >= 0
    out, ob = g.ijk()
    want = torch.cat([jidx[inside][:, None], rows[inside]], dim=1)
    both = torch.cat([torch.cat([ob[:, None], out], dim=1), want]).long()
    m = both.min(dim=0).values
    width = (both.max(dim=0).values - m + 1).tolist()
    key = ((both[:, 0] - m[0]) * width[1] + both[:, 1] - m[1]) * width[2] + both[:, 2] - m[2]
    assert width[0] * width[1] * width[2] * width[3] < 2 ** 63
    key = key * width[3] + both[:, 3] - m[3]
    have, ref = key[: out.shape[0]].sort().values, torch.unique(key[out.shape[0]:])
    assert torch.equal(have, ref)
    idx = g.ijk_to_index(rows[inside].contiguous(), jidx[inside].contiguous())
    assert torch.equal(out[idx.long()], rows[inside]) and torch.equal(ob[idx.long()], jidx[inside])


def _rows(n, side, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-side, side, (n, 3), generator=gen, device="cuda", dtype=torch.int32)


@pytest.mark.parametrize("n,side", [(65_536, 20), (69_633, 300), (300_000, 60), (1_048_577, 200), (4_200_001, 150), (8_390_000, 300), (17_000_000, 120)])
def test_piece_sizes(n, side):
    rows = _rows(n, side, n)
    joff = np.array([[0, n]])
    _check(fx.build_index_grid(rows, joff), rows, joff)


@pytest.mark.parametrize("n", [100_000, 1_000_000, 9_000_000])
def test_rows_in_the_order_of_their_voxels(n):
    # a solid block row by row: a piece holds few leaves, whole
    side = int(round(n ** (1 / 3))) + 1
    ax = torch.arange(side, dtype=torch.int32, device="cuda") - 9
    rows = torch.cartesian_prod(ax, ax, ax)
    joff = np.array([[0, rows.shape[0]]])
    g = fx.build_index_grid(rows, joff)
    assert g.num_voxels == rows.shape[0]
    _check(g, rows, joff)


@pytest.mark.parametrize("where", ["first", "last", "all"])
def test_records_of_two_words(where):
    # coordinates beyond 2^19 in one piece, or in every one
    n = 200_000
    rows = _rows(n, 90, 3)
    far = {"first": slice(0, 1), "last": slice(n - 70, n), "all": slice(0, n, 1000)}[where]
    rows[far, 1] += 700_000
    joff = np.array([[0, n]])
    _check(fx.build_index_grid(rows, joff), rows, joff)


@pytest.mark.parametrize("B", [2, 5, 8, 9, 16, 17, 40])
def test_batches_with_rows_between_the_grids(B):
    n = 150_000
    rows = _rows(n, 40, B)
    cut = np.linspace(100, n - 5000, 2 * B).astype(np.int64)
    joff = np.stack([cut[0::2], cut[1::2]], axis=1)
    joff[0, 1] = joff[0, 0]                                    # an empty grid
    _check(fx.build_index_grid(rows, joff), rows, joff)


@pytest.mark.parametrize("B,far", [(16, False), (16, True), (17, False), (40, False)])
@pytest.mark.parametrize("n", [150_000, 1_200_000])
def test_scattered_rows_of_many_grids(n, B, far):
    """Nearly as many leaves as rows, more than a bucket's table holds: several rounds over runs of records of one word, of two in some
    pieces (coordinates beyond 2^19), and of two in all (more than 16 grids)."""
    rows = _rows(n, 700, n + B)
    if far:
        rows[n // 3: n // 2, 2] += 600_000
    cut = np.sort(np.random.default_rng(B).integers(0, n, B + 1))
    joff = np.stack([cut[:-1], cut[1:]], axis=1)
    g = fx.build_index_grid(rows, joff)
    assert g.counts()[0] > 0.9 * (cut[-1] - cut[0])
    _check(g, rows, joff)


@pytest.mark.parametrize("size", [1.0, 0.05, 0.3, 7.7, 1e-3])
@pytest.mark.parametrize("n", [3_000, 40_000, 90_000])
def test_cells_of_points_near_faces(size, n):
    # multiples of the voxel size and their neighbours in single precision, where quotient and reciprocal may differ
    rng = np.random.default_rng(int(n * size))
    s, o = np.float32(size), np.float32(0.37)
    k = rng.integers(-400, 400, size=(n, 3))
    x = (k.astype(np.float32) * s + o).astype(np.float32)
    for _ in range(3):
        x = np.where(rng.random((n, 3)) < 0.5, np.nextafter(x, np.float32(rng.choice([-9e9, 9e9]))), x)
    cells = np.floor((x - o) / s).astype(np.int32)
    assert x.dtype == np.float32
    joff = np.array([[0, n]])
    g = fx.build_index_grid_from_points(torch.from_numpy(x).cuda(), joff, [float(o)] * 3, [float(s)] * 3)
    _check(g, torch.from_numpy(cells).cuda(), joff)


def test_points_that_no_cell_holds_are_refused():
    x = torch.rand((100_000, 3), device="cuda") * 100
    x[99_000, 2], x[5, 0] = float("nan"), float("inf")
    with pytest.raises(fx.FxError, match="^.*2 point coordinates"):
        fx.build_index_grid_from_points(x, np.array([[0, 100_000]]))

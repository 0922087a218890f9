"""Tiles that need about as many, and more, input rows than the tile kernels stage (816, two buffers of them, 1022 for the
weight gradient), grids split between the tile and leaf-window kernels, and the lines between those kernels, against sums in 64
bits over the dense map, which other tests compare with the oracle.

Tolerance: a product of two 16-bit numbers is exact in fp32; a sum of N of them in any order is off by at most 2^-24 sqrt(N)
of its size times a small factor, N <= 27 * 128 for a row and 2e5 for a weight: 3.5e-6 of a row's norm and 2.7e-5 of an
offset's, taken four times; results rounded to 16 bits add half a unit in the last place, at most 2^-8 (bf16) or 2^-11 (f16) of a value."""
import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx

pytestmark = pytest.mark.gpu

CAP = 816


def _index(pts):
    return fx.build_index_grid(torch.from_numpy(np.ascontiguousarray(pts.astype(np.int32))).cuda(), np.array([[0, pts.shape[0]]]))


def _norm_ok(y, ref, rel):
    return bool(((y.double() - ref).flatten(1).norm(dim=1) <= rel * ref.flatten(1).norm(dim=1) + 1e-30).all())


def _check(km, dtype, c_in, c_out):
    half = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda").to(H.TORCH_DT[dtype])
    x, w, gy = rand(km.g_in.num_voxels, c_in), rand(27, c_in, c_out), rand(km.n_out, c_out)
    t = km.dense().long()
    ref_y = torch.zeros((km.n_out, c_out), dtype=torch.float64, device="cuda")
    ref_x = torch.zeros((x.shape[0], c_in), dtype=torch.float64, device="cuda")
    ref_w = torch.zeros((27, c_in, c_out), dtype=torch.float64, device="cuda")
    for k in range(27):
        o = (t[:, k] >= 0).nonzero()[:, 0]
        i = t[o, k]
        ref_y[o] += x[i].double() @ w[k].double()
        ref_x[i] += gy[o].double() @ w[k].double().t()         # an input meets an offset at most once
        ref_w[k] = x[i].double().t() @ gy[o].double()
    y = fx.sparse_conv_fwd(km, x, w, out=H.nan_filled(ref_y.shape, H.TORCH_DT[dtype]))
    assert _norm_ok(y, ref_y, 1.4e-5 + half)
    y32 = fx.sparse_conv_fwd(km, x, w, out_dtype=torch.float32, out=H.nan_filled(ref_y.shape, torch.float32))
    assert _norm_ok(y32, ref_y, 1.4e-5) and torch.equal(y32.to(y.dtype), y)
    assert _norm_ok(fx.sparse_conv_bwd_data(km, gy, w, out_dtype=torch.float32), ref_x, 1.4e-5)
    assert _norm_ok(fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32), ref_w, 1.1e-4)


def _tile_rows(km):
    t = km.dense()
    return [int(torch.unique(t[s:s + 512][t[s:s + 512] >= 0]).numel()) for s in range(0, km.n_out, 512)]


def _inputs_for(g_out, rows, rng):
    """Input voxels such that tile t of outputs two apart reads rows[t % len(rows)] different ones of its surroundings."""
    out = g_out.ijk()[0].cpu().numpy()
    d = np.stack(np.meshgrid(*[np.arange(-1, 2)] * 3, indexing="ij"), axis=-1).reshape(1, 27, 3)
    have = {}
    for t, s in enumerate(range(0, out.shape[0], 512)):
        cells = np.unique((out[s:s + 512, None, :] + d).reshape(-1, 3), axis=0)
        keys = [tuple(c) for c in cells]
        want = min(rows[t % len(rows)], len(keys)) - sum(have.get(k, False) for k in keys)
        free = [k for k in keys if k not in have]
        for n, f in enumerate(rng.permutation(len(free))):
            have[free[f]] = n < want                # cells that are refused stay empty, those of earlier tiles stay what they are
    return np.array([k for k, v in have.items() if v])


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 32), ("bf16", 128, 96), ("f16", 40, 64)])
@pytest.mark.parametrize("rows", [[CAP - 1], [CAP, CAP + 1], [CAP + 1], [2 * CAP - 1, 2 * CAP, 2 * CAP + 1], [2 * CAP, 100, CAP], [1021, 1022, 500, 1023, 400], [2500, 1200, 300, CAP + 16, 815]])
def test_rows_of_a_tile(rows, dtype, c_in, c_out):
    rng = np.random.default_rng(len(rows) * 1000 + rows[0])
    lattice = np.stack(np.meshgrid(np.arange(40), np.arange(8), np.arange(56), indexing="ij"), axis=-1).reshape(-1, 3) * 2
    g_out = _index(lattice[:17_700])
    km = fx.build_kernel_map_onto(_index(_inputs_for(g_out, rows, rng)), g_out, 3)
    seen = _tile_rows(km)
    assert all(seen.count(r) >= 1 for r in rows if r <= 2 * CAP + 1), (rows, sorted(set(seen)))
    _check(km, dtype, c_in, c_out)


def _between(rows, tiles, shared):
    """A map onto a grid whose first tiles read rows[t % len(rows)] inputs each; `shared`: onto a grid at least twice the input's
    size, by outputs far off, whose tiles hold every row once."""
    lattice = np.stack(np.meshgrid(np.arange(40), np.arange(8), np.arange(56), indexing="ij"), axis=-1).reshape(-1, 3) * 2
    out = lattice[:512 * tiles - 220]
    pts = _inputs_for(_index(out), rows, np.random.default_rng(len(rows) * 1000 + rows[0]))
    if shared:
        side = int(np.ceil((2 * len(pts)) ** (1 / 3)))
        out = np.concatenate([out, 4000 + 3 * np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)])
    g_in, g_out = _index(pts), _index(out)
    assert (g_out.num_voxels >= 2 * g_in.num_voxels) == shared
    return fx.build_kernel_map_onto(g_in, g_out, 3)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 32), ("bf16", 128, 96), ("f16", 40, 64)])
@pytest.mark.parametrize("rows", [[CAP - 1], [CAP, CAP + 1], [CAP + 1], [1023, 1024, 100, CAP], [1021, 1022, 500, 1023, 400], [2500, 1200, 300, CAP + 16, 815]])
def test_rows_of_a_tile_between_two_grids(rows, dtype, c_in, c_out):
    """Staged in one half and in both (to 1024 rows, what a tile between two grids holds once each), and a row per pair beyond."""
    km = _between(rows, 35, True)
    seen = _tile_rows(km)
    assert all(seen.count(r) >= 1 for r in rows if r <= 1024), (rows, sorted(set(seen)))
    _check(km, dtype, c_in, c_out)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 160), ("bf16", 40, 24)])
@pytest.mark.parametrize("rows,tiles,shared,some", [([1022, 1000, 300], 24, True, 0), ([1024, 1022, 900], 24, True, 1), ([1024, 1023, 1400], 24, True, 17), ([900], 24, False, 17)])
def test_weight_gradient_between_two_grids(rows, tiles, shared, some, dtype, c_in, c_out):
    """All tiles staged by the weight gradient, up to 16 that are not and are listed, more than 16, and a map whose tiles list a row per pair."""
    km = _between(rows, tiles, shared)
    n = sum(r > 1022 for r in _tile_rows(km)) if shared else km.n_out // 512
    assert n == 0 if some == 0 else n > 16 if some > 16 else 1 <= n <= 16
    _check(km, dtype, c_in, c_out)


SHEETS = [[1631, 815, 816, 817, 1021, 1022, 1023, 700], [1632, 1500, 512, 1000, 1536, 900, 600, 1100], [1633, 1200, 1300, 2000, 850, 816, 1400, 513],
          [2048, 817, 1022, 1023, 2400, 1536, 1537, 800]]


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 32), ("bf16", 128, 96), ("f16", 40, 64), ("bf16", 160, 32)])
@pytest.mark.parametrize("sheets", [SHEETS[:1], SHEETS[1:3], SHEETS])
def test_rows_of_a_tile_of_one_grid(sheets, dtype, c_in, c_out):
    """One half of the row buffer, both to the last row, one row more, and tiles of a row per pair (more than 1024 rows far off), in turn."""
    km = fx.build_kernel_map(_index(H.facing_sheets(sheets)), 3, 1)
    counts = H.tile_row_counts(km.dense().cpu().numpy()).tolist()
    assert all(counts[i:i + 8] == s for s, i in zip(sheets, [counts.index(s[0]) for s in sheets]))
    _check(km, dtype, c_in, c_out)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 32), ("bf16", 96, 128)])
@pytest.mark.parametrize("last", [False, True])
def test_long_tiles_of_every_kind_first(last, dtype, c_in, c_out):
    """Few enough long tiles beside others that all are started first: both halves filled, rows beyond them, a row per pair."""
    side = -1 if last else 1
    cloud = np.unique(np.random.default_rng(15).integers(0, 500, size=(200_000, 3)), axis=0)[:199_680] + side * 4096
    short = [[1631, 512, 600, 700, 512, 640, 512, 650], [2048, 513, 1700, 512, 1500, 512, 700, 512]]
    km = fx.build_kernel_map(_index(np.concatenate([H.facing_sheets(short), cloud])), 3, 1)
    counts = H.tile_row_counts(km.dense().cpu().numpy())
    n_slices = (c_out + (31 if c_out <= 32 else 63)) // (32 if c_out <= 32 else 64)
    half = torch.cuda.get_device_properties(0).multi_processor_count // 2
    assert 5 <= (counts > CAP).sum() <= 32 and (counts > CAP).sum() * n_slices <= half < 2 * half < counts.size * n_slices
    assert ((counts > CAP) & (counts <= 2 * CAP)).any() and (counts > 2 * CAP).any()
    _check(km, dtype, c_in, c_out)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 64, 128)])
@pytest.mark.parametrize("p", [0.24, 0.285, 0.33])
def test_long_tiles_of_a_thin_block(p, dtype, c_in, c_out):
    a = np.stack(np.meshgrid(np.arange(64), np.arange(48), np.arange(40), indexing="ij"), axis=-1).reshape(-1, 3)
    km = fx.build_kernel_map(_index(a[np.random.default_rng(7).random(a.shape[0]) < p]), 3, 1)
    assert p < 0.3 or max(_tile_rows(km)) > CAP
    _check(km, dtype, c_in, c_out)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 64, 128)])
@pytest.mark.parametrize("thin", [144, 204, 205])
def test_grid_split_with_thin_leaves(thin, dtype, c_in, c_out, fx_opt):
    """Full leaves, leaves with exactly `thin` voxels and sheets through leaves, side by side: tiles that keep all, some and none
    of their outputs."""
    fx_opt("leaf_dispatch", 2)
    rng = np.random.default_rng(thin)
    cell = np.stack(np.meshgrid(*[np.arange(8)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    pts = []
    for b, org in enumerate(np.stack(np.meshgrid(np.arange(8), np.arange(6), np.arange(7), indexing="ij"), axis=-1).reshape(-1, 3)):
        kind = rng.integers(0, 4)
        pick = cell if kind == 0 else cell[rng.permutation(512)[:thin]] if kind < 3 else cell[cell[:, 1] == b % 8]
        pts.append(pick + 8 * org)
    pts.append(np.unique(rng.integers(80, 400, size=(60_000, 3)), axis=0))       # so that the mean leaf is not dense
    g = _index(np.concatenate(pts))
    km = fx.build_kernel_map(g, 3, 1)
    fx.profile_enable(True)
    fx.profile_reset()
    fx.sparse_conv_fwd(km, torch.zeros((g.num_voxels, c_in), device="cuda", dtype=H.TORCH_DT[dtype]),
                       torch.zeros((27, c_in, c_out), device="cuda", dtype=H.TORCH_DT[dtype]))
    torch.cuda.synchronize()
    slots = fx.profile_read()
    fx.profile_enable(False)
    assert "k_conv_leaf" in slots and "k_conv_mfma" in slots
    _check(km, dtype, c_in, c_out)


def _reduction_grid(n, seed):
    rng = np.random.default_rng(seed)
    side = int(round(4.5 * n ** (1 / 3)))
    return _index(np.unique(rng.integers(0, side, size=(n, 3)), axis=0))


@pytest.mark.parametrize("n,dtype,c_in,c_out", [(98_500, "f16", 4, 32), (104_000, "f16", 4, 32), (104_000, "bf16", 32, 32), (140_000, "bf16", 64, 64),
                                                (140_000, "f16", 8, 32), (140_000, "bf16", 32, 160)])
def test_partial_sums_of_a_small_weight_gradient(n, dtype, c_in, c_out):
    """192, 200 and 256 ranges: above 192 a small tensor's sums are added by eight waves."""
    _check(fx.build_kernel_map(_reduction_grid(n, n), 3, 1), dtype, c_in, c_out)


@pytest.mark.parametrize("p,thick,dtype,c_in,c_out", [(0.38, 28, "bf16", 64, 64), (0.47, 24, "bf16", 64, 64), (0.47, 48, "f16", 32, 64), (0.57, 40, "bf16", 96, 64),
                                                      (0.62, 40, "bf16", 64, 64), (1.0, 20, "f16", 64, 64), (1.0, 40, "bf16", 64, 128)])
def test_either_side_of_the_lines_of_dense_grids(p, thick, dtype, c_in, c_out):
    """Random voxels of a cube of whole leaves and solid cubes across them: mean occupancies below 0.40, to 0.60 and above, of fewer
    and more than 16 k voxels, weight gradients with few and with many tiles that are not staged."""
    a = np.stack(np.meshgrid(*[np.arange(thick)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) - 4 * (thick % 16 != 0)
    _check(fx.build_kernel_map(_index(a[np.random.default_rng(8).random(a.shape[0]) < p]), 3, 1), dtype, c_in, c_out)


@pytest.mark.parametrize("share", [0.5, 0.6])
def test_either_side_of_the_line_of_a_split(share):
    """Full leaves with half and with six tenths of a grid's voxels."""
    rng = np.random.default_rng(9)
    cloud = np.unique(rng.integers(100, 300, size=(int(13_824 * (1 - share) / share), 3)), axis=0)
    cube = np.stack(np.meshgrid(*[np.arange(24)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    _check(fx.build_kernel_map(_index(np.concatenate([cube, cloud])), 3, 1), "bf16", 64, 64)


@pytest.mark.parametrize("dtype,c_in,c_out,split", [("bf16", 64, 64, False), ("f16", 128, 128, True), ("bf16", 32, 64, False), ("bf16", 128, 192, True),
                                                    ("f16", 192, 256, True), ("f16", 256, 256, False)])
def test_weight_gradient_split_by_size(dtype, c_in, c_out, split):
    """A solid cube with 11 % of the voxels, all tiles staged: alone where few blocks of channels share them, split per leaf from
    (0.30 - share) x outputs x blocks of 32 x 64 channels = 2^18 on; the layers that are summed from lists of pairs are not split."""
    cloud = np.unique(np.random.default_rng(12).integers(200, 460, size=(269_000, 3)), axis=0)
    cube = np.stack(np.meshgrid(*[np.arange(32)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    km = fx.build_kernel_map(_index(np.concatenate([cube, cloud])), 3, 1)
    share = 32768 / km.n_out
    assert 0.10 < share < 0.12 and max(_tile_rows(km)) <= 1022
    assert ((0.30 - share) * km.n_out * (c_in // 32) * (c_out // 64) >= 2 ** 18 and (c_in % 256 != 0 or c_out % 256 != 0)) == split
    x = torch.zeros((km.n_out, c_in), device="cuda", dtype=H.TORCH_DT[dtype])
    gy = torch.zeros((km.n_out, c_out), device="cuda", dtype=H.TORCH_DT[dtype])
    fx.profile_enable(True)
    fx.profile_reset()
    fx.sparse_conv_bwd_weight(km, x, gy)
    torch.cuda.synchronize()
    slots = fx.profile_read()
    fx.profile_enable(False)
    assert slots["k_wgrad"][1] == (2 if split else 1)               # the dense leaves' kernel and the tiles', or the tiles' alone
    _check(km, dtype, c_in, c_out)


@pytest.mark.parametrize("p,n_more,c_in,leaf", [(0.53, True, 64, False), (0.55, True, 64, True), (0.55, True, 192, True), (0.55, True, 224, False), (0.55, False, 64, False),
                                                (0.61, False, 64, True)])
def test_line_of_large_dense_grids(p, n_more, c_in, leaf):
    """Random voxels of a block of leaves, as many as 2^20 or one fewer: the leaf window from 0.54 on at up to 192 channels, or
    from 0.60 on."""
    n = 2 ** 20 - (0 if n_more else 1)
    cells = np.random.default_rng(13).permutation(512 * int(n / (512 * p)))[:n]
    g = _index(8 * np.stack(np.unravel_index(cells // 512, (16,) * 3), axis=1) + np.stack(np.unravel_index(cells % 512, (8,) * 3), axis=1))
    occupancy = n / (512 * g.counts()[0])
    assert abs(occupancy - p) < 0.001 and (occupancy >= (0.54 if n_more and c_in <= 192 else 0.60)) == leaf
    km = fx.build_kernel_map(g, 3, 1)
    gen = torch.Generator(device="cuda").manual_seed(14)
    x = torch.randn((n, c_in), generator=gen, device="cuda").bfloat16()
    w = torch.randn((27, c_in, 64), generator=gen, device="cuda").bfloat16()
    fx.profile_enable(True)
    fx.profile_reset()
    y = fx.sparse_conv_fwd(km, x, w, out_dtype=torch.float32, out=H.nan_filled((n, 64), torch.float32))
    torch.cuda.synchronize()
    slots = fx.profile_read()
    fx.profile_enable(False)
    assert ("k_conv_leaf" in slots) == leaf
    at = torch.cat([torch.arange(s, s + 512, device="cuda") for s in (0, n // 2, n - 512)])
    t, ref = km.dense()[at].long(), 0.0
    for k in range(27):
        ref = ref + torch.where((t[:, k] >= 0)[:, None], x[t[:, k].clamp(min=0)].double(), 0.0) @ w[k].double()
    assert _norm_ok(y[at], ref, 1.4e-5 * 2)                          # 27 * 224 products a sum, where 27 * 128 give 1.4e-5


@pytest.mark.parametrize("dtype,c_in,c_out,tiles,leaves,leaf", [
    ("bf16", 32, 64, 513, 1024, True), ("bf16", 32, 64, 513, 1025, False), ("f16", 32, 64, 512, 1024, False), ("f16", 64, 64, 1024, 1800, False),
    ("bf16", 64, 64, 880, 1536, True), ("bf16", 64, 64, 880, 1537, False), ("bf16", 64, 64, 1025, 2000, False), ("f16", 32, 192, 590, 1000, True),
    ("f16", 64, 128, 590, 1000, False), ("bf16", 96, 64, 590, 1000, True), ("bf16", 96, 128, 590, 1000, False), ("bf16", 32, 128, 1024, 1860, True), ("bf16", 32, 64, 1024, 1860, False),
    ("bf16", 32, 128, 1023, 1860, False)])
def test_rounds_of_tiles_and_leaves(dtype, c_in, c_out, tiles, leaves, leaf):
    """Random voxels of a block of leaves between the lines: three or four rounds of tiles against fewer of leaves, as many, and at 32
    channels 2^19 voxels.  Forward pass and, where the counts allow it, the input gradient."""
    n = 512 * tiles
    assert (torch.cuda.get_device_properties(0).multi_processor_count, 0.40 < tiles / leaves) == (256, True)
    cells = np.random.default_rng(tiles).permutation(512 * leaves)[:n]
    g = _index(8 * np.stack(np.unravel_index(cells // 512, (16,) * 3), axis=1) + np.stack(np.unravel_index(cells % 512, (8,) * 3), axis=1))
    assert g.num_voxels == n and g.counts()[0] == leaves
    km = fx.build_kernel_map(g, 3, 1)
    gen = torch.Generator(device="cuda").manual_seed(16)
    x = torch.randn((n, c_in), generator=gen, device="cuda").to(H.TORCH_DT[dtype])
    w = torch.randn((27, c_in, c_out), generator=gen, device="cuda").to(H.TORCH_DT[dtype])
    at = torch.cat([torch.arange(s, s + 512, device="cuda") for s in (0, n // 2, n - 512)])
    t = km.dense()[at].long()
    for back in ([False, True] if c_in == c_out else [False]):
        fx.profile_enable(True)
        fx.profile_reset()
        y = (fx.sparse_conv_bwd_data if back else fx.sparse_conv_fwd)(km, x, w, out_dtype=torch.float32, out=H.nan_filled((n, c_out), torch.float32))
        torch.cuda.synchronize()
        slots = fx.profile_read()
        fx.profile_enable(False)
        assert ("k_conv_leaf" in slots) == leaf
        ref = 0.0
        for k in range(27):                                          # an input is the neighbour at the opposite offset of its outputs
            m = t[:, 26 - k] if back else t[:, k]
            ref = ref + torch.where((m >= 0)[:, None], x[m.clamp(min=0)].double(), 0.0) @ (w[k].double().t() if back else w[k].double())
        assert _norm_ok(y[at], ref, 1.4e-5)


@pytest.mark.parametrize("dtype,c_in,c_out,n,p,listed,leaf", [
    ("bf16", 64, 64, 20_000, 0.59, 1, False), ("bf16", 64, 64, 24_000, 0.58, 2, True), ("f16", 64, 128, 24_000, 0.58, 2, True),
    ("bf16", 96, 128, 24_000, 0.58, 2, False), ("f16", 32, 64, 100_000, 0.53, 3, True), ("bf16", 64, 64, 90_000, 0.55, 2, True),
    ("f16", 64, 64, 100_000, 0.53, 3, False), ("bf16", 64, 128, 90_000, 0.55, 2, False)])
def test_dense_grids_with_few_listed_tiles(dtype, c_in, c_out, n, p, listed, leaf, fx_opt):
    """The weight gradient between 0.40 and 0.60 mean occupancy: one tile that is not staged, and more on either side of the sizes
    at which their launch is worth it.  Which kernel ran shows in the bits."""
    side = int(round((n / p) ** (1 / 3) / 8)) * 8
    depth = int(round(n / p / (side * side) / 8)) * 8
    g = _index(np.argwhere(np.random.default_rng(n).random((side, side, depth)) < p))
    km = fx.build_kernel_map(g, 3, 1)
    assert 0.40 <= km.n_out / (512 * g.counts()[0]) < 0.60 and (H.tile_row_counts(km.dense().cpu().numpy()) > 1022).sum() == listed
    assert (listed >= 2 and (c_in * c_out == 32 * 64 or c_in * c_out <= 4 * 32 * 64 and c_in * c_out * km.n_out < 32 * 64 * 200_000)) == leaf
    gen = torch.Generator(device="cuda").manual_seed(17)
    x, gy = (torch.randn((km.n_out, c), generator=gen, device="cuda").to(H.TORCH_DT[dtype]) for c in (c_in, c_out))
    gw = fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32)
    for switch in (0, 1):
        fx_opt("leaf_dispatch", switch)
        assert torch.equal(gw, fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32)) == (switch == int(leaf))
    fx_opt("leaf_dispatch", -1)
    _check(km, dtype, c_in, c_out)

"""GPU parity of per-leaf dispatch: one call of the 3x3x3 submanifold convolution (or its input gradient) on a grid
that mixes locally dense leaves with sparse ones runs the leaf-window kernel on the dense leaves and the tile kernel
on everything else; every output row against the oracle, outputs NaN before the call."""
import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx
from oracle import cpu_oracle as O
from workloads import generators as G

pytestmark = pytest.mark.gpu


def _kernels_of(fn):
    fx.profile_enable(True)
    fx.profile_reset()
    out = fn()
    torch.cuda.synchronize()
    slots = fx.profile_read()
    fx.profile_enable(False)
    return out, slots


def _check_forward_and_input_gradient(pts, jo, dtype, c_in, c_out, expect_both, seed=61):
    g, og = H.both_grids(pts, jo)
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(seed, og.num_voxels, c_in, c_out, 27, dtype)
    gy = G.round_to_dtype(np.random.default_rng(seed + 1).standard_normal((og.num_voxels, c_out)).astype(np.float32), dtype)
    d_x, d_w, d_gy = (H.to_device_storage(a, dtype) for a in (feat, wt, gy))
    out = H.nan_filled((og.num_voxels, c_out), H.TORCH_DT[dtype])
    _, slots = _kernels_of(lambda: fx.sparse_conv_fwd(km, d_x, d_w, out=out))
    if expect_both:
        assert "k_conv_leaf" in slots and "k_conv_mfma" in slots
    y = out.float().cpu().numpy()
    assert np.isfinite(y).all()
    H.conv_tolerance_check(y, O.conv(og, og, 3, 1, feat, wt, threads=H.ORACLE_THREADS), dtype, 27, c_in)
    gx = H.nan_filled((og.num_voxels, c_in), torch.float32)
    fx.sparse_conv_bwd_data(km, d_gy, d_w, out_dtype=torch.float32, out=gx)
    gx = gx.cpu().numpy()
    assert np.isfinite(gx).all()
    H.conv_tolerance_check(gx, O.conv_bwd_data(og, og, 3, 1, gy, wt, threads=min(4, H.ORACLE_THREADS)), dtype, 27, c_out)
    # the weight gradient is split the same way: dense leaves' pairs from the leaf window, the others from the tiles
    gw, wslots = _kernels_of(lambda: fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32))
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((gw.cpu().numpy().astype(np.float64) - ref) ** 2).sum(axis=(1, 2)))
    den = np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))
    assert (num / den).max() <= 2e-3
    assert torch.equal(gw, fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32))      # fixed order of the sums
    return g


@pytest.mark.parametrize("switch", [None, 2])
@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 32, 128)])
def test_mixed_grid_is_split_between_the_two_kernels(switch, dtype, c_in, c_out, fx_opt):
    if switch is not None:
        fx_opt("leaf_dispatch", switch)
    w = G.workload("mixed_small")
    ijk, jo = w.jagged_ijk(dup_fraction=0.01)
    g = _check_forward_and_input_gradient(ijk, jo, dtype, c_in, c_out, expect_both=True)
    cnt = np.diff(np.append(g.leaf_table()["offset"], g.num_voxels))
    assert 0.1 < cnt[cnt >= 205].sum() / g.num_voxels < 0.9          # the automatic rule applies to this grid


def test_forced_split_with_no_dense_leaf_and_with_only_dense_leaves(fx_opt):
    fx_opt("leaf_dispatch", 2)
    w = G.workload("lidar_small")                                   # no leaf reaches 205 voxels: the leaf kernel gets an empty list
    ijk, jo = w.jagged_ijk()
    _check_forward_and_input_gradient(ijk, jo, "bf16", 64, 64, expect_both=False)
    a = np.arange(-16, 16, dtype=np.int32)                            # 64 full leaves: every tile of the split map is empty
    blk = np.stack(np.meshgrid(a, a, a, indexing="ij"), axis=-1).reshape(-1, 3)
    _check_forward_and_input_gradient(blk, np.array([[0, blk.shape[0]]], np.int64), "bf16", 64, 64, expect_both=False)
    # a batch: one member dense, one sparse, one empty
    grids = [blk[:8192], w.grids[0][:20000], np.zeros((0, 3), np.int32)]
    pts, jo = G.make_jagged(grids)
    _check_forward_and_input_gradient(pts, jo, "f16", 32, 64, expect_both=False)


def test_full_size_mixed_grid_every_row():
    """697 301 voxels, 62 % of them in locally dense leaves, mean leaf occupancy 0.16: the automatic rule splits it."""
    w = G.workload("mixed1m")
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = w.feats_weights()
    out = H.nan_filled((og.num_voxels, w.c_out), torch.bfloat16)
    _, slots = _kernels_of(lambda: fx.sparse_conv_fwd(km, H.to_device_storage(feat, "bf16"), H.to_device_storage(wt, "bf16"), out=out))
    assert "k_conv_leaf" in slots and "k_conv_mfma" in slots
    y = out.float().cpu().numpy()
    assert np.isfinite(y).all()
    H.conv_tolerance_check(y, O.conv(og, og, 3, 1, feat, wt, threads=H.ORACLE_THREADS), "bf16", 27, 64)


@pytest.mark.parametrize("switch", [None, 2])
@pytest.mark.parametrize("corner", [-2000, 1000])
@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 96, 128)])
def test_split_weight_gradient_with_listed_tiles(dtype, c_in, c_out, corner, switch, fx_opt):
    # full leaves for the leaf-window kernel, a sparse cloud whose tiles are staged, and a block at a third of its voxels, below
    # the line of a dense leaf, whose few tiles are not staged: one sum of three kernels' partial sums, the first or the last tiles
    if switch is not None:
        fx_opt("leaf_dispatch", switch)
    rng = np.random.default_rng(91)
    box = lambda dims, at: np.stack(np.meshgrid(*[np.arange(d, dtype=np.int64) + at for d in dims], indexing="ij"), axis=-1).reshape(-1, 3)
    third = box((32, 32, 24), corner)
    pts = np.concatenate([rng.integers(-300, 300, size=(30000, 3)), box((32, 32, 16), corner + 512), third[rng.random(third.shape[0]) < 0.34]]).astype(np.int32)
    g, og = H.both_grids(pts[rng.permutation(pts.shape[0])], np.array([[0, pts.shape[0]]]))
    n, km = og.num_voxels, fx.build_kernel_map(g, 3, 1)
    cnt = np.diff(np.append(g.leaf_table()["offset"], n))
    sparse_out = np.repeat(cnt < 205, cnt)
    assert (cnt == 512).sum() == 32 and n / (512 * cnt.size) < 0.20 and 0.1 < cnt[cnt >= 205].sum() / n < 0.5
    # tiles without their dense leaves' outputs: some whose rows do not fit (792), no more than are listed (16)
    table, tiles = km.dense().cpu().numpy(), range((n + 511) // 512)
    rows = [np.unique(table[512 * t:512 * t + 512][sparse_out[512 * t:512 * t + 512]]) for t in tiles]
    assert 1 <= sum(r.size - 1 > 792 for r in rows) and sum(np.union1d(r, np.arange(512) + 512 * t).size - 1 > 792 for t, r in enumerate(rows)) <= 16
    feat, _ = G.features_and_weights(92, n, c_in, c_out, 27, dtype)
    gy = G.round_to_dtype(np.random.default_rng(93).standard_normal((n, c_out)).astype(np.float32), dtype)
    gw = H.nan_filled((27, c_in, c_out), torch.float32)
    fx.sparse_conv_bwd_weight(km, H.to_device_storage(feat, dtype), H.to_device_storage(gy, dtype), out_dtype=torch.float32, out=gw)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((gw.cpu().numpy().astype(np.float64) - ref) ** 2).sum(axis=(1, 2)))
    assert (num / np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))).max() <= 2e-3


@pytest.mark.parametrize("switch", [None, 2])
@pytest.mark.parametrize("corner", [-2000, 1000])
@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 64), ("f16", 96, 128)])
def test_automatic_split_weight_gradient_with_listed_tiles(dtype, c_in, c_out, corner, switch, fx_opt):
    # full leaves for the leaf-window kernel, whose tiles in the whole map are too long for the weight gradient to stage (more than are
    # listed, so that the automatic rule splits), a sparse cloud whose tiles are staged, and sheets that face one another, of some
    # voxels a leaf, with a few tiles that are not staged: one sum of three kernels' partial sums, the first or the last tiles
    if switch is not None:
        fx_opt("leaf_dispatch", switch)
    rng = np.random.default_rng(91)
    sheets = H.facing_sheets([[1023, 1022, 700, 1400, 1024, 816, 1200, 512], [1900, 1021, 900, 1300, 1023, 512, 640, 817]]) + np.array([corner // 128 * 128] * 3)
    pts = np.concatenate([rng.integers(-300, 300, size=(30000, 3)), H.box((32, 32, 32), (500, 500, 500)), H.box((24,) * 3, (corner + 2000,) * 3), sheets]).astype(np.int32)
    g, og = H.both_grids(pts[rng.permutation(pts.shape[0])], np.array([[0, pts.shape[0]]]))
    n, km = og.num_voxels, fx.build_kernel_map(g, 3, 1)
    cnt = np.diff(np.append(g.leaf_table()["offset"], n))
    sparse_out = np.repeat(cnt < 205, cnt)
    assert n / (512 * cnt.size) < 0.40 and 0.1 < cnt[cnt >= 205].sum() / n < 0.5
    # the rows that tiles without their dense leaves' outputs hold: those around the outputs that are left, and the tile's own if all are
    table, tiles = km.dense().cpu().numpy(), range((n + 511) // 512)
    assert (H.tile_row_counts(table) > 1022).sum() > 16
    rows = []
    for t in tiles:
        left = table[512 * t:512 * t + 512][sparse_out[512 * t:512 * t + 512]]
        whole = left.shape[0] == min(512, n - 512 * t)
        rows.append(np.union1d(left[left >= 0], np.arange(512) + 512 * t if whole else []).size)
    assert 4 <= sum(r > 1022 for r in rows) <= 16
    feat, _ = G.features_and_weights(92, n, c_in, c_out, 27, dtype)
    gy = G.round_to_dtype(np.random.default_rng(93).standard_normal((n, c_out)).astype(np.float32), dtype)
    gw = H.nan_filled((27, c_in, c_out), torch.float32)
    d_x, d_gy = H.to_device_storage(feat, dtype), H.to_device_storage(gy, dtype)
    _, slots = _kernels_of(lambda: fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32, out=gw))
    assert slots["k_wgrad"][1] == 2                                  # the dense leaves', and the tiles' (with the listed ones)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((gw.cpu().numpy().astype(np.float64) - ref) ** 2).sum(axis=(1, 2)))
    assert (num / np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))).max() <= 2e-3


@pytest.mark.parametrize("op,kernel,stride,c_in,c_out,line", [
    ("fwd", 1, 1, 24, 200, 6250), ("bwd_data", 1, 1, 200, 24, 6250), ("fwd", 2, 2, 24, 200, 7500), ("bwd_data", 2, 2, 24, 200, 4166),
    ("bwd_data of outputs", 2, 2, 40, 40, 1562), ("bwd_data of outputs", 2, 2, 48, 96, 325), ("bwd_data of outputs", 2, 2, 16, 16, 5859),
    ("transposed of outputs", 2, 2, 40, 40, 4531), ("transposed of outputs", 2, 2, 40, 136, 4365)])
@pytest.mark.parametrize("past", [0, 1])
def test_partial_chunks_of_few_products_take_the_scalar_kernel(op, kernel, stride, c_in, c_out, line, past):
    # one offset a voxel, or one pair an input: up to a number of products the scalar kernel, which packs no weights, is the
    # faster one; both sides of the line, in inputs or in outputs, against the oracle
    rng = np.random.default_rng(71)
    pts = np.unique(rng.integers(-20, 20, size=(3 * line, 3)).astype(np.int32), axis=0)
    pts = pts[rng.permutation(pts.shape[0])[:line + past]]
    if op.endswith(" of outputs"):                     # some of the children of every output
        op, pts = op[:-len(" of outputs")], 2 * pts
        pts = np.concatenate([pts, pts[::2] + 1, pts[::3] + np.array([0, 1, 0], np.int32)])
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km, ogo = fx.build_kernel_map(g, kernel, stride), O.output_grid(og, kernel, stride)
    assert line + past in (og.num_voxels, ogo.num_voxels)
    feat, wt = G.features_and_weights(72, og.num_voxels, c_in, c_out, kernel ** 3, "bf16")
    gy = G.round_to_dtype(np.random.default_rng(73).standard_normal((ogo.num_voxels, c_out)).astype(np.float32), "bf16")
    wt_t = np.ascontiguousarray(wt.transpose(0, 2, 1))
    dev = lambda a: H.to_device_storage(a, "bf16")
    run, ref, contracted = {
        "fwd": (lambda: fx.sparse_conv_fwd(km, dev(feat), dev(wt)), lambda: O.conv(og, ogo, kernel, stride, feat, wt), c_in),
        "bwd_data": (lambda: fx.sparse_conv_bwd_data(km, dev(gy), dev(wt)), lambda: O.conv_bwd_data(og, ogo, kernel, stride, gy, wt), c_out),
        "transposed": (lambda: fx.sparse_conv_transpose_fwd(km, dev(gy), dev(wt_t)), lambda: O.conv_transpose(og, ogo, kernel, stride, gy, wt_t), c_out),
    }[op]
    y, slots = _kernels_of(run)
    assert ("k_pack_weights" in slots) == bool(past)
    H.conv_tolerance_check(y.float().cpu().numpy(), ref(), "bf16", kernel ** 3, contracted)


@pytest.mark.parametrize("corner", [-4000, 3000])
def test_list_of_dense_leaves_is_the_same_for_every_map(corner):
    # 48 k leaves of one voxel and 512 full ones at either end of the leaf order (the list is made in steps of 32 k leaves):
    # forward and weight gradient against the scalar kernel, and the same bits from every map of the grid
    rng = np.random.default_rng(81)
    cells = np.unique(rng.integers(-150, 150, size=(48500, 3)), axis=0) * 16 + 5
    a = [np.arange(n, dtype=np.int64) + corner for n in (64, 64, 64)]
    pts = np.concatenate([cells, np.stack(np.meshgrid(*a, indexing="ij"), axis=-1).reshape(-1, 3)]).astype(np.int32)
    g, og = H.both_grids(pts[rng.permutation(pts.shape[0])], np.array([[0, pts.shape[0]]]))
    cnt = np.diff(np.append(g.leaf_table()["offset"], g.num_voxels))
    assert cnt.size > 32768 and (cnt >= 205).sum() >= 512
    feat, wt = G.features_and_weights(82, og.num_voxels, 64, 64, 27, "bf16")
    gy = G.round_to_dtype(np.random.default_rng(83).standard_normal((og.num_voxels, 64)).astype(np.float32), "bf16")
    d_x, d_w, d_gy = (H.to_device_storage(v, "bf16") for v in (feat, wt, gy))
    first = None
    for _ in range(6):
        km = fx.build_kernel_map(g, 3, 1)
        gw, slots = _kernels_of(lambda: fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32))
        first = gw if first is None else first
        assert torch.equal(gw.view(torch.int32), first.view(torch.int32))
    y, slots = _kernels_of(lambda: fx.sparse_conv_fwd(km, d_x, d_w))
    assert "k_conv_leaf" in slots and "k_conv_mfma" in slots
    for s in (0, og.num_voxels // 2, og.num_voxels - 400):
        H.conv_tolerance_check(y[s:s + 400].float().cpu().numpy(), O.conv(og, og, 3, 1, feat, wt, s, s + 400)[s:s + 400], "bf16", 27, 64)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((first.cpu().numpy().astype(np.float64) - ref) ** 2).sum(axis=(1, 2)))
    assert (num / np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * 64)).max() <= 2e-3

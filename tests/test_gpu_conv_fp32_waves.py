"""fp32 convolution by one wave per 16 voxels (few tiles, strided maps, up to 32 produced channels): forward and input
gradient against the oracle at the fp32 bar, at the edges of its 16-voxel and 16-channel blocks."""
import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx
from oracle import cpu_oracle as O
from workloads import generators as G

pytestmark = pytest.mark.gpu


def _cloud(n):
    rng = np.random.default_rng(n)
    solid = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    side = 40 if n < 10_000 else 120
    return np.unique(np.concatenate([solid[: n // 2], rng.integers(-side, side, size=(n, 3))])[:n].astype(np.int32), axis=0)


def _check(n, K, stride, c_in, c_out, shift=0):
    pts = _cloud(n)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, K, stride)
    ogo = O.output_grid(og, K, stride)
    feat, wt = G.features_and_weights(31, og.num_voxels, c_in, c_out, K ** 3, "f32")
    gy = np.random.default_rng(32).standard_normal((ogo.num_voxels, c_out)).astype(np.float32)

    def dev(a):          # shift: rows that start `shift` elements into an allocation
        flat = torch.empty(a.size + shift, device="cuda")
        flat[shift:] = torch.from_numpy(np.ascontiguousarray(a)).cuda().reshape(-1)
        return flat[shift:].view(a.shape)

    y = H.nan_filled((ogo.num_voxels, c_out), torch.float32)
    fx.sparse_conv_fwd(km, dev(feat), dev(wt), out=y)
    H.conv_tolerance_check(y.cpu().numpy(), O.conv(og, ogo, K, stride, feat, wt), "f32", K ** 3, c_in)
    gx = fx.sparse_conv_bwd_data(km, dev(gy), dev(wt)).cpu().numpy()
    H.conv_tolerance_check(gx, O.conv_bwd_data(og, ogo, K, stride, gy, wt), "f32", K ** 3, c_out)


@pytest.mark.parametrize("n", [1, 15, 17, 33, 513, 3000])
@pytest.mark.parametrize("c_in,c_out", [(16, 1), (16, 5), (32, 32), (48, 20), (64, 80)])
def test_block_edges(n, c_in, c_out):
    _check(n, 3, 1, c_in, c_out)


@pytest.mark.parametrize("K,stride", [(1, 1), (2, 2), (3, 2)])
@pytest.mark.parametrize("c_in,c_out", [(16, 33), (32, 64), (80, 48)])
def test_other_maps(K, stride, c_in, c_out):
    _check(3000, K, stride, c_in, c_out)


@pytest.mark.parametrize("c_in,c_out", [(16, 64), (64, 16), (32, 32), (16, 30)])
def test_two_column_blocks_a_wave(c_in, c_out):
    # 20 k rows: four waves for every SIMD without the second block at 64 produced channels; 70 k at 32 and below
    _check(20_000 if max(c_in, c_out) == 64 else 70_000, 3, 1, c_in, c_out)


@pytest.mark.parametrize("c_in,c_out", [(16, 32), (32, 16)])
def test_unaligned_rows_take_the_scalar_kernel(c_in, c_out):
    _check(500, 3, 1, c_in, c_out, shift=1)


@pytest.mark.parametrize("K,stride,n,c_in,c_out", [(3, 1, 700, 32, 32), (3, 1, 700, 16, 5), (3, 1, 20_000, 64, 64), (2, 2, 3000, 32, 64),
                                                   (3, 2, 3000, 48, 40)])
@pytest.mark.parametrize("backward", [False, True])
def test_non_finite_weights_reach_only_the_rows_with_that_tap(K, stride, n, c_in, c_out, backward):
    # 0 * inf is NaN: an infinite or NaN weight of one offset must not reach rows without a neighbour there.  One output
    # column holds the infinity, another the NaN; the others stay finite everywhere.
    pts = _cloud(n)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, K, stride)
    ogo = O.output_grid(og, K, stride)
    n_src, n_dst = (ogo, og) if backward else (og, ogo)
    x, wt = G.features_and_weights(33, n_src.num_voxels, c_in, c_out, K ** 3, "f32")
    wt[1, 0, 2] = np.inf
    wt[K ** 3 - 2, c_in - 1, c_out - 1] = np.nan
    if backward:
        wt = np.ascontiguousarray(wt.transpose(0, 2, 1))
        y = fx.sparse_conv_bwd_data(km, torch.from_numpy(x).cuda(), torch.from_numpy(wt).cuda())
        ref = O.conv_bwd_data(og, ogo, K, stride, x, wt)
    else:
        y = fx.sparse_conv_fwd(km, torch.from_numpy(x).cuda(), torch.from_numpy(wt).cuda())
        ref = O.conv(og, ogo, K, stride, x, wt)
    y = y.cpu().numpy()
    assert np.array_equal(np.isnan(y), np.isnan(ref)) and np.array_equal(np.isinf(y), np.isinf(ref))
    assert np.array_equal(y[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    assert 0 < (~ok).sum() < 2 * n_dst.num_voxels
    # the row-wise bar of the finite case, over the columns that are finite everywhere
    cols = ok.all(axis=0)
    H.conv_tolerance_check(y[:, cols], ref[:, cols], "f32", K ** 3, c_in)

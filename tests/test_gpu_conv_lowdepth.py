"""GPU parity at up to 16 contracted channels of a 16-bit type: forward, input gradient and weight gradient against the oracle.

Tolerances as in the other convolution tests: per-row relative L2 <= 2e-2 for 16-bit outputs (one rounding of fp32 sums of
exact products is 2^-9), and per-offset relative Frobenius <= 2e-3 for the fp32 weight gradient."""
import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx
from oracle import cpu_oracle as O
from workloads import generators as G

pytestmark = pytest.mark.gpu


def _cloud(n):
    """n rows: a solid corner (every tap present) and scattered voxels (hardly any)."""
    rng = np.random.default_rng(n)
    solid = np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    far = rng.integers(-40, 40, size=(n, 3))
    return np.unique(np.concatenate([solid[: n // 2], far])[:n].astype(np.int32), axis=0)


# row counts around the 32-row blocks and 64-voxel chunks; channel counts below, at and above the padded 4, 8 and 16 and
# the 32- and 64-column slices (odd ones leave element-wise loads and stores)
@pytest.mark.parametrize("n", [1, 31, 64, 65, 3000])
@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 4, 32), ("bf16", 3, 32), ("bf16", 1, 20), ("f16", 8, 64), ("bf16", 5, 33),
                                              ("f16", 12, 100), ("bf16", 16, 31), ("f16", 16, 64)])
def test_low_depth_against_the_oracle(n, dtype, c_in, c_out):
    pts = _cloud(n)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(21, og.num_voxels, c_in, c_out, 27, dtype)
    gy = G.round_to_dtype(np.random.default_rng(22).standard_normal((og.num_voxels, c_out)).astype(np.float32), dtype)
    d_x, d_w, d_gy = (H.to_device_storage(a, dtype) for a in (feat, wt, gy))
    y = H.nan_filled((og.num_voxels, c_out), H.TORCH_DT[dtype])
    fx.sparse_conv_fwd(km, d_x, d_w, out=y)
    H.conv_tolerance_check(y.float().cpu().numpy(), O.conv(og, og, 3, 1, feat, wt), dtype, 27, c_in)
    y32 = fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32)
    assert np.abs(y32.cpu().numpy() - O.conv(og, og, 3, 1, feat, wt)).max() <= 1e-4 * np.sqrt(27 * c_in)
    # the other way round: c_in channels contracted by the input gradient of a c_out -> c_in layer
    wt_b = np.ascontiguousarray(wt.transpose(0, 2, 1))
    gx = fx.sparse_conv_bwd_data(km, d_x, H.to_device_storage(wt_b, dtype)).float().cpu().numpy()
    H.conv_tolerance_check(gx, O.conv_bwd_data(og, og, 3, 1, feat, wt_b), dtype, 27, c_in)
    gw = H.nan_filled((27, c_in, c_out), torch.float32)
    fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32, out=gw)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((gw.cpu().numpy() - ref) ** 2).sum(axis=(1, 2)))
    den = np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))
    assert (num / den).max() <= 2e-3
    assert torch.equal(gw, fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32))


@pytest.mark.parametrize("K,stride", [(1, 1), (5, 1), (2, 2), (3, 2)])
@pytest.mark.parametrize("c_in,c_out", [(4, 32), (8, 40), (16, 64)])
def test_low_depth_other_kernel_sizes(K, stride, c_in, c_out):
    # 5x5x5 at more than four channels does not fit and stays on the scalar kernel
    pts = _cloud(2000)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, K, stride)
    ogo = O.output_grid(og, K, stride)
    feat, wt = G.features_and_weights(23, og.num_voxels, c_in, c_out, K ** 3, "bf16")
    gy = G.round_to_dtype(np.random.default_rng(24).standard_normal((ogo.num_voxels, c_out)).astype(np.float32), "bf16")
    d_x, d_w, d_gy = (H.to_device_storage(a, "bf16") for a in (feat, wt, gy))
    y = fx.sparse_conv_fwd(km, d_x, d_w).float().cpu().numpy()
    H.conv_tolerance_check(y, O.conv(og, ogo, K, stride, feat, wt), "bf16", K ** 3, c_in)
    gw = fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32).cpu().numpy()
    ref = O.conv_bwd_weight(og, ogo, K, stride, feat, gy)
    num = np.sqrt(((gw - ref) ** 2).sum(axis=(1, 2)))
    den = np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))
    assert (num / den).max() <= 2e-3


def _same_non_finite(y, ref):
    """Infinities and NaN exactly where the reference has them; returns the elements that are finite in both."""
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(ref), ref, 0), np.where(np.isinf(y), y, 0))
    return np.isfinite(ref)


@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 4, 32), ("bf16", 3, 40), ("bf16", 8, 100), ("f16", 16, 64)])
@pytest.mark.parametrize("backward", [False, True])
def test_non_finite_weights_reach_only_the_rows_with_that_tap(dtype, c_in, c_out, backward):
    # a sum runs over existing neighbours: an infinite or NaN weight of one offset must not turn rows without a neighbour
    # there into NaN (0 * inf).  One output column holds the infinity, another the NaN; the rest stay finite everywhere.
    pts = _cloud(700)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(41, og.num_voxels, c_in, c_out, 27, dtype)
    wt[3, 0, 5] = np.inf
    wt[22, c_in - 1, c_out - 1] = np.nan
    d_x = H.to_device_storage(feat, dtype)
    if backward:
        wt_b = np.ascontiguousarray(wt.transpose(0, 2, 1))
        y = fx.sparse_conv_bwd_data(km, d_x, H.to_device_storage(wt_b, dtype), out_dtype=torch.float32)
        ref = O.conv_bwd_data(og, og, 3, 1, feat, wt_b)
    else:
        y = fx.sparse_conv_fwd(km, d_x, H.to_device_storage(wt, dtype), out_dtype=torch.float32)
        ref = O.conv(og, og, 3, 1, feat, wt)
    y = y.cpu().numpy()
    ok = _same_non_finite(y, ref)
    assert 0 < (~ok).sum() < 2 * og.num_voxels
    assert np.abs(y[ok] - ref[ok]).max() <= 1e-4 * np.sqrt(27 * c_in)


@pytest.mark.parametrize("n", [200, 3000])
@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 4, 32), ("bf16", 3, 40), ("bf16", 8, 100), ("f16", 16, 31), ("bf16", 16, 64)])
def test_non_finite_output_gradients_reach_only_the_offsets_their_voxels_have(n, dtype, c_in, c_out):
    # 0 * inf is NaN: infinities and NaN in gout must not reach the weight gradient of offsets where their voxel has no
    # neighbour.  A few columns hold one, one column is not finite anywhere, the others stay finite.
    pts = _cloud(n)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, 3, 1)
    feat, _ = G.features_and_weights(43, og.num_voxels, c_in, c_out, 27, dtype)
    gy = G.round_to_dtype(np.random.default_rng(44).standard_normal((og.num_voxels, c_out)).astype(np.float32), dtype)
    gy[og.num_voxels // 2, 3] = np.inf
    gy[0, 9] = -np.inf
    gy[og.num_voxels - 1, c_out - 1] = np.nan
    gy[:, 17] = np.inf
    gw = H.nan_filled((27, c_in, c_out), torch.float32)
    fx.sparse_conv_bwd_weight(km, H.to_device_storage(feat, dtype), H.to_device_storage(gy, dtype), out_dtype=torch.float32, out=gw)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    y = gw.cpu().numpy()
    ok = _same_non_finite(y, ref)
    assert ok[:, :, [3, 9, c_out - 1]].any() and not ok[:, :, [3, 9, c_out - 1]].all()
    num = np.sqrt((np.subtract(y, ref, where=ok, out=np.zeros_like(ref)) ** 2).sum(axis=(1, 2)))
    den = np.maximum(np.sqrt((np.where(ok, ref, 0) ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))
    assert (num / den).max() <= 2e-3


def test_weight_gradient_of_many_columns_over_fewer_ranges():
    # 16 -> 256: the partial sums are limited to 64 MB, 128 ranges on 256 compute units, which 33 k rows reach
    pts = np.unique(np.random.default_rng(45).integers(-24, 24, size=(60_000, 3)).astype(np.int32), axis=0)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    assert og.num_voxels > 33_000
    km = fx.build_kernel_map(g, 3, 1)
    feat, _ = G.features_and_weights(46, og.num_voxels, 16, 256, 27, "bf16")
    gy = G.round_to_dtype(np.random.default_rng(47).standard_normal((og.num_voxels, 256)).astype(np.float32), "bf16")
    d_x, d_gy = H.to_device_storage(feat, "bf16"), H.to_device_storage(gy, "bf16")
    gw = H.nan_filled((27, 16, 256), torch.float32)
    fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32, out=gw)
    ref = O.conv_bwd_weight(og, og, 3, 1, feat, gy)
    num = np.sqrt(((gw.cpu().numpy() - ref) ** 2).sum(axis=(1, 2)))
    assert (num / np.sqrt((ref ** 2).sum(axis=(1, 2)))).max() <= 2e-3
    assert torch.equal(gw, fx.sparse_conv_bwd_weight(km, d_x, d_gy, out_dtype=torch.float32))

"""GPU parity: sparse convolution forward against the oracle, within the stated tolerances."""
import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx
from oracle import cpu_oracle as O
from workloads import generators as G

pytestmark = pytest.mark.gpu


def _run(w: G.Workload, out_f32=False, c_in=None, c_out=None, dtype=None, dup=0.01):
    c_in, c_out, dtype = c_in or w.c_in, c_out or w.c_out, dtype or w.dtype
    ijk, jo = w.jagged_ijk(dup_fraction=dup)
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, w.kernel_size, w.stride)
    ogo = O.output_grid(og, w.kernel_size, w.stride)
    feat, wt = G.features_and_weights(w.feat_seed, og.num_voxels, c_in, c_out, w.k3, dtype)
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype),
                           out_dtype=torch.float32 if out_f32 else None)
    ref = O.conv(og, ogo, w.kernel_size, w.stride, feat, wt)
    return y.float().cpu().numpy(), ref, dtype, w.k3, c_in


def test_config1_sphere_fp32():
    y, ref, dt, k3, c_in = _run(G.workload("sphere64"))
    H.conv_tolerance_check(y, ref, dt, k3, c_in)


@pytest.mark.parametrize("name", ["indoor_small", "lidar_small", "lidar_small_down"])
@pytest.mark.parametrize("out_f32", [False, True])
def test_mfma_path_small_workloads(name, out_f32):
    y, ref, dt, k3, c_in = _run(G.workload(name), out_f32=out_f32)
    H.conv_tolerance_check(y, ref, dt, k3, c_in)


@pytest.mark.parametrize("name", ["lidar_small", "lidar_small_down", "sheets_small", "indoor_small"])
@pytest.mark.parametrize("gather", ["0", "1"])
def test_both_mfma_kernels_serve_every_map(name, gather, fx_opt):
    # by default strided maps take the gather kernel and the others the LDS-staged kernel; each kernel
    # must also be right on the other kind of map
    fx_opt("conv_gather", gather)
    y, ref, dt, k3, c_in = _run(G.workload(name))
    H.conv_tolerance_check(y, ref, dt, k3, c_in)


@pytest.mark.parametrize("lds_weights", ["0", "1", "-1"])
def test_gather_kernel_with_and_without_weights_in_lds(lds_weights, fx_opt):
    # strided maps: by default the packed weights of one or two output slices sit in LDS when they fit
    # (64 -> 128 and 32 -> 256: two slices; 32 -> 64 and 64 -> 192: one); the switch sends the same map to
    # the one-slice form or to the kernel that fetches them per step
    fx_opt("gather_lds", lds_weights)
    for name, c_in, c_out in (("lidar_small_down", 64, 128), ("lidar_small_down", 32, 64), ("lidar_small_down", 32, 256),
                              ("lidar_small_down", 64, 192), ("sheets_small", 32, 64)):
        if name == "sheets_small":
            fx_opt("conv_gather", "1")      # K = 3: 27 x 32 channels no longer fit, falls back
        y, ref, dt, k3, ci = _run(G.workload(name), c_in=c_in, c_out=c_out, dtype="bf16")
        H.conv_tolerance_check(y, ref, dt, k3, ci)


def test_mfma_path_deep_channels():
    y, ref, dt, k3, c_in = _run(G.workload("sheets_small"))
    H.conv_tolerance_check(y, ref, dt, k3, c_in)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("c_in,c_out", [(64, 192), (128, 64), (32, 64), (48, 40), (8, 16)])
def test_channel_shapes_mfma_and_scalar(dtype, c_in, c_out):
    y, ref, dt, k3, ci = _run(G.workload("sheets_small"), c_in=c_in, c_out=c_out, dtype=dtype)
    H.conv_tolerance_check(y, ref, dt, k3, ci)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 32, 40), ("f16", 64, 34), ("bf16", 96, 2), ("f32", 16, 16),
                                             ("f32", 32, 96), ("f32", 48, 6), ("f32", 64, 64)])
@pytest.mark.parametrize("name", ["sheets_small", "lidar_small_down"])
def test_tile_kernel_with_fp32_rows_and_padded_output_channels(name, dtype, c_in, c_out, fx_opt):
    # input rows in whole 64-byte chunks (32 channels of a 16-bit type, 16 of fp32) and an even number
    # of output channels run on the matrix units; fp32 keeps true fp32 products (the fp32 bar applies).
    # Small fp32 grids go to the scalar kernel by default; the switch sends them to the tile kernel.
    fx_opt("fp32_tiles", "1")
    y, ref, dt, k3, ci = _run(G.workload(name), c_in=c_in, c_out=c_out, dtype=dtype)
    H.conv_tolerance_check(y, ref, dt, k3, ci)


@pytest.mark.parametrize("K,dtype,c_in,c_out", [(1, "bf16", 64, 64), (1, "f16", 32, 128), (5, "bf16", 16, 16),
                                               (5, "f32", 8, 8)])
def test_pointwise_and_5x5x5_kernels(K, dtype, c_in, c_out):
    # K = 1 runs the tiled MFMA path with a single offset (a per-voxel GEMM); K = 5 (125 offsets)
    # keeps a dense map and takes the scalar path
    pts = np.random.default_rng(3).integers(-20, 40, size=(6000, 3)).astype(np.int32)
    g, og = H.both_grids(pts, np.array([[0, 2500], [2500, 6000]], np.int64))
    km = fx.build_kernel_map(g, K, 1)
    feat, wt = G.features_and_weights(17, og.num_voxels, c_in, c_out, K ** 3, dtype)
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype))
    ref = O.conv(og, og, K, 1, feat, wt)
    H.conv_tolerance_check(y.float().cpu().numpy(), ref, dtype, K ** 3, c_in)
    if K == 1:
        # K = 1 is out = in . W[0] (closed form, independent of the map code)
        closed = feat.astype(np.float64) @ wt[0].astype(np.float64)
        H.conv_tolerance_check(y.float().cpu().numpy(), closed, dtype, 1, c_in)


@pytest.mark.parametrize("tiles", ["0", "1", "scalar"])
def test_fp32_scalar_and_tile_kernels_on_config1(tiles, fx_opt):
    # 0: one wave per 16 voxels, 1: the tile kernel, scalar: neither
    if tiles == "scalar":
        fx_opt("force_scalar", "1")
    else:
        fx_opt("fp32_tiles", tiles)
    w = G.workload("sphere64")
    fx.profile_enable(True)
    fx.profile_reset()
    y, ref, dt, k3, c_in = _run(w)
    ran = fx.profile_read()
    fx.profile_enable(False)
    assert {"0": "k_conv_gather", "1": "k_conv_mfma", "scalar": "k_conv_scalar"}[tiles] in ran
    H.conv_tolerance_check(y, ref, dt, k3, c_in)


def test_fp32_full_size_takes_the_tile_kernel():
    """Config 3's grid with fp32 features, 32 -> 32 channels: large enough for the fp32 matrix path
    by default; sampled output rows against the oracle at the fp32 bar."""
    w = G.workload("lidar1m")
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(31, og.num_voxels, 32, 32, 27, "f32")
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, "f32"), H.to_device_storage(wt, "f32")).cpu().numpy()
    n = og.num_voxels
    for s in (0, n // 2, n - 300):
        ref = O.conv(og, og, 3, 1, feat.astype(np.float64), wt.astype(np.float64), s, s + 300)
        H.conv_tolerance_check(y[s:s + 300], ref[s:s + 300], "f32", 27, 32)


@pytest.mark.parametrize("dtype,c_in,c_out", [("bf16", 64, 128), ("f16", 32, 64), ("f32", 16, 8), ("bf16", 24, 10)])
def test_3x3x3_stride_2(dtype, c_in, c_out):
    # output grid = the coarse grid of the 2x2x2 case, output p reads 2p + {-1,0,1}^3; the windows of
    # neighbouring outputs overlap, so an input row is used by up to 8 outputs
    w = G.workload("lidar_small")
    ijk, jo = w.jagged_ijk(dup_fraction=0.01)
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 2)
    ogc = og.coarsen2()
    feat, wt = G.features_and_weights(71, og.num_voxels, c_in, c_out, 27, dtype)
    d_x, d_w = H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype)
    y = fx.sparse_conv_fwd(km, d_x, d_w)
    H.conv_tolerance_check(y.float().cpu().numpy(), O.conv(og, ogc, 3, 2, feat, wt), dtype, 27, c_in)
    # weight gradient on the same map
    gy = G.round_to_dtype(np.random.default_rng(72).standard_normal((ogc.num_voxels, c_out)).astype(np.float32), dtype)
    gw = fx.sparse_conv_bwd_weight(km, d_x, H.to_device_storage(gy, dtype), out_dtype=torch.float32).cpu().numpy()
    ref = O.conv_bwd_weight(og, ogc, 3, 2, feat, gy)
    num = np.sqrt(((gw - ref) ** 2).sum(axis=(1, 2)))
    den = np.maximum(np.sqrt((ref ** 2).sum(axis=(1, 2))), 1e-3 * np.sqrt(c_in * c_out))
    assert (num / den).max() <= (1e-4 if dtype == "f32" else 2e-3)
    # input gradient and transposed convolution: an input is shared by up to 8 outputs, both gather
    # through the inverse table of the map
    gx = fx.sparse_conv_bwd_data(km, H.to_device_storage(gy, dtype), d_w).float().cpu().numpy()
    H.conv_tolerance_check(gx, O.conv_bwd_data(og, ogc, 3, 2, gy, wt), dtype, 27, c_out)
    _, wt_t = G.features_and_weights(73, 1, c_out, c_in, 27, dtype)          # [27, c_out, c_in]: coarse c_out -> fine c_in
    up = fx.sparse_conv_transpose_fwd(km, H.to_device_storage(gy, dtype), H.to_device_storage(wt_t, dtype))
    assert up.shape == (og.num_voxels, c_in)
    H.conv_tolerance_check(up.float().cpu().numpy(), O.conv_transpose(og, ogc, 3, 2, gy, wt_t), dtype, 27, c_out)


@pytest.mark.parametrize("lds_weights", ["0", "1"])
@pytest.mark.parametrize("dtype,c_in,c_out", [("f32", 8, 16), ("bf16", 8, 16), ("f16", 4, 32), ("f32", 12, 8)])
def test_low_depth_scalar_kernel_with_and_without_weights_in_lds(dtype, c_in, c_out, lds_weights, fx_opt):
    # depths the matrix kernels do not take on a sparse grid: the scalar kernel, weights in LDS by default
    fx_opt("scalar_lds", lds_weights)
    fx_opt("leaf_dispatch", "0")
    for name in ("lidar_small", "lidar_small_down"):
        y, ref, dt, k3, ci = _run(G.workload(name), c_in=c_in, c_out=c_out, dtype=dtype)
        H.conv_tolerance_check(y, ref, dt, k3, ci)


def test_identity_tap_is_bit_exact_in_bf16():
    w = G.workload("lidar_small")
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    nb = O.kernel_map(og, og, 3, 1)
    feat = G.round_to_dtype(np.random.default_rng(5).standard_normal((og.num_voxels, 64)).astype(np.float32), "bf16")
    d_feat = H.to_device_storage(feat, "bf16")
    for kappa in (0, 13, 20):
        wt = np.zeros((27, 64, 64), dtype=np.float32)
        wt[kappa] = np.eye(64)
        y = fx.sparse_conv_fwd(km, d_feat, H.to_device_storage(wt, "bf16")).float().cpu().numpy()
        expect = np.where(nb[:, kappa:kappa + 1] >= 0, feat[np.maximum(nb[:, kappa], 0)], 0.0)
        assert np.array_equal(y, expect)


@pytest.mark.parametrize("lds_weights", ["-1", "1", "0"])
def test_identity_taps_on_a_strided_map_are_bit_exact(lds_weights, fx_opt):
    # 2x2x2 stride 2, 64 -> 128: W[kappa] = [I | 2 I] for one offset copies the child's row into both output slices
    # (every gather kernel: two slices per workgroup, one, weights fetched per step); then the input gradient and
    # the transposed convolution of the same map with one-offset weights, which copy parents' rows to children
    fx_opt("gather_lds", lds_weights)
    w = G.workload("lidar_small_down")
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 2, 2)
    ogc = og.coarsen2()
    nb = O.kernel_map(og, ogc, 2, 2)
    feat = G.round_to_dtype(np.random.default_rng(6).standard_normal((og.num_voxels, 64)).astype(np.float32), "bf16")
    d_feat = H.to_device_storage(feat, "bf16")
    for kappa in (0, 3, 7):
        wt = np.zeros((8, 64, 128), dtype=np.float32)
        wt[kappa, :, :64] = np.eye(64)
        wt[kappa, :, 64:] = 2.0 * np.eye(64)
        y = fx.sparse_conv_fwd(km, d_feat, H.to_device_storage(wt, "bf16")).float().cpu().numpy()
        child = np.where(nb[:, kappa:kappa + 1] >= 0, feat[np.maximum(nb[:, kappa], 0)], 0.0)
        assert np.array_equal(y, np.concatenate([child, 2.0 * child], axis=1))
    gy = G.round_to_dtype(np.random.default_rng(7).standard_normal((ogc.num_voxels, 128)).astype(np.float32), "bf16")
    d_gy = H.to_device_storage(gy, "bf16")
    for kappa in (1, 6):
        # input gradient: gin[child] = W[kappa] . gout[parent] = first half of the parent's row for children at kappa
        wt = np.zeros((8, 64, 128), dtype=np.float32)
        wt[kappa, :, :64] = np.eye(64)
        gx = fx.sparse_conv_bwd_data(km, d_gy, H.to_device_storage(wt, "bf16")).float().cpu().numpy()
        expect = np.zeros((og.num_voxels, 64), dtype=np.float32)
        has = nb[:, kappa] >= 0
        expect[nb[has, kappa]] = gy[has, :64]
        assert np.array_equal(gx, expect)
        # transposed convolution 128 -> 64 with W[kappa] = [0 ; I]: the second half of the parent's row
        wtt = np.zeros((8, 128, 64), dtype=np.float32)
        wtt[kappa, 64:, :] = np.eye(64)
        up = fx.sparse_conv_transpose_fwd(km, d_gy, H.to_device_storage(wtt, "bf16")).float().cpu().numpy()
        expect = np.zeros((og.num_voxels, 64), dtype=np.float32)
        expect[nb[has, kappa]] = gy[has, 64:]
        assert np.array_equal(up, expect)


def test_all_ones_counts_neighbours_exactly_in_f16():
    w = G.workload("sheets_small")
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    nb = O.kernel_map(og, og, 3, 1)
    ones_f = torch.ones((og.num_voxels, 64), dtype=torch.float16, device="cuda")
    ones_w = torch.ones((27, 64, 64), dtype=torch.float16, device="cuda")
    y = fx.sparse_conv_fwd(km, ones_f, ones_w).float().cpu().numpy()
    assert np.array_equal(y, np.repeat(64.0 * (nb >= 0).sum(1)[:, None], 64, axis=1))


def test_scalar_and_mfma_paths_agree_with_oracle_on_empty_and_tiny_grids():
    g, og = H.both_grids(np.zeros((0, 3), np.int32), np.array([[0, 0]], np.int64))
    km = fx.build_kernel_map(g, 3, 1)
    y = fx.sparse_conv_fwd(km, torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda"),
                           torch.zeros((27, 64, 64), dtype=torch.bfloat16, device="cuda"))
    assert y.shape == (0, 64)
    pts = np.array([[0, 0, 0], [0, 0, 1], [5, 5, 5], [-1, 0, 0]], dtype=np.int32)   # a single partial tile
    g, og = H.both_grids(pts, np.array([[0, 4]], np.int64))
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(7, 4, 64, 64, 27, "bf16")
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, "bf16"), H.to_device_storage(wt, "bf16"))
    H.conv_tolerance_check(y.float().cpu().numpy(), O.conv(og, og, 3, 1, feat, wt), "bf16", 27, 64)


def test_dense_block_uses_rows_beyond_the_lds_budget(fx_opt):
    # a dense 24^3 block: every tile is one full leaf whose 10^3 footprint has more distinct
    # input rows than the convolution stages in LDS, so part of them is read from global memory
    fx_opt("leaf_dispatch", "0")      # this test is about the tile kernel's general variant
    a = np.arange(24, dtype=np.int32)
    pts = np.stack(np.meshgrid(a, a, a, indexing="ij"), axis=-1).reshape(-1, 3)
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(11, og.num_voxels, 64, 64, 27, "bf16")
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, "bf16"), H.to_device_storage(wt, "bf16"))
    H.conv_tolerance_check(y.float().cpu().numpy(), O.conv(og, og, 3, 1, feat, wt), "bf16", 27, 64)


@pytest.mark.parametrize("name", ["lidar1m", "indoor4", "lidar1m_down", "sheets4", "volume1m_c64", "dense96",
                                  "volume1m_c64:tiles", "dense96:tiles"])
def test_full_size_configs_sampled_rows(name, fx_opt):
    """Configs 3, 2, 4 and 5 at full size in the benchmark's launch configuration; the oracle
    computes a sample of output rows one by one (a few thousand rows spread over the grid, the
    first and the last rows included).  The volumetric and the dense grid run twice: through the
    leaf-window kernels, which the convolution picks for them, and (":tiles") through the tile kernel."""
    if name.endswith(":tiles"):
        fx_opt("leaf_dispatch", "0")
        name = name[:-6]
    w = G.workload(name)
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, w.kernel_size, w.stride)
    ogo = O.output_grid(og, w.kernel_size, w.stride)
    assert km.n_out == ogo.num_voxels
    feat, wt = w.feats_weights()
    y = fx.sparse_conv_fwd(km, H.to_device_storage(feat, w.dtype), H.to_device_storage(wt, w.dtype))
    y = y.float().cpu().numpy()
    n = ogo.num_voxels
    starts = list(range(0, n - 300, n // 12)) + [n - 300]
    f64, w64 = feat.astype(np.float64), wt.astype(np.float64)
    for s in starts:
        ref = O.conv(og, ogo, w.kernel_size, w.stride, f64, w64, s, s + 300)
        H.conv_tolerance_check(y[s:s + 300], ref[s:s + 300], w.dtype, w.k3, w.c_in)


# The 16-bit path's own error model (exact products, fp32 accumulation of <= K^3*C_in terms, one rounding to an
# 8-bit significand) puts the per-row relative error near 2^-9 = 2e-3 for bf16 outputs and ~1e-6 for fp32 outputs;
# the asserted bar stays the stated 2e-2, the figure below is printed so that a drift towards it shows in the log.
def _report(tag, y, ref):
    print(f"[row-error] {tag}: max per-row relative L2 error {H.row_error_report(y, ref):.3e}", flush=True)


@pytest.mark.parametrize("name", ["lidar1m", "lidar1m_down", "sheets4", "indoor4"])
def test_full_size_every_output_row(name):
    """Configs 3, 4, 5 and 2 at full size in the benchmark's launch configuration, every output row against the
    oracle.  The output buffer starts as NaN, so a row that no workgroup wrote fails; a tile claimed twice or
    skipped by the persistent kernel's work lists cannot hide among sampled rows."""
    w = G.workload(name)
    ijk, jo = w.jagged_ijk()
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, w.kernel_size, w.stride)
    ogo = O.output_grid(og, w.kernel_size, w.stride)
    assert km.n_out == ogo.num_voxels
    feat, wt = w.feats_weights()
    out = H.nan_filled((km.n_out, w.c_out), H.TORCH_DT[w.dtype])
    fx.sparse_conv_fwd(km, H.to_device_storage(feat, w.dtype), H.to_device_storage(wt, w.dtype), out=out)
    y = out.float().cpu().numpy()
    assert np.isfinite(y).all()
    ref = O.conv(og, ogo, w.kernel_size, w.stride, feat, wt, threads=H.ORACLE_THREADS)
    _report(name, y, ref)
    H.conv_tolerance_check(y, ref, w.dtype, w.k3, w.c_in)


@pytest.mark.parametrize("dtype,out_f32", [("bf16", False), ("f16", True)])
def test_many_work_items_per_workgroup_under_a_full_compare(dtype, out_f32):
    """196 tiles x 8 output slices = 1568 work items on at most 256 persistent workgroups: every workgroup claims
    several items through the per-XCD counters, announces them in the LDS ring and hands its weight pipeline from
    item to item -- all compared row by row, outputs NaN before the call."""
    w = G.workload("lidar_small")
    ijk, jo = w.jagged_ijk(dup_fraction=0.01)
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(9100, og.num_voxels, 64, 512, 27, dtype)
    odt = torch.float32 if out_f32 else H.TORCH_DT[dtype]
    out = H.nan_filled((km.n_out, 512), odt)
    fx.sparse_conv_fwd(km, H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype), out_dtype=odt, out=out)
    y = out.float().cpu().numpy()
    assert np.isfinite(y).all()
    ref = O.conv(og, og, 3, 1, feat, wt, threads=H.ORACLE_THREADS)
    _report(f"lidar_small 64->512 {dtype}", y, ref)
    H.conv_tolerance_check(y, ref, dtype, 27, 64)
    # identity tap on the same launch shape: bit-exact rows, so a row written by the wrong item shows
    wid = np.zeros((27, 64, 512), dtype=np.float32)
    for s in range(8):
        wid[(3 * s + 1) % 27, :, 64 * s:64 * s + 64] = np.eye(64)
    out.fill_(float("nan"))
    fx.sparse_conv_fwd(km, H.to_device_storage(feat, dtype), H.to_device_storage(wid, dtype), out_dtype=odt, out=out)
    y = out.float().cpu().numpy()
    nb = O.kernel_map(og, og, 3, 1)
    for s in range(8):
        col = nb[:, (3 * s + 1) % 27]
        expect = np.where(col[:, None] >= 0, feat[np.maximum(col, 0)], 0.0)
        assert np.array_equal(y[:, 64 * s:64 * s + 64], expect)


def _one_voxel_leaves(n_side=13, seed=4242):
    """A lattice of leaves with ONE active voxel each (random position inside its leaf): every tile of 512
    consecutive outputs spans 512 different leaves -- the densest leaf list a tile can have."""
    rng = np.random.default_rng(seed)
    a = np.arange(n_side, dtype=np.int32) - n_side // 2
    leaf = np.stack(np.meshgrid(a, a, a, indexing="ij"), axis=-1).reshape(-1, 3) * 8
    return (leaf + rng.integers(0, 8, size=leaf.shape)).astype(np.int32)


@pytest.mark.parametrize("K,stride", [(3, 1), (2, 2), (3, 2), (1, 1)])
def test_tiles_of_512_one_voxel_leaves(K, stride):
    """2197 voxels in 2197 leaves (four full tiles and a tail): the map is compared entry by entry and the
    convolution row by row; slot 511 of a full tile lies in the tile's 512th leaf."""
    pts = _one_voxel_leaves()
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]], np.int64))
    assert g.counts()[0] == pts.shape[0] == og.num_voxels
    km = fx.build_kernel_map(g, K, stride)
    ogo = O.output_grid(og, K, stride)
    assert np.array_equal(km.dense().cpu().numpy(), O.kernel_map(og, ogo, K, stride))
    feat, wt = G.features_and_weights(4243, og.num_voxels, 64, 64, K ** 3, "bf16")
    out = H.nan_filled((km.n_out, 64), torch.bfloat16)
    fx.sparse_conv_fwd(km, H.to_device_storage(feat, "bf16"), H.to_device_storage(wt, "bf16"), out=out)
    H.conv_tolerance_check(out.float().cpu().numpy(), O.conv(og, ogo, K, stride, feat, wt), "bf16", K ** 3, 64)
    if (K, stride) == (3, 2):           # the inverse map's tiles list leaves of the fine grid the same way
        gy = G.round_to_dtype(np.random.default_rng(4244).standard_normal((ogo.num_voxels, 64)).astype(np.float32), "bf16")
        gx = fx.sparse_conv_bwd_data(km, H.to_device_storage(gy, "bf16"), H.to_device_storage(wt, "bf16"))
        H.conv_tolerance_check(gx.float().cpu().numpy(), O.conv_bwd_data(og, ogo, K, stride, gy, wt), "bf16", 27, 64)


@pytest.mark.parametrize("corner", [-2000, 1000])
@pytest.mark.parametrize("dims,c_in,c_out", [((40, 24, 8), 32, 512), ((40, 24, 8), 96, 320), ((26, 26, 26), 32, 512)])
def test_long_tiles_among_more_items_than_workgroups(corner, dims, c_in, c_out, fx_opt):
    # a cloud with one solid block, in the first or in the last tiles: a few tiles whose rows are not all staged start
    # first, their workgroups' own items are claimed by others, claims pass the long ones over (40 x 24 x 8, with one and
    # with several phases an item); more of them than are listed leave the order alone (26^3).  Every row is written once.
    fx_opt("leaf_dispatch", "0")
    rng = np.random.default_rng(500 + dims[0])
    cloud = rng.integers(-300, 300, size=(40000, 3)).astype(np.int32)
    ax = [np.arange(d, dtype=np.int32) + corner for d in dims]
    block = np.stack(np.meshgrid(*ax, indexing="ij"), axis=-1).reshape(-1, 3)
    pts = np.concatenate([cloud, block])[rng.permutation(40000 + block.shape[0])]
    g, og = H.both_grids(pts, np.array([[0, pts.shape[0]]]))
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(21, og.num_voxels, c_in, c_out, 27, "bf16")
    d_x, d_w = H.to_device_storage(feat, "bf16"), H.to_device_storage(wt, "bf16")
    y = H.nan_filled((og.num_voxels, c_out), torch.bfloat16)
    fx.sparse_conv_fwd(km, d_x, d_w, out=y)
    y = y.float().cpu().numpy()
    fx_opt("force_scalar", "1")                    # every row against the scalar kernel, some against the oracle
    H.conv_tolerance_check(y, fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32).cpu().numpy(), "bf16", 27, c_in)
    for s in list(range(0, og.num_voxels - 300, 6000)) + [og.num_voxels - 300]:
        H.conv_tolerance_check(y[s:s + 300], O.conv(og, og, 3, 1, feat, wt, s, s + 300)[s:s + 300], "bf16", 27, c_in)


@pytest.mark.parametrize("dtype,out_f32", [("f16", False), ("bf16", True)])
@pytest.mark.parametrize("c_in,c_out", [(32, 2), (32, 32), (96, 34), (64, 40), (32, 96), (64, 160)])
def test_slices_of_32_output_channels(dtype, out_f32, c_in, c_out):
    # few tiles, or up to 32 channels: work items of 32 channels, whole, partial and past the last whole slice of 64
    w = G.workload("sheets_small")
    ijk, jo = w.jagged_ijk(dup_fraction=0.0)
    g, og = H.both_grids(ijk, jo)
    km = fx.build_kernel_map(g, 3, 1)
    feat, wt = G.features_and_weights(23, og.num_voxels, c_in, c_out, 27, dtype)
    y = H.nan_filled((og.num_voxels, c_out), torch.float32 if out_f32 else H.TORCH_DT[dtype])
    fx.sparse_conv_fwd(km, H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype), out_dtype=y.dtype, out=y)
    H.conv_tolerance_check(y.float().cpu().numpy(), O.conv(og, og, 3, 1, feat, wt), dtype, 27, c_in)


@pytest.mark.parametrize("corner", [-2000, 1000])
@pytest.mark.parametrize("dtype,c_in,c_out,cloud", [("bf16", 32, 512, 40000), ("bf16", 96, 320, 40000), ("f32", 32, 320, 40000), ("bf16", 48, 320, 40000),
                                                    ("f16", 32, 32, 180000), ("bf16", 40, 24, 180000), ("f16", 64, 128, 660000)])
def test_long_tiles_first_every_row(dtype, c_in, c_out, cloud, corner, fx_opt):
    # long tiles start first: slices of 64 and of 32 channels, fp32, rows that end inside a chunk, with one to some ten items
    # a workgroup.  Every row against the scalar kernel, the first, last and some other rows against the oracle.
    fx_opt("leaf_dispatch", "0")
    rng = np.random.default_rng(520 + cloud)
    pts = rng.integers(-300, 300, size=(cloud, 3)).astype(np.int32)
    ax = [np.arange(d, dtype=np.int32) + corner for d in (40, 24, 8)]
    pts = np.concatenate([pts, np.stack(np.meshgrid(*ax, indexing="ij"), axis=-1).reshape(-1, 3)])
    g, og = H.both_grids(pts[rng.permutation(pts.shape[0])], np.array([[0, pts.shape[0]]]))
    n, km = og.num_voxels, fx.build_kernel_map(g, 3, 1)
    # the call is on the path: tiles whose rows (their own and the neighbours outside) are more than fit in LDS
    table, own = km.dense().cpu().numpy(), np.arange(512)
    n_tiles = (n + 511) // 512
    n_long = sum(np.union1d(table[512 * t:512 * t + 512].ravel(), own + 512 * t).size - 1 > 792 for t in range(n_tiles))
    n_slices, half = (c_out + (31 if c_out <= 32 else 63)) // (32 if c_out <= 32 else 64), torch.cuda.get_device_properties(0).multi_processor_count // 2
    assert 0 < n_long <= 32 and n_long * n_slices <= half < 2 * half < n_tiles * n_slices
    feat, wt = G.features_and_weights(33, n, c_in, c_out, 27, dtype)
    d_x, d_w = H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype)
    y = fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32, out=H.nan_filled((n, c_out), torch.float32))
    fx_opt("force_scalar", "1")
    ref = fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32)
    # both sum the same products in 32 bits, of a sum with unit variance: 27 * c_in roundings of partial sums below 8 each
    assert ((y - ref).abs().amax(1) <= 2 * 27 * c_in * 2.0 ** -24 * 8).all()
    for s in [0] + list(range(20000, n - 300, 60000)) + [n - 300]:
        H.conv_tolerance_check(y[s:s + 300].cpu().numpy(), O.conv(og, og, 3, 1, feat, wt, s, s + 300)[s:s + 300], "f32" if dtype == "f32" else dtype, 27, c_in)


@pytest.mark.parametrize("dtype,c_in,c_out,cloud", [("bf16", 32, 512, 40000), ("bf16", 96, 320, 40000), ("f32", 32, 320, 40000), ("bf16", 48, 320, 40000),
                                                    ("f16", 32, 32, 180000), ("bf16", 40, 24, 180000), ("f16", 64, 128, 660000)])
def test_long_tiles_of_a_block_before_a_cloud_first(dtype, c_in, c_out, cloud, fx_opt):
    # the same of tiles of more than 816 rows, which one half of the row buffer does not hold: in front of a cloud it takes a larger block,
    # behind one the block's tiles straddle its leaves.  Every row against the scalar kernel, the first, last and some other rows against the oracle.
    fx_opt("leaf_dispatch", "0")
    rng = np.random.default_rng(520 + cloud)
    pts = rng.integers(-300, 300, size=(cloud, 3)).astype(np.int32)
    pts = np.concatenate([pts, H.box((40, 24, 16), (-2000,) * 3).astype(np.int32)])
    g, og = H.both_grids(pts[rng.permutation(pts.shape[0])], np.array([[0, pts.shape[0]]]))
    n, km = og.num_voxels, fx.build_kernel_map(g, 3, 1)
    # the call is on the path: tiles whose rows (their own and the neighbours outside) are more than one half of the row buffer holds
    counts = H.tile_row_counts(km.dense().cpu().numpy())
    n_tiles, n_long = counts.size, int((counts > 816).sum())
    n_slices, half = (c_out + (31 if c_out <= 32 else 63)) // (32 if c_out <= 32 else 64), torch.cuda.get_device_properties(0).multi_processor_count // 2
    assert 0 < n_long <= 32 and n_long * n_slices <= half < 2 * half < n_tiles * n_slices
    feat, wt = G.features_and_weights(33, n, c_in, c_out, 27, dtype)
    d_x, d_w = H.to_device_storage(feat, dtype), H.to_device_storage(wt, dtype)
    y = fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32, out=H.nan_filled((n, c_out), torch.float32))
    fx_opt("force_scalar", "1")
    ref = fx.sparse_conv_fwd(km, d_x, d_w, out_dtype=torch.float32)
    # both sum the same products in 32 bits, of a sum with unit variance: 27 * c_in roundings of partial sums below 8 each
    assert ((y - ref).abs().amax(1) <= 2 * 27 * c_in * 2.0 ** -24 * 8).all()
    for s in [0] + list(range(20000, n - 300, 60000)) + [n - 300]:
        H.conv_tolerance_check(y[s:s + 300].cpu().numpy(), O.conv(og, og, 3, 1, feat, wt, s, s + 300)[s:s + 300], "f32" if dtype == "f32" else dtype, 27, c_in)

"""Weight gradient of wide layers (multiples of 256 channels on both sides) as a product over the pairs of an offset, against
the same sums in 64 bits: torch on the dense map, which other tests compare with the oracle.

Tolerance: a sum of N exact products in fp32, in any order, is off by about 2^-24 sqrt(N) of its size; N is at most 2e5
here, which gives 2.7e-5 of an offset's norm, and the bar is four times that."""
import ctypes as C
import gc

import numpy as np
import pytest
import torch

import gpu_common as H
import paper_2407_01781_amd as fx

pytestmark = pytest.mark.gpu


def _grid(n, seed, thick=0):
    """n random voxels, and a cube of `thick` voxels per side of which a third is there: its tiles need more rows than the
    tile kernels stage, its leaves are not dense enough for the leaf-window kernels."""
    rng = np.random.default_rng(seed)
    side = int(round(1.6 * n ** (1 / 3)))
    pts = [rng.integers(-side, side, size=(n, 3))]
    if thick:
        cube = np.stack(np.meshgrid(*[np.arange(thick)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) + 3 * side
        pts.append(cube[rng.random(cube.shape[0]) < 0.33])
    pts = np.unique(np.concatenate(pts).astype(np.int32), axis=0)
    return fx.build_index_grid(torch.from_numpy(pts[rng.permutation(pts.shape[0])]).cuda(), np.array([[0, pts.shape[0]]]))


def _reference(table, x, gy):
    gw = torch.zeros((table.shape[1], x.shape[1], gy.shape[1]), dtype=torch.float64, device="cuda")
    for k in range(table.shape[1]):
        o = (table[:, k] >= 0).nonzero()[:, 0]
        gw[k] = x[table[o, k].long()].double().t() @ gy[o].double()
    return gw


def _check(km, dtype, c_in, c_out, spoil=False):
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((km.g_in.num_voxels, c_in), generator=gen, device="cuda").to(H.TORCH_DT[dtype])
    gy = torch.randn((km.n_out, c_out), generator=gen, device="cuda").to(H.TORCH_DT[dtype])
    if spoil:
        x[km.g_in.num_voxels // 2, 1], gy[0, 5], gy[-1, c_out - 1] = float("inf"), float("-inf"), float("nan")
    gw = H.nan_filled((km.dense().shape[1], c_in, c_out), torch.float32)
    fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32, out=gw)
    ref = _reference(km.dense(), x, gy)
    ok = torch.isfinite(ref)
    assert bool(ok.all()) != spoil
    assert torch.equal(torch.isnan(gw), torch.isnan(ref)) and torch.equal(gw[torch.isinf(ref)].double(), ref[torch.isinf(ref)])
    diff = torch.where(ok, gw.double() - ref, 0.0).flatten(1).norm(dim=1)
    assert bool((diff <= 1.1e-4 * torch.where(ok, ref, 0.0).flatten(1).norm(dim=1)).all())
    assert torch.equal(gw.view(torch.int32), fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32).view(torch.int32))
    low = H.nan_filled(gw.shape, H.TORCH_DT[dtype])
    fx.sparse_conv_bwd_weight(km, x, gy, out=low)
    assert torch.equal(low.view(torch.int16), gw.to(H.TORCH_DT[dtype]).view(torch.int16)) or spoil


# 6 k outputs at four blocks and 24 k at one are the smallest sizes that come here; the last tile holds one voxel and more
@pytest.mark.parametrize("n,dtype,c_in,c_out", [(27_000, "bf16", 256, 256), (30_000, "f16", 256, 256), (14_500, "bf16", 256, 512), (7_000, "f16", 512, 512),
                                                (60_000, "bf16", 512, 256)])
@pytest.mark.parametrize("thick", [0, 24])
def test_block_counts(n, dtype, c_in, c_out, thick):
    g = _grid(n, n, thick)
    assert g.num_voxels * (c_in // 256) * (c_out // 256) >= 24_000
    _check(fx.build_kernel_map(g, 3, 1), dtype, c_in, c_out)


def test_other_maps():
    g = _grid(30_000, 5)
    _check(fx.build_kernel_map(g, 1, 1), "bf16", 256, 256)                  # one offset, every run has units of it
    _check(fx.build_kernel_map_onto(g, g.pad(1), 3), "f16", 256, 256)


@pytest.fixture
def nan_scratch():
    """The library's device memory from one arena of NaNs that is handed out once, so that what no kernel wrote shows."""
    arena, at = torch.full((100 << 20,), float("nan"), device="cuda"), [256]

    def take(nbytes, stream, ctx):
        at[0] += (nbytes + 255) // 256 * 256
        return arena.data_ptr() + at[0] - (nbytes + 255) // 256 * 256 if at[0] <= 4 * arena.numel() else None

    alloc = C.CFUNCTYPE(C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p)(take)
    free = C.CFUNCTYPE(None, C.c_void_p, C.c_void_p, C.c_void_p)(lambda p, stream, ctx: None)
    fx.binding._check(fx.binding.lib.fx_set_allocator(C.cast(alloc, C.c_void_p), C.cast(free, C.c_void_p), None))
    yield lambda: at[0]
    gc.collect()                                                            # maps and grids of the test go back before the arena does
    torch.cuda.synchronize()
    fx.binding._check(fx.binding.lib.fx_set_allocator(None, None, None))


@pytest.mark.parametrize("kernel,c_in,c_out", [(3, 256, 256), (1, 256, 256), (3, 512, 256)])
@pytest.mark.parametrize("touched", [0, 1, 2, 4, 5, 9, 10, 57])
def test_fewer_units_than_runs(touched, kernel, c_in, c_out, nan_scratch):
    """Two grids that meet in a few places only: inputs in the neighbourhood of `touched` of the output's 59 tiles, so that the pairs
    make fewer units than there are workgroups, or just as many."""
    out = np.stack(np.meshgrid(np.arange(62), np.arange(62), np.arange(8), indexing="ij"), axis=-1).reshape(-1, 3)[:30_000] * 2
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.int32))).cuda()
    g_out = fx.build_index_grid(dev(out), np.array([[0, out.shape[0]]]))
    at = g_out.ijk()[0].cpu().numpy()[512 * np.arange(touched) + 17]        # an output of each of those tiles, its neighbours, and something far off
    d = np.stack(np.meshgrid(*[np.arange(-1, 2)] * 3, indexing="ij"), axis=-1).reshape(1, 27, 3)
    pts = np.concatenate([np.unique((at[:, None] + d).reshape(-1, 3), axis=0), np.arange(-3000, -2000, 100)[:, None].repeat(3, axis=1)])
    km = fx.build_kernel_map_onto(fx.build_index_grid(dev(pts), np.array([[0, pts.shape[0]]])), g_out, kernel)
    t = (km.dense() >= 0).cpu().numpy()
    pairs = np.array([t[s:s + 512].sum(0) for s in range(0, t.shape[0], 512)])
    assert (pairs.sum(1) > 0).sum() >= touched and (touched or not pairs.any())
    runs = torch.cuda.get_device_properties(0).multi_processor_count // ((c_in // 256) * (c_out // 256))
    assert touched > 9 or kernel == 3 or ((pairs + 31) // 32).sum() < runs
    before = nan_scratch()
    _check(km, "bf16", c_in, c_out)
    assert nan_scratch() - before >= 3 * 4 * kernel ** 3 * c_in * c_out     # its scratch came from the arena


@pytest.mark.parametrize("kernel,spread,full,line,c_in,c_out", [(1, 3.0, 0, 40_000, 256, 256), (1, 3.0, 0, 10_000, 512, 512), (3, 6.0, 0, 32_000, 256, 256),
                                                                (3, 6.0, 0, 8_000, 512, 512), (3, 2.2, 0, 24_000, 256, 256), (3, 6.0, 1, 32_000, 256, 256),
                                                                (3, 6.0, 2, 24_000, 256, 256)])
@pytest.mark.parametrize("past", [0, 1])
def test_either_side_of_the_line(kernel, spread, full, line, c_in, c_out, past, nan_scratch):
    """A voxel fewer than the line, and as many: 1x1x1 maps, some two voxels a leaf, and some forty; full leaves with less and more
    than one voxel in 32.  The lists show by the size of their scratch memory, which the tile kernel's partial sums stay below."""
    n = line - 1 + past
    rng = np.random.default_rng(line + past)
    pts = np.unique(rng.integers(0, int(spread * n ** (1 / 3)), size=(2 * n, 3)), axis=0)
    leaves = np.stack(np.meshgrid(-17 - np.arange(8 * full), np.arange(8), np.arange(8), indexing="ij"), axis=-1).reshape(-1, 3)
    pts = np.ascontiguousarray(np.concatenate([leaves, rng.permutation(pts)[:n - len(leaves)]]).astype(np.int32))
    g = fx.build_index_grid(torch.from_numpy(pts).cuda(), np.array([[0, n]]))
    assert g.num_voxels == n and (n >= 8 * g.counts()[0]) == (spread < 4)
    km = fx.build_kernel_map(g, kernel, 1)
    x, gy = (torch.ones((n, c), dtype=torch.bfloat16, device="cuda") for c in (c_in, c_out))
    fx.sparse_conv_bwd_weight(km, x, gy)                                    # what the map keeps is there now
    before = nan_scratch()
    gw = fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32)
    jobs = (c_in // 256) * (c_out // 256)
    runs = torch.cuda.get_device_properties(0).multi_processor_count // jobs // 8 * 8
    assert (nan_scratch() - before >= 4 * jobs * (runs + kernel ** 3) * 256 * 256) == bool(past)
    assert torch.equal(gw, (km.dense() >= 0).sum(0).float()[:, None, None].expand_as(gw))


def test_pieces_longer_than_the_table():
    # 16 blocks leave 16 runs; every run has more than the 3072 units that are looked up at a time
    g = _grid(260_000, 6, 84)
    km = fx.build_kernel_map(g, 3, 1)
    assert int((km.dense() >= 0).sum()) > 16 * 3072 * 32
    _check(km, "bf16", 1024, 1024)


def test_values_that_are_not_finite_stay_with_their_pairs():
    _check(fx.build_kernel_map(_grid(30_000, 7), 3, 1), "bf16", 256, 256, spoil=True)

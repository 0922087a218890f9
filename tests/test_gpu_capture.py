"""A layer's forward pass and gradients recorded into a HIP graph, on maps of every route that decides by something counted or built
on a map's first call: after such a call, and as the map's first call.  Every replay against the same calls made directly, with direct
calls on the map in between."""
import gc

import numpy as np
import pytest
import torch

import paper_2407_01781_amd as fx

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def torch_memory():
    """The library's memory from PyTorch's allocator: a graph's own pool while it is recorded."""
    gc.collect()
    fx.use_torch_allocator(True)
    yield
    gc.collect()
    torch.cuda.synchronize()
    fx.use_torch_allocator(False)


def _index(pts):
    return fx.build_index_grid(torch.from_numpy(np.ascontiguousarray(pts.astype(np.int32))).cuda(), np.array([[0, pts.shape[0]]]))


def _box(*dims):
    return np.stack(np.meshgrid(*[np.arange(d) for d in dims], indexing="ij"), axis=-1).reshape(-1, 3)


def _cloud(n, side, seed):
    return np.unique(np.random.default_rng(seed).integers(0, side, size=(n, 3)), axis=0)


def _thinned(box, p):
    return box[np.random.default_rng(21).random(len(box)) < p]


GRIDS = {
    "cloud": lambda: _cloud(30_000, 90, 1),
    "tiles that are not staged": lambda: _thinned(_box(64, 48, 40), 0.37),
    "occupancy 0.7": lambda: _thinned(_box(48, 48, 48), 0.7),
    "occupancy 0.47": lambda: _thinned(_box(48, 48, 48), 0.47),
    "a cube with a ninth of the voxels": lambda: np.concatenate([_box(32, 32, 32), 200 + _cloud(269_000, 260, 12)]),
    "a cube with most of the voxels": lambda: np.concatenate([_box(32, 32, 32), 200 + _cloud(15_000, 100, 2)]),
}


@pytest.mark.parametrize("called_before", [True, False])
@pytest.mark.parametrize("name,c_in,c_out", [("cloud", 64, 64), ("cloud", 256, 256), ("tiles that are not staged", 64, 64), ("occupancy 0.47", 64, 128),
                                             ("a cube with a ninth of the voxels", 128, 128), ("a cube with most of the voxels", 64, 64),
                                             ("padded cloud", 64, 64), ("occupancy 0.7", 64, 64)])
def test_replays_of_a_layer(name, c_in, c_out, called_before):
    g = _index(GRIDS[name.replace("padded ", "")]())
    onto = name.startswith("padded")
    km = fx.build_kernel_map_onto(g, g.pad(1), 3) if onto else fx.build_kernel_map(g, 3, 1)
    gen = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda: [torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((g.num_voxels, c_in), (27, c_in, c_out), (km.n_out, c_out))]
    x, w, gy = draw()

    def layer(x, w, gy, km=km):
        y = fx.sparse_conv_fwd(km, x, w, out_dtype=torch.float32)
        # (between two grids the input gradient builds its map on the first call)
        gx = y if onto and not called_before else fx.sparse_conv_bwd_data(km, gy, w, out_dtype=torch.float32)
        return y, gx, fx.sparse_conv_bwd_weight(km, x, gy, out_dtype=torch.float32)

    if called_before:
        layer(x, w, gy)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        out = layer(x, w, gy)
    # sums of N exact products in fp32, each off by 2^-24 sqrt(N) of its size, N up to 3e5, twice, and a factor of four: what
    # two kernels may differ by
    close = lambda a, b: float((a - b).norm()) <= 2.6e-4 * float(b.norm())
    # before the first replay nothing that was recorded has run: the map's first direct call is as on another map
    other = fx.build_kernel_map_onto(g, km.g_out, 3) if onto else fx.build_kernel_map(g, 3, 1)
    assert all(close(a, b) for a, b in zip(layer(x, w, gy), layer(x, w, gy, other)))
    for _ in range(4):
        new = draw()
        for a, b in zip((x, w, gy), new):
            a.copy_(b)
        graph.replay()
        torch.cuda.synchronize()
        for a, ref in zip(out, layer(*new)):
            assert torch.equal(a, ref) if called_before else close(a, ref)      # the first call may take another kernel
    del graph, out

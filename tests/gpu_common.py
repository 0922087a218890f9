"""Helpers shared by the GPU parity tests: build the HIP path's objects and the oracle's on
the same seeded inputs."""
import os

import numpy as np
import torch

import paper_2407_01781_amd as fx
from oracle import cpu_oracle as O
from workloads import generators as G

TORCH_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ORACLE_THREADS = max(1, min(16, os.cpu_count() or 1))     # host threads the oracle's range-parallel harness may use


def nan_filled(shape, dtype) -> torch.Tensor:
    """An output buffer no element of which can pass a comparison unless the kernel wrote it."""
    return torch.full(tuple(shape), float("nan"), dtype=dtype, device="cuda")


def row_error_report(y: np.ndarray, ref: np.ndarray) -> float:
    """Largest per-row relative L2 error (the quantity the 16-bit bar bounds), for the test log."""
    num = np.linalg.norm(y.astype(np.float64) - ref, axis=1)
    den = np.maximum(np.linalg.norm(ref, axis=1), 1e-3 * np.sqrt(ref.shape[1]))
    return float((num / den).max()) if y.size else 0.0


def to_device_storage(x_f32: np.ndarray, dtype: str) -> torch.Tensor:
    """fp32 array holding values already rounded to `dtype` -> CUDA tensor of that dtype (same bits)."""
    t = torch.from_numpy(np.ascontiguousarray(x_f32))
    return t.to(TORCH_DT[dtype]).cuda().contiguous()


def both_grids(ijk: np.ndarray, joffsets: np.ndarray):
    d_ijk = torch.from_numpy(np.ascontiguousarray(ijk, dtype=np.int32).reshape(-1, 3)).cuda()
    g = fx.build_index_grid(d_ijk, joffsets)
    og = O.OracleGrid(ijk, joffsets)
    return g, og


def check_grid(g, og, ijk=None):
    assert g.num_voxels == og.num_voxels
    assert g.counts() == og.counts()
    assert np.array_equal(g.voxel_joffsets(), og.voxel_joffsets())
    c, j = g.ijk()
    oc, oj = og.ijk()
    assert np.array_equal(c.cpu().numpy(), oc)
    assert np.array_equal(j.cpu().numpy(), oj)
    lt, olt = g.leaf_table(), og.leaf_table()
    assert lt.tobytes() == olt.tobytes()


def conv_tolerance_check(y: np.ndarray, ref: np.ndarray, dtype: str, k3: int, c_in: int):
    """fp32: max-abs <= 1e-4*sqrt(K^3*C_in); fp16/bf16: per-row relative L2 <= 2e-2 (floor on the
    reference norm: 1e-3*sqrt(C_out))."""
    y = y.astype(np.float64)
    if dtype == "f32":
        err = np.abs(y - ref).max() if y.size else 0.0
        assert err <= 1e-4 * np.sqrt(k3 * c_in), err
        return err
    num = np.linalg.norm(y - ref, axis=1)
    den = np.maximum(np.linalg.norm(ref, axis=1), 1e-3 * np.sqrt(ref.shape[1]))
    rel = (num / den).max() if y.size else 0.0
    assert rel <= 2e-2, rel
    return rel


def box(dims, at=(0, 0, 0)) -> np.ndarray:
    """All integer points of a box, in coordinate order."""
    return np.stack(np.meshgrid(*[np.arange(d) + a for d, a in zip(dims, at)], indexing="ij"), axis=-1).reshape(-1, 3)


def facing_sheets(rows) -> np.ndarray:
    """Voxels of a grid whose tile 8 m' + t (m' depends on the sheets before) of 512 voxels reads exactly rows[m][t] rows (512 to
    2417), its own among them: 128^3 cells per m, in which a plane of every second voxel, eight tiles, faces a plane of as many
    voxels next to each tile's as it is to read, 4096 rows behind it and more; filled up to whole tiles by voxels without neighbours."""
    parts = []
    for m, counts in enumerate(rows):
        assert len(counts) == 8 and all(512 <= c <= 512 + 15 * 127 for c in counts)
        plane = np.stack(np.meshgrid([7], np.arange(0, 128, 2), np.arange(0, 128, 2), indexing="ij"), axis=-1).reshape(-1, 3)
        rng = np.random.default_rng(100 + m)
        sheet = [box((1, 15, 127), (8, 16 * t, 0))[np.sort(rng.permutation(15 * 127)[:c - 512])] for t, c in enumerate(counts)]
        n_sheet = sum(len(s) for s in sheet)
        alone = np.stack(np.meshgrid([20], np.arange(0, 128, 4), np.arange(0, 128, 4), indexing="ij"), axis=-1).reshape(-1, 3)[:-n_sheet % 512]
        parts.append(np.concatenate([plane] + sheet + [alone]) + [0, 0, 128 * m])
    return np.concatenate(parts)


def tile_row_counts(table: np.ndarray) -> np.ndarray:
    """Rows that every tile of 512 outputs of a submanifold map holds: its own and all that it reads."""
    own = np.arange(512)
    return np.array([np.union1d(table[s:s + 512][table[s:s + 512] >= 0], own[:len(table) - s] + s).size for s in range(0, len(table), 512)])

"""Dense transform by banded hulls (sides up to 2048 x 1024 x 1024) and the
envelope form beyond them, against the oracle bit for bit at the edges of
bands (32 rows), column groups (32 columns) and the two forms' border, with
obstacles that make the columns' values random, convex, concave and flat; and
the incremental form on the same shapes.  The sparse field's radii beyond 64
use the same hulls over runs of blocks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2105_04419_amd import DenseField, Field, dense_global

pytestmark = pytest.mark.gpu

SHAPES = [(31, 32, 31), (33, 64, 33), (64, 65, 32), (96, 31, 70), (2, 1024, 33), (2, 1025, 33),
          (1024, 3, 34), (1025, 3, 34), (3, 2, 2048), (3, 2, 2049), (1, 1, 32), (1, 40, 1)]


@pytest.fixture(scope="module", autouse=True)
def _setup():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    oracle.build(force=False)


def draw(shape, kind):
    nz, ny, nx = shape
    rng = np.random.default_rng(nx + 3 * ny + 7 * nz + len(kind))
    occ = np.zeros(shape, np.uint8)
    z, y = np.meshgrid(np.arange(nz), np.arange(ny), indexing="ij")
    if kind == "scattered":
        occ[rng.random(shape) < 40.0 / occ.size] = 1
    elif kind == "slope":              # the nearest x walks along the rows
        occ[z, y, (y + z) % nx] = 1
    elif kind == "bowl":               # distances along x grow with the square of y - mid
        occ[z, y, np.minimum(nx - 1, (y - ny // 2) ** 2 // 8 + (z - nz // 2) ** 2 // 8)] = 1
    else:                              # one wall, everything flat behind it
        occ[:, :, nx // 2] = 1
    occ.reshape(-1)[0] = 1
    return occ


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def ref(occ, d_max):
    return oracle.edt_separable(occ, d_max) if d_max else oracle.edt_uncapped(occ)


@pytest.mark.parametrize("kind", ["scattered", "slope", "bowl", "wall"])
@pytest.mark.parametrize("shape", SHAPES)
def test_edges_match_the_oracle(shape, kind):
    occ = draw(shape, kind)
    for d_max in (0, 300):
        got = dense_global(cu(occ), d_max).cpu().numpy()
        assert np.array_equal(got, ref(occ, d_max)), (shape, kind, d_max)


def test_occupancy_at_any_address():
    occ = draw((5, 40, 77), "scattered")
    flat = torch.zeros(occ.size + 64, dtype=torch.uint8, device="cuda")
    for off in (1, 2, 7, 13):
        v = flat[off:off + occ.size].view(occ.shape)
        v.copy_(cu(occ))
        assert np.array_equal(dense_global(v).cpu().numpy(), ref(occ, 0)), off


@pytest.mark.parametrize("shape", [(33, 70, 65), (2, 1024, 40), (130, 33, 31), (1025, 2, 34)])
def test_updates_match_the_oracle(shape):
    nz, ny, nx = shape
    rng = np.random.default_rng(sum(shape))
    occ = draw(shape, "scattered")
    f = DenseField((nx, ny, nz), 0, max_changes=64)
    f.global_(cu(occ))
    for _ in range(4):
        xyz = np.stack([rng.integers(0, nx, 40), rng.integers(0, ny, 40),
                        rng.integers(0, nz, 40)], 1).astype(np.int32)
        xyz[:4] = np.argwhere(occ)[rng.integers(0, int(occ.sum()), 4)][:, ::-1]
        st = (rng.random(40) < 0.4).astype(np.uint8)
        for (x, y, z), v in zip(xyz, st):
            occ[z, y, x] = v
        f.update(cu(xyz), cu(st))
        assert np.array_equal(f.field().cpu().numpy(), ref(occ, 0)), shape
    assert f.error() == 0


@pytest.mark.parametrize("d_max", [65, 72, 129, 255])
@pytest.mark.parametrize("shape", [(17, 9, 600), (9, 600, 20), (600, 20, 9), (40, 264, 33),
                                   (8, 8, 8), (70, 70, 70)])
def test_sparse_field_beyond_radius_64(shape, d_max):
    # work items longer than a run (64 blocks), band and block remainders, and
    # rows whose context spans several tiles; then updates through the lists
    nz, ny, nx = shape
    rng = np.random.default_rng(sum(shape) + d_max)
    occ = np.zeros(shape, np.uint8)
    occ.reshape(-1)[rng.integers(0, occ.size, 12)] = 1
    f = Field((nx, ny, nz), d_max, max_changes=64)
    f.global_(cu(occ))
    assert np.array_equal(f.dense().cpu().numpy(), oracle.edt_separable(occ, d_max)), "global"
    for step in range(2):
        xyz = np.stack([rng.integers(0, nx, 12), rng.integers(0, ny, 12),
                        rng.integers(0, nz, 12)], 1).astype(np.int32)
        xyz[:4] = np.argwhere(occ)[:4][:, ::-1]
        st = (rng.random(12) < 0.5).astype(np.uint8)
        st[:4] = 0
        for (x, y, z), v in zip(xyz, st):
            occ[z, y, x] = v
        f.update(cu(xyz), cu(st))
        assert np.array_equal(f.dense().cpu().numpy(), oracle.edt_separable(occ, d_max)), step
    assert f.error() == 0


def test_a_small_field_made_after_a_large_one():
    # the passes of both are the same kernels with very different needs of LDS
    rng = np.random.default_rng(6)
    shapes = [(1040, 9, 11), (9, 1040, 11), (16, 16, 16)]
    maps = [(rng.random(s) < 4.0 / np.prod(s)).astype(np.uint8) for s in shapes]
    fields = [Field(s[::-1], 255 if max(s) > 16 else 65, max_changes=16) for s in shapes]
    for f, occ in reversed(list(zip(fields, maps))):
        occ.reshape(-1)[0] = 1
        f.global_(cu(occ))
        occ[tuple(n // 2 for n in occ.shape)] = 1
        f.update(cu(np.array([[n // 2 for n in occ.shape[::-1]]], np.int32)), cu(np.ones(1, np.uint8)))
        assert np.array_equal(f.dense().cpu().numpy(), oracle.edt_separable(occ, f.d_max)), occ.shape
        assert f.error() == 0


def test_captured_transform_of_the_longest_columns():
    shape = (1024, 1024, 3)
    occ, small = draw(shape, "scattered"), draw((8, 8, 8), "scattered")
    src = cu(occ)
    out = torch.empty(shape, dtype=torch.int32, device="cuda")
    ws = torch.empty(8 * occ.size, dtype=torch.uint8, device="cuda")
    dense_global(src, 0, out=out, workspace=ws)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        dense_global(src, 0, out=out, workspace=ws)
    for seed in range(3):
        occ = np.roll(occ, 5, axis=1)
        src.copy_(cu(occ))
        assert np.array_equal(dense_global(cu(small)).cpu().numpy(), ref(small, 0))
        out.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), ref(occ, 0)), seed

"""Batched maps at the edges of the passes' layouts, against the oracle bit for
bit: rows shorter than a word or than a group of four voxels, sides around 32
and 64, planes of odd size (whose lines start anywhere), single voxels and
empty maps, occupancy and fields at any address, both window representations
(radii up to 40 and beyond) and every launch mode and schedule."""
import numpy as np
import pytest
import torch

import oracle
from paper_2105_04419_amd import FUSED, PER_MAP, PHASED, Batch

pytestmark = pytest.mark.gpu

# (nx, ny, nz)
SHAPES = [(1, 1, 1), (3, 40, 9), (31, 7, 33), (32, 17, 8), (33, 33, 33), (35, 64, 5), (64, 9, 65),
          (65, 31, 24), (130, 5, 3), (2, 130, 2), (1, 1, 100), (97, 23, 41), (300, 4, 4)]


@pytest.fixture(scope="module", autouse=True)
def _setup():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    oracle.build(force=False)


def draw(seed):
    rng = np.random.default_rng(seed)
    maps = []
    for k, (nx, ny, nz) in enumerate(SHAPES):
        occ = (rng.random((nz, ny, nx)) < (0.0, 0.002, 0.05, 0.5)[(k + seed) % 4]).astype(np.uint8)
        if (k + seed) % 4 == 1:
            occ.reshape(-1)[rng.integers(0, occ.size)] = 255
        maps.append(occ)
    return maps


def check(b, maps, out, d_max, what):
    for (nx, ny, nz), occ, got in zip(SHAPES, maps, b.unpack(out)):
        want = oracle.edt_separable((occ != 0).astype(np.uint8), d_max)
        assert np.array_equal(got.cpu().numpy(), want), (what, (nx, ny, nz), d_max)


@pytest.mark.parametrize("d_max", [1, 7, 8, 9, 24, 40, 41, 64])
def test_layout_edges(d_max):
    maps = draw(d_max)
    b = Batch(SHAPES, d_max)
    flat = b.pack(maps)
    check(b, maps, b.run(flat, mode=PHASED, tune={"schedule": 1, "lrun": 2}), d_max, "phased")
    check(b, maps, b.run(flat), d_max, "default")


@pytest.mark.parametrize("mode", [FUSED, PER_MAP, PHASED])
@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("lrun,chunk,wg_waves", [(1, 1, 1), (3, 64, 8), (64, 2, 4)])
def test_modes_and_schedules(mode, schedule, lrun, chunk, wg_waves):
    maps = draw(3)
    b = Batch(SHAPES, 20)
    out = b.run(b.pack(maps), mode=mode, tune={"schedule": schedule, "lrun": lrun, "chunk": chunk,
                                               "wg_waves": wg_waves, "waves_per_cu": 8})
    check(b, maps, out, 20, (mode, schedule, lrun))


def test_occupancy_and_field_at_any_address():
    maps = draw(2)
    b = Batch(SHAPES, 24)
    flat = b.pack(maps)
    for off in (1, 3, 8, 17):
        occ = torch.zeros(b.total + 64, dtype=torch.uint8, device="cuda")
        occ[off:off + b.total] = flat
        out = torch.full((b.total + 64,), -7, dtype=torch.int32, device="cuda")
        b.run(occ[off:off + b.total], out=out[off:off + b.total], mode=PHASED)
        check(b, maps, out[off:off + b.total], 24, off)
        assert (out[:off] == -7).all() and (out[off + b.total:] == -7).all()


@pytest.mark.parametrize("d_max", [8, 9, 24, 40, 41, 64])
def test_items_out_of_reach(d_max):
    # one obstacle a map, at every distance from the items (runs of 1 or 2 blocks)
    # along y and z: items just within its reach, at its end and beyond it
    shapes, maps = [], []
    for k in range(0, 200, 5):
        for axis in (0, 1):
            nz, ny, nx = (200, 3, 18) if axis == 0 else (3, 200, 18)
            occ = np.zeros((nz, ny, nx), np.uint8)
            occ[(k, 1, 7) if axis == 0 else (1, k, 7)] = 1
            shapes.append((nx, ny, nz))
            maps.append(occ)
    b = Batch(shapes, d_max)
    for lrun in (1, 16):
        out = b.run(b.pack(maps), mode=PHASED, tune={"lrun": lrun, "schedule": 1})
        for sh, occ, got in zip(shapes, maps, b.unpack(out)):
            assert np.array_equal(got.cpu().numpy(), oracle.edt_separable(occ, d_max)), (sh, lrun)

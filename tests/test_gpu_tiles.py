"""Dense ingest and window passes where whole columns, half columns or quarter
columns of a tile go to a wave (one tile to more than 64), at ragged extents,
occupancy at any address and every window representation, against the oracle
bit for bit; and a pool that fills up during the ingest."""
import numpy as np
import pytest
import torch

import oracle
from paper_2105_04419_amd import EDT_ERR_CAPACITY, Field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _setup():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    oracle.build(force=False)


@pytest.mark.parametrize("d_max", [3, 16, 20, 33, 41, 64])
@pytest.mark.parametrize("shape", [(64, 64, 64), (130, 70, 9), (200, 180, 60), (31, 300, 70),
                                   (520, 530, 12)])
def test_extents_of_one_tile_to_many(shape, d_max):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx + ny + nz + d_max)
    occ = np.zeros((nz, ny, nx), np.uint8)
    occ.reshape(-1)[rng.integers(0, occ.size, max(3, occ.size // 4000))] = rng.integers(1, 256)
    occ[:2, :5, nx - 3:] = 1
    f = Field(shape, d_max)
    flat = torch.zeros(occ.size + 16, dtype=torch.uint8, device="cuda")
    want = oracle.edt_separable((occ != 0).astype(np.uint8), d_max)
    for off in (0, 5):
        v = flat[off:off + occ.size].view(occ.shape)
        v.copy_(torch.from_numpy(occ))
        f.global_(v)
        assert np.array_equal(f.dense().cpu().numpy(), want), (shape, d_max, off)
        assert np.array_equal(f.occupancy().cpu().numpy(), (occ != 0).astype(np.uint8))
    st = f.stats()
    blocks = np.pad(occ, [(0, -nz % 8), (0, -ny % 8), (0, -nx % 8)]).reshape(
        (nz + 7) // 8, 8, (ny + 7) // 8, 8, (nx + 7) // 8, 8).any(axis=(1, 3, 5))
    assert st["obstacle_blocks"] == int(blocks.sum()) and st["error"] == 0


def test_pool_full_during_the_ingest():
    occ = np.ones((16, 64, 64), np.uint8)
    f = Field((64, 64, 16), 8, max_blocks=50)
    f.global_(torch.from_numpy(occ).cuda())
    assert f.error() == EDT_ERR_CAPACITY
    f.global_(torch.from_numpy(occ).cuda(), grow=True)
    assert (f.dense() == 0).all()

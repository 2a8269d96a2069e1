"""Scan integration by blocks (k_scan_clear) against the oracle where the
split of the rays can go wrong: numbers of rays around a workgroup's 64, rays
long enough for the wide products, rays along axes and diagonals (ties), and
a list that is exactly full.  Occupancy is compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2105_04419_amd import EDT_ERR_CAPACITY, Field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _setup():
    oracle.build(force=False)


def dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a).astype(dtype)).cuda()


def integrated(f, occ, origin, ends, hits):
    f.global_(dev(occ, np.uint8))
    f.integrate_scan(dev(origin, np.int32), dev(ends, np.int32), dev(hits, np.uint8))
    return f.occupancy().cpu().numpy()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, 4097])
@pytest.mark.parametrize("shape", [(70, 45, 33), (300, 9, 8)])
def test_ray_counts(shape, n):
    rng = np.random.default_rng(n)
    occ = (rng.random(shape[::-1]) < 0.3).astype(np.uint8)
    origin = np.array([rng.integers(0, s) for s in shape])
    ends = np.stack([rng.integers(0, s, n) for s in shape], 1)
    ends[rng.random(n) < 0.1] = -1                      # outside: no voxel
    hits = (rng.random(n) < 0.5).astype(np.uint8)
    f = Field(shape, 5)
    for t in range(2):                                  # the list starts empty again
        got = integrated(f, occ, origin, ends, hits)
        want, _ = oracle.integrate_scan(occ.copy(), origin, ends, hits)
        assert np.array_equal(got, want), t


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_long_rays(axis):
    shape = [12, 12, 12]
    shape[axis] = 70000
    rng = np.random.default_rng(axis)
    occ = (rng.random(shape[::-1]) < 0.05).astype(np.uint8)
    origin = [5, 6, 7]
    origin[axis] = 69990
    ends = np.stack([rng.integers(0, s, 20) for s in shape], 1)
    ends[0] = origin
    ends[1] = 0
    ends[2, axis] = 0
    got = integrated(Field(shape, 3), occ, np.array(origin), ends, np.ones(20, np.uint8))
    want, _ = oracle.integrate_scan(occ.copy(), np.array(origin), ends, np.ones(20, np.uint8))
    assert np.array_equal(got, want)


def test_ties_on_a_full_map():
    occ = np.ones((40, 40, 40), np.uint8)
    origin = np.array([17, 21, 20])
    ends = origin + np.array([[k * a, k * b, k * c] for k in (1, 7, 8, 9, 16) for a in (-1, 0, 1)
                              for b in (-1, 0, 1) for c in (-1, 0, 1)])
    f = Field((40, 40, 40), 4)
    for e in ends:
        got = integrated(f, occ, origin, e[None], np.zeros(1))
        want, _ = oracle.integrate_scan(occ.copy(), origin, e[None], np.zeros(1, np.uint8))
        assert np.array_equal(got, want), e


@pytest.mark.parametrize("spare", [0, 1])
def test_full_list(spare):
    # one ray of 31 voxels to free: the list holds them exactly, or all but one
    occ = np.ones((8, 8, 31), np.uint8)
    f = Field((31, 8, 8), 4, max_changes=1 + 31 - spare)
    got = integrated(f, occ, np.array([0, 3, 3]), np.array([[30, 3, 3]]), np.zeros(1))
    assert (occ - got).sum() == 31 - spare
    assert f.error() == (EDT_ERR_CAPACITY if spare else 0)

"""The neighbour search against the FP64 oracle where its queues, its window of
seeds and its shells change behaviour: vertex counts around the window and a
wave, list lengths of every kind, cells far fuller than the queues, and
vertices so sparse that shells have to grow far.  Neighbour lists are whole
numbers: they are equal or wrong."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu


def positions(kind, n, rng):
    if kind == "uniform":
        return rng.random((n, 3))
    if kind == "clump":      # most vertices in a few cells, the rest far from them
        p = 0.3 + 0.004 * rng.random((n, 3))
        p[:: 7] = rng.random((len(p[:: 7]), 3))
        return p
    p = rng.random((n, 3))   # "sheet": two thin layers on opposite faces of the cube
    p[:, 2] = np.where(p[:, 2] < 0.5, 0.0, 1.0 - 1e-6)
    return p


@pytest.mark.parametrize("kind", ["uniform", "clump", "sheet"])
@pytest.mark.parametrize("n,k", [(2, 2), (16, 16), (17, 9), (18, 17), (33, 16), (64, 8), (65, 33), (257, 64),
                                 (1000, 12), (4099, 16)])
def test_neighbours_match_oracle(kind, n, k):
    rng = np.random.default_rng(n * 31 + k)
    sc = synthetic(positions(kind, n, rng), rng)
    print(f"knn {kind} n={n} k={k}", flush=True)
    ref = oracle.knn(sc.pos, k)
    for shift in (0, 13, 20):
        _, col = pg.pg_knn(pg.DevicePaths(sc), k, shift)
        assert np.array_equal(col.cpu().numpy().reshape(n, min(k, n)), ref), shift

"""The neighbour search with 8, 4 and 2 lanes a query, on both sides of the lines in N K that choose
between them, against the FP64 oracle.  Neighbour lists are whole numbers: they are equal or wrong."""
import numpy as np
import pytest

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu

SIZES = [(n, k) for k in (3, 7) for n in (7, 40, 2 ** 16 // k, 2 ** 16 // k + 1)]
SIZES += [(2 ** 16 // k + i, k) for k in range(8, 18) for i in (0, 1)]
SIZES += [(2 ** 19 // k + i, k) for k in (11, 14, 16, 17) for i in (0, 1)]


@pytest.mark.parametrize("n,k", SIZES)
def test_groups_match_oracle(n, k):
    rng = np.random.default_rng(n + k)
    pos = rng.random((n, 3))
    pos[::3] = 0.25 + 0.05 * pos[::3]       # a dense part: queues fill, lists merge over many shells
    pos[1::50] = pos[::50][:len(pos[1::50])]    # equal distances: the lower id first
    sc = synthetic(pos, rng)
    print(f"knn groups n={n} k={k}", flush=True)
    ref = oracle.knn(sc.pos, k)
    for shift in (0, 14):
        _, col = pg.pg_knn(pg.DevicePaths(sc), k, shift)
        assert np.array_equal(col.cpu().numpy().reshape(n, min(k, n)), ref), shift

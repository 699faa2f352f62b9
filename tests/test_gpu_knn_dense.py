"""Neighbour lists where cells hold many vertices, which are searched before their neighbours are: blobs on cell
corners, a plane, coincident vertices, cells around the count from which that is done; against the oracle's lists."""
import numpy as np
import pytest

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu


def positions(kind, n, rng):
    if kind == "corner blob":
        p = 0.5 + 0.01 * rng.standard_normal((n, 3))
        p[::50] = rng.random((len(p[::50]), 3))
    elif kind == "plane":
        p = rng.random((n, 3))
        p[:, 2] = 0.5
    elif kind == "coincident":
        p = np.repeat(rng.random((-(-n // 90), 3)), 90, axis=0)[:n]
    else:   # cells of 62 to 67 vertices beside empty ones
        cells = rng.permutation(4096)[:n // 64 + 1]
        at = np.repeat(cells, rng.integers(62, 68, len(cells)))[:n]
        at = np.concatenate([at, rng.integers(0, 4096, n - len(at))])
        p = (np.stack([at % 16, at // 16 % 16, at // 256], 1) + 0.1 + 0.8 * rng.random((n, 3))) / 16
    return np.clip(p, 0.0, 1.0).astype(np.float32)[rng.permutation(n)]


@pytest.mark.parametrize("kind,shift", [("corner blob", 0), ("plane", 0), ("coincident", 0), ("counts", 16)])
@pytest.mark.parametrize("k", [2, 9, 16, 17, 20, 40])
def test_lists_match_oracle(kind, shift, k):
    n = (1 << 19) // k + 33   # the size from which populous cells come first
    print(f"knn {kind} n={n} k={k}", flush=True)
    rng = np.random.default_rng(k)
    sc = synthetic(positions(kind, n, rng), rng)
    sc.width, sc.height = n, 1
    _, col = pg.pg_knn(pg.DevicePaths(sc), k, shift)
    rows = rng.choice(n, 600, replace=False).astype(np.int32)
    assert np.array_equal(col.cpu().numpy().reshape(n, k)[rows], oracle.knn(sc.pos, k, rows=rows))

"""pg_propagate in path order, where a row stores at its predecessor: odd and even numbers of iterations,
paths of one vertex, empty paths and paths that end at the edge of a block, against 64-bit arithmetic."""
import numpy as np
import pytest
import torch

import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [False, True])
@pytest.mark.parametrize("D", [1, 2, 3, 8])
@pytest.mark.parametrize("lengths,k", [([1], 1), ([2], 2), ([1, 1, 1], 3), ([0, 3, 0, 1, 60, 0, 64, 1, 128], 8),
                                       ([16] * 64, 13), ([255, 1, 0, 257, 511], 33)])
def test_propagation_along_paths(lengths, k, D, grid):
    print(f"propagate paths {lengths[:9]} k={k} D={D} grid={grid}", flush=True)
    rng = np.random.default_rng(k)
    n = sum(lengths)
    sc = synthetic(rng.random((n, 3)), rng, lengths=np.array(lengths))
    # a constant grid: the interpolation gives the value itself to a rounding or two
    paths = pg.DevicePaths(sc, albedo_grid=np.full((2, 2, 2), 0.75, np.float32) if grid else None)
    K = min(k, n)
    col = rng.integers(0, n, (n, K))
    w, b, x = rng.random((n, K), dtype=np.float32) / K, rng.random((n, 3), dtype=np.float32), rng.random(
        (n, 3), dtype=np.float32)
    alpha = np.full(n, 0.75) if grid else sc.albedo.astype(np.float64)
    off = np.concatenate([[0], np.cumsum(lengths)])
    last = np.unique(off[1:][np.array(lengths) > 0] - 1)
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t)  # noqa: E731
    got, traj = pg.pg_propagate(paths, pg.params(k=k, D=D), dev(np.arange(n + 1) * K, torch.int64),
                                dev(col.reshape(-1), torch.int32), dev(w.reshape(-1), torch.float32),
                                dev(b, torch.float32), dev(x, torch.float32), traj=True)
    assert torch.equal(got, traj[D - 1])
    ref = x.astype(np.float64)
    for t in range(D):
        y = b + alpha[:, None] * (w[:, :, None].astype(np.float64) * ref[col]).sum(1)
        ref = np.zeros_like(y)
        ref[:-1] = y[1:]
        ref[last] = 0.0
        # every term is positive: K + 4 roundings an iteration of half a unit each, and alpha's own two
        bound = (t + 1) * (K + 6) * 2.0 ** -24 * ref
        assert (np.abs(traj[t].cpu().numpy() - ref) <= bound).all(), t

"""pg_propagate over the three orders that it may iterate a large graph in: neighbours near in space but far in path
order (moved to the spatial order), near in path order (kept there), far in both (the caller's rows); and mixtures.
Each equals the path-order iteration bit for bit, also with ids out of range and values that are not finite."""
import numpy as np
import pytest
import torch

import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic
from tests.test_gpu_propagate_sorted import N, propagate

pytestmark = pytest.mark.gpu


def neighbours(kind, paths, k, rng):
    row = np.arange(N)[:, None]
    near = (row + rng.integers(-50, 51, (N, k))) % N
    far = rng.integers(0, N, (N, k))
    space = pg.pg_knn(paths, k)[1].cpu().numpy().reshape(N, k).astype(np.int64)
    if kind == "space":
        return space
    if kind == "space, some far":
        return np.where(rng.random((N, k)) < 0.2, far, space)
    if kind == "paths, some far":
        return np.where(rng.random((N, k)) < 0.3, far, near)
    if kind == "far, some near":
        return np.where(rng.random((N, k)) < 0.3, near, far)
    return np.where(rng.random((N, 1)) < 0.5, space, far)   # rows of both kinds


@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 12, 16, 17, 24, 29, 32])
@pytest.mark.parametrize("kind", ["space", "space, some far", "paths, some far", "far, some near", "rows"])
def test_every_order_equals_path_order(kind, k):
    print(f"propagate places {kind} k={k}", flush=True)
    rng = np.random.default_rng(k)
    lengths = np.full(N // 29 + 1, 29)
    lengths[-1] = N - 29 * (len(lengths) - 1)
    paths = pg.DevicePaths(synthetic(rng.random((N, 3)), rng, lengths=lengths))
    col = neighbours(kind, paths, k, rng)
    bad = rng.random((N, k)) < 1e-3
    col[bad] = rng.choice([-1, N, -2 ** 31, 2 ** 31 - 1], int(bad.sum()))
    x = rng.random((N, 3), dtype=np.float32)
    x[7], x[N - 5] = np.inf, np.nan
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t)  # noqa: E731
    args = (dev(np.arange(N + 1) * k, torch.int64), dev(col.reshape(-1), torch.int32),
            dev(rng.random(N * k) / k, torch.float32), dev(rng.random((N, 3)), torch.float32), dev(x, torch.float32))
    q = pg.params(k=k, D=max(4, -(-(1 << 26) // (N * k))))
    got, ref = propagate(paths, q, *args, small=False), propagate(paths, q, *args, small=True)
    for a, b in zip(got, ref):
        assert torch.equal(a.isnan(), b.isnan())
        assert torch.equal(a.view(torch.int32)[~a.isnan()], b.view(torch.int32)[~b.isnan()])
    assert got[0].isfinite().any()

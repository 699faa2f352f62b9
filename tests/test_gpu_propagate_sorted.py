"""pg_propagate on graphs large enough for its sorted order against the same
call with a workspace that only holds the path-order iteration (which the
other tests pin against the oracle): the sums are taken in the same order, so
L+_D and the whole trajectory are equal bit for bit, also with ids out of
range, rows that do not begin with themselves, far neighbours and values that
are not finite."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu

N = (1 << 18) + 37


def propagate(paths, q, row_ptr, col, w, b, x, small):
    L, s = pg.lib(), paths.struct()
    nb = ctypes.c_size_t()
    pg._check(L.pg_propagate_workspace_size(ctypes.byref(s), ctypes.byref(q), ctypes.byref(nb)))
    path_order = 24 * N + 8192
    assert nb.value > path_order   # these sizes do take the sorted order
    _, ws, n = pg._workspace(path_order if small else nb.value, paths.device)
    traj = torch.full((q.D, N, 3), float("nan"), device=paths.device)
    x = x.clone()
    pg._check(L.pg_propagate(ctypes.byref(s), ctypes.byref(q), pg._ptr(row_ptr), pg._ptr(col), pg._ptr(w), pg._ptr(b),
                             pg._ptr(x), pg._ptr(traj), pg._ptr(ws), n, pg._stream(paths.device)))
    torch.cuda.synchronize()
    return x, traj


@pytest.mark.parametrize("k", [1, 2, 3, 8, 13, 16, 21, 32])
@pytest.mark.parametrize("reach", [64, N])
def test_sorted_order_equals_path_order(k, reach):
    print(f"propagate sorted k={k} reach={reach}", flush=True)
    rng = np.random.default_rng(k)
    lengths = np.full(N // 37 + 1, 37)
    lengths[-1] = N - 37 * (len(lengths) - 1)
    paths = pg.DevicePaths(synthetic(rng.random((N, 3)), rng, lengths=lengths))
    row = np.arange(N)[:, None]
    col = (row + rng.integers(-reach, reach + 1, (N, k))) % N
    col[::3, 0] = np.arange(N)[::3]
    bad = rng.random((N, k)) < 1e-3
    col[bad] = rng.choice([-1, N, -2 ** 31, 2 ** 31 - 1], int(bad.sum()))
    x = rng.random((N, 3), dtype=np.float32)
    x[5], x[N - 3] = np.inf, np.nan
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", t)  # noqa: E731
    args = (dev(np.arange(N + 1) * k, torch.int64), dev(col.reshape(-1), torch.int32),
            dev(rng.random(N * k) / k, torch.float32), dev(rng.random((N, 3)), torch.float32),
            dev(x, torch.float32))
    q = pg.params(k=k, D=-(-(1 << 26) // (N * k)))   # the least work that is moved to the sorted order
    got, ref = propagate(paths, q, *args, small=False), propagate(paths, q, *args, small=True)
    for a, b in zip(got, ref):
        assert torch.equal(a.view(torch.int32)[~a.isnan()], b.view(torch.int32)[~b.isnan()])
        assert torch.equal(a.isnan(), b.isnan())
    assert got[0].isfinite().any()

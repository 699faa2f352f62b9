"""The iteration on both sides of the sizes at which its stores change their cache hint, forward against
64-bit arithmetic over the exported graph, backward with the stored sums against the recomputing sweep."""
import numpy as np
import pytest
import torch

import paper_2404_11894_amd as pg
from tests.gpu_util import synthetic

pytestmark = pytest.mark.gpu

LINES = [(4 << 20) // 24, (12 << 20) // 24]


@pytest.mark.parametrize("k", [5, 16, 24])
@pytest.mark.parametrize("n", [m + d for m in LINES for d in (0, 1)])
def test_iteration_matches_graph(n, k):
    D = 3
    print(f"iteration stores n={n} k={k}", flush=True)
    rng = np.random.default_rng(n + k)
    sc = synthetic(rng.random((n, 3)), rng, lengths=np.append(np.full(n // 7, 7), n % 7))
    paths = pg.DevicePaths(sc, albedo_grid=rng.uniform(0.6, 0.95, (8, 8, 8)).astype(np.float32))
    q = pg.params(k=k, D=D, g=0.5, init="zero", flags=pg.PG_FLAG_CHECK)
    img, gr = pg.pg_render(paths, q, graph=True)
    gi = torch.rand(img.shape, generator=torch.Generator().manual_seed(k))
    base = dict(k=k, D=D, g=0.5)
    a = pg.pg_backward(paths, pg.params(**base, flags=pg.PG_FLAG_STORE_Z), gi)
    b = pg.pg_backward(paths, pg.params(**base), gi)
    # positive terms (a voxel's vertices, some 400 sums each of a few roundings): far below 1e-5
    assert torch.allclose(a["grad_grid"], b["grad_grid"], rtol=1e-5, atol=1e-5 * float(b["grad_grid"].abs().max()))
    assert torch.allclose(a["grad_g"], b["grad_g"], rtol=1e-4)

    paths = pg.DevicePaths(sc)
    _, gr = pg.pg_render(paths, q, graph=True)
    col, w, rhs = gr["col"].view(n, k).long(), gr["w_ind"].view(n, k).double(), gr["b"].double()
    alpha = torch.from_numpy(sc.albedo).to("cuda", torch.float64)[:, None]
    last = torch.from_numpy(sc.path_offsets[1:] - 1).to("cuda")
    x = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    for _ in range(D):
        y = rhs + alpha * (w[:, :, None] * x[col]).sum(1)
        x = torch.zeros_like(x)
        x[:-1] = y[1:]
        x[last] = 0.0
    assert ((gr["lplus"].double() - x).abs() <= D * (k + 4) * 2.0 ** -24 * x).all()

"""The cluster render where its blocks' spans change: sizes about a word of the heads, a block and two, a
cluster larger than the staged span, and vertices enough for loads past the caches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import grad_close, synthetic
from tests.test_gpu_clusters import compare_graph, gpu_cluster_render, keyed

pytestmark = pytest.mark.gpu


def scene(n, rng, coincident=0):
    pos = rng.random((n, 3))
    pos[:coincident] = 0.5   # no split ends: each round only peels single members off
    lengths = rng.integers(1, 9, n)
    lengths = lengths[:np.searchsorted(np.cumsum(lengths), n) + 1]
    lengths[-1] -= lengths.sum() - n
    return keyed(synthetic(pos, rng, lengths=lengths), seed=n)


@pytest.mark.parametrize("n,k,coincident", [(1, 4, 0), (63, 8, 0), (64, 1, 0), (65, 16, 0), (255, 2, 0), (256, 64, 0),
                                            (257, 8, 0), (512, 16, 0), (513, 33, 0), (2000, 64, 0), (1100, 8, 700)])
def test_spans_match_oracle(n, k, coincident):
    print(f"cluster spans n={n} k={k} coincident={coincident}", flush=True)
    sc = scene(n, np.random.default_rng(n), coincident)
    img, gr = gpu_cluster_render(sc, k, 3, 0.5)
    ref_img, ref = oracle.render(sc, oracle.params(k=k, D=3, g=0.5, neighbours="clusters"), trace=True)
    if coincident:
        assert np.diff(ref["row_ptr"]).max() > 512   # past the span that a block stages
    compare_graph(sc, img, gr, ref_img, ref, f"{n}/{k}")


@pytest.mark.parametrize("n,k,coincident", [(257, 8, 0), (1100, 8, 700)])
def test_adjoint_over_spans_matches_oracle(n, k, coincident):
    print(f"cluster adjoint spans n={n} k={k} coincident={coincident}", flush=True)
    rng = np.random.default_rng(n)
    sc = scene(n, rng, coincident)
    gimg = rng.standard_normal((sc.height, sc.width, 3))
    op = oracle.params(k=k, D=3, g=0.5, neighbours="clusters")
    ref, mag = oracle.backward(sc, op, gimg), oracle.backward(sc, op, np.abs(gimg))
    q = pg.params(k=k, D=3, g=0.5, flags=pg.PG_FLAG_CHECK | pg.PG_FLAG_CLUSTERS)
    out = pg.pg_backward(pg.DevicePaths(sc), q, torch.from_numpy(gimg.astype(np.float32)), grad_grid=False,
                         grad_albedo=True)
    grad_close(out["grad_albedo"].cpu().numpy(), ref["grad_alpha"], "grad albedo", mag["grad_alpha"])
    grad_close([out["grad_g"].item()], [ref["grad_g"]], "grad g", [mag["grad_g"]])


def test_iteration_past_the_caches():
    n, k, D = (256 << 20) // 72 + 1, 8, 2
    print(f"cluster iteration n={n}", flush=True)
    rng = np.random.default_rng(5)
    sc = synthetic(rng.random((n, 3)), rng, lengths=np.append(np.full(n // 7, 7), n % 7))
    sc = keyed(sc)
    paths = pg.DevicePaths(sc)
    q = pg.params(k=k, D=D, g=0.5, init="zero", flags=pg.PG_FLAG_CHECK | pg.PG_FLAG_CLUSTERS)
    _, gr = pg.pg_render(paths, q, graph=True)
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), gr["row_ptr"].diff())
    w, col, b = gr["w_ind"].double()[:, None], gr["col"].long(), gr["b"].double()
    alpha = torch.from_numpy(sc.albedo).to("cuda", torch.float64)[:, None]
    last = torch.from_numpy(sc.path_offsets[1:] - 1).to("cuda")
    x = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    for _ in range(D):
        y = b + alpha * torch.zeros_like(x).index_add_(0, rows, w * x[col])
        x = torch.zeros_like(x)
        x[:-1] = y[1:]
        x[last] = 0.0
    # positive terms: a rounding a member in the sum, 16 in a weight that is evaluated twice, each iteration
    members = int(gr["row_ptr"].diff().max())
    assert ((gr["lplus"].double() - x).abs() <= D * (members + 16) * 2.0 ** -24 * x).all()

"""The cluster render where a cluster of more members than a block has rows ends in the last, short block: the
block stages all of the span before its rows (kernels: aggregation, reverse rows, reverse columns)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import grad_close, synthetic
from tests.test_gpu_clusters import compare_graph, gpu_cluster_render, keyed

pytestmark = pytest.mark.gpu

BLOCK, SPAN = 256, 512   # rows of a block, members that it stages at most


def scene(before, members, after, rng):
    """`members` coincident vertices (no split ends them) between others, along the curve that orders the vertices:
    its first octant is the one at the origin, the cluster's cell lies in the opposite one."""
    n = before + members + after
    pos = np.full((n, 3), 0.5)
    pos[:before] = rng.random((before, 3)) * 0.2
    pos[before + members:] = [0.85, 0.05, 0.05] + 0.1 * rng.random((after, 3))
    lengths = rng.integers(1, 9, n)
    lengths = lengths[:np.searchsorted(np.cumsum(lengths), n) + 1]
    lengths[-1] -= lengths.sum() - n
    return keyed(synthetic(pos[rng.permutation(n)], rng, lengths=lengths), seed=n)


# (before, members, after): up to 492 members of the last block's span come before its rows
CASES = [(100, 450, 50), (150, 450, 0), (250, 262, 1), (20, 493, 0), (513, 300, 0), (506, 263, 0)]


def check_layout(ref):
    assert BLOCK < np.diff(ref["row_ptr"]).max() <= SPAN


@pytest.mark.parametrize("before,members,after", CASES)
def test_render_matches_oracle(before, members, after):
    print(f"last block: {before} {members} {after}", flush=True)
    sc = scene(before, members, after, np.random.default_rng(members))
    ref_img, ref = oracle.render(sc, oracle.params(k=8, D=3, g=0.5, neighbours="clusters"), trace=True)
    check_layout(ref)
    img, gr = gpu_cluster_render(sc, 8, 3, 0.5)
    compare_graph(sc, img, gr, ref_img, ref, f"{before}/{members}/{after}")


@pytest.mark.parametrize("before,members,after", CASES[:3])
def test_adjoint_matches_oracle(before, members, after):
    print(f"last block adjoint: {before} {members} {after}", flush=True)
    rng = np.random.default_rng(members)
    sc = scene(before, members, after, rng)
    gimg = rng.standard_normal((sc.height, sc.width, 3))
    op = oracle.params(k=8, D=3, g=0.5, neighbours="clusters")
    ref, mag = oracle.backward(sc, op, gimg), oracle.backward(sc, op, np.abs(gimg))
    q = pg.params(k=8, D=3, g=0.5, flags=pg.PG_FLAG_CHECK | pg.PG_FLAG_CLUSTERS)
    out = pg.pg_backward(pg.DevicePaths(sc), q, torch.from_numpy(gimg.astype(np.float32)), grad_grid=False,
                         grad_albedo=True)
    grad_close(out["grad_albedo"].cpu().numpy(), ref["grad_alpha"], "grad albedo", mag["grad_alpha"])
    grad_close([out["grad_g"].item()], [ref["grad_g"]], "grad g", [mag["grad_g"]])

"""Prefix sums whose n + 1 results fill their buffer to its last aligned byte, over enough counts for the passes of
several blocks: the total stays inside (of clusters' members, of exported rows, of traced paths)."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
import scenegen
from tests.gpu_util import synthetic
from tests.test_gpu_clusters import compare_graph, gpu_cluster_render, keyed
from tests.test_gpu_trace import compare

pytestmark = pytest.mark.gpu

N = 258 * 64 - 1   # N + 1 elements of 4 bytes are a multiple of 256 bytes; one block scans up to 16384


@pytest.mark.parametrize("n", [N, N + 1])
def test_cluster_rows(n):
    print(f"scan ends: clusters n={n}", flush=True)
    rng = np.random.default_rng(n)
    sc = keyed(synthetic(rng.random((n, 3)), rng, width=n), seed=n)
    img, gr = gpu_cluster_render(sc, 8, 1, 0.5)
    ref_img, ref = oracle.render(sc, oracle.params(k=8, D=1, g=0.5, neighbours="clusters"), trace=True)
    compare_graph(sc, img, gr, ref_img, ref, f"n={n}")


def test_traced_paths():
    print("scan ends: traced paths", flush=True)
    w, h = 209, 79
    assert w * h == N
    compare(replace(scenegen.WORKLOADS["tiny"].scene, width=w, height=h, spp=1))

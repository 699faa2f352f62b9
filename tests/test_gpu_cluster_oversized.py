"""A cluster above the member limit (keys that are not uniform) beside ordinary ones: it is reported, and the rows of
the others are those of a scene without it."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import paper_2404_11894_amd as pg
from tests.gpu_util import PIX_ABS, PIX_REL, assert_within, synthetic
from tests.test_gpu_clusters import keyed

pytestmark = pytest.mark.gpu


def radiance(sc, reported=False):
    """L+ of every vertex, written whether or not the call reports a cluster."""
    q = pg.params(k=8, D=4, g=0.5, flags=pg.PG_FLAG_CHECK | pg.PG_FLAG_CLUSTERS)
    paths = pg.DevicePaths(sc)
    lplus = torch.empty(sc.n_vertices, 3, device="cuda")
    render = pg.Renderer(paths, q)
    if reported:
        with pytest.raises(pg.PathGraphError, match="more than 4096 members"):
            render(graph={"lplus": lplus})
    else:
        render(graph={"lplus": lplus})
    torch.cuda.synchronize()
    return lplus.cpu().numpy()


def part(sc, a, b):
    """The paths of the vertices a to b alone (one vertex pixel each)."""
    off = sc.path_offsets
    pa, pb = np.searchsorted(off, a), np.searchsorted(off, b)
    cut = {n: getattr(sc, n)[a:b] for n in ("pos", "dir_in", "dir_out", "albedo", "l_sun", "dir_env", "l_env", "l_phase",
                                            "cluster_key")}
    return replace(sc, width=int(pb - pa), height=1, path_offsets=off[pa:pb + 1] - off[pa], e_cam=sc.e_cam[pa:pb], **cut)


@pytest.mark.parametrize("before,members,after", [(3000, 4098, 3000), (130, 9002, 70), (0, 12346, 1501), (1500, 6001, 0)])
def test_ordinary_clusters_beside_an_oversized_one(before, members, after):
    print(f"oversized cluster: {before} {members} {after}", flush=True)
    rng = np.random.default_rng(members)
    n = before + members + after
    pos = np.concatenate([0.02 + 0.3 * rng.random((before, 3)), 0.55 + 0.1 * rng.random((members, 3)),
                          [0.9, 0.02, 0.02] + 0.08 * rng.random((after, 3))])
    sc = keyed(synthetic(pos, rng, lengths=np.append(np.full(n // 2, 2), np.full(n % 2, 1))), seed=n)
    key = sc.cluster_key.copy()
    key[before:before + members] = 0xffffffff
    key[before] = 1   # its only centre
    key[0] = 2        # of the vertices before
    key[n - 1] = 3 if after else key[n - 1]
    sc = replace(sc, cluster_key=key)
    got = radiance(sc, reported=True)
    for a, b in ((0, before), (before + members, n)):
        if b > a:
            assert_within(got[a:b], radiance(part(sc, a, b)), PIX_REL, PIX_ABS, f"vertices {a} to {b}")

"""The output and its adjoint with extra emitter samples at the first vertices: counts around those from which a
group of lanes shares them, for group sizes from one lane to a wave, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_11894_amd as pg
from tests.gpu_util import PIX_ABS, PIX_REL, assert_within, grad_close, synthetic, unit

pytestmark = pytest.mark.gpu


def scene(rng, M, spp):
    lengths = rng.integers(0, 4, 17 * 3 * spp)
    sc = synthetic(rng.random((int(lengths.sum()), 3)), rng, spp=spp, width=17, lengths=lengths)
    P = len(lengths)
    sc.fb_l_sun = rng.random((P, M, 3), dtype=np.float32)
    sc.fb_l_env = rng.random((P, M, 3), dtype=np.float32)
    sc.fb_dir_env = unit(rng, P * M).reshape(P, M, 3)
    return sc


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 16, 65])
@pytest.mark.parametrize("k,spp,fg", [(1, 1, 0), (3, 2, 0), (8, 3, 1), (16, 5, 0), (20, 1, 1), (33, 2, 0), (64, 3, 0)])
def test_image_matches_oracle(M, k, spp, fg):
    print(f"extra samples M={M} k={k} spp={spp} fg={fg}", flush=True)
    sc = scene(np.random.default_rng(100 * M + k), M, spp)
    q = pg.params(k=k, D=2, g=0.4, final_gather=fg, flags=pg.PG_FLAG_CHECK)
    img = pg.pg_render(pg.DevicePaths(sc), q)
    ref = oracle.render(sc, oracle.params(k=k, D=2, g=0.4, final_gather=fg))
    assert_within(img.cpu().numpy(), ref, PIX_REL, PIX_ABS, "image")


@pytest.mark.parametrize("M,k,fg", [(1, 8, 0), (3, 16, 0), (16, 3, 1), (16, 20, 0), (65, 64, 0)])
def test_adjoint_matches_oracle(M, k, fg):
    print(f"extra samples adjoint M={M} k={k} fg={fg}", flush=True)
    rng = np.random.default_rng(100 * M + k)
    sc = scene(rng, M, 3)
    gimg = rng.standard_normal((sc.height, sc.width, 3))
    op = oracle.params(k=k, D=2, g=0.4, final_gather=fg)
    ref, mag = oracle.backward(sc, op, gimg), oracle.backward(sc, op, np.abs(gimg))
    q = pg.params(k=k, D=2, g=0.4, final_gather=fg, flags=pg.PG_FLAG_CHECK)
    out = pg.pg_backward(pg.DevicePaths(sc), q, torch.from_numpy(gimg.astype(np.float32)), grad_grid=False,
                         grad_albedo=True)
    grad_close(out["grad_albedo"].cpu().numpy(), ref["grad_alpha"], "grad albedo", mag["grad_alpha"])
    grad_close([out["grad_g"].item()], [ref["grad_g"]], "grad g", [mag["grad_g"]])

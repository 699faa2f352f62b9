"""Tracing an empty medium under majorants that no positive float reaches: every path escapes, as with 0."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import scenegen
import paper_2404_11894_amd as pg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("majorant", [0.0, 1e-300, float(np.finfo(float).tiny), 2.0 ** -150, 2.0 ** -149, 1e-30])
def test_empty_medium(majorant):
    cfg = replace(scenegen.WORKLOADS["tiny"].scene, width=9, height=8, spp=3, extra_samples=2)
    print(f"trace an empty medium, majorant {majorant}", flush=True)
    rec = pg.pg_trace(scenegen.tracer_settings(cfg), np.zeros((cfg.R,) * 3, np.float32), None, majorant)
    torch.cuda.synchronize()
    assert rec.n_vertices == 0 and not rec.path_offsets.any()
    assert torch.equal(rec.e_cam, torch.tensor(cfg.env_L, dtype=torch.float32, device="cuda").expand(9 * 8 * 3, 3))
    assert not rec.fb_l_sun.any() and not rec.fb_dir_env.any() and not rec.fb_l_env.any()

"""The tracer's path queue where it can go wrong: fewer paths than a wave, path
counts around a wave and a block, paths that all end at the first vertex or
mostly miss the medium, and the optional rays.  Same criterion as the tracer's
other tests (records within 2 float ulps of the host generator's)."""
from dataclasses import replace

import numpy as np
import pytest

import scenegen
from tests.test_gpu_trace import compare, traced

pytestmark = pytest.mark.gpu

PL = dict(pl_I=(1.5, 1.0, 0.5), pl_pos=(0.5, 1.1, 0.5))


@pytest.mark.parametrize("w,h,spp,more", [(1, 1, 1, {}), (7, 9, 1, {}), (5, 13, 1, PL), (16, 17, 1, {}), (64, 61, 5, {}),
                                          (33, 31, 2, dict(max_depth=1)), (40, 40, 1, dict(vfov_deg=140.0)),
                                          (31, 29, 3, dict(max_depth=64, sigma_max=40.0, **PL))])
def test_traced_records_match_the_generator(w, h, spp, more):
    cfg = replace(scenegen.WORKLOADS["tiny"].scene, width=w, height=h, spp=spp, **more)
    print(f"trace {w}x{h}x{spp} {more}", flush=True)
    compare(cfg)


@pytest.mark.parametrize("more", [{}, PL])
def test_extra_samples_of_queued_paths(more):
    cfg = replace(scenegen.WORKLOADS["tiny"].scene, width=45, height=23, spp=3, extra_samples=2, **more)
    print(f"trace extra samples {more}", flush=True)
    ref, rec = scenegen.generate(cfg), traced(cfg)
    for f in ("fb_l_sun", "fb_dir_env", "fb_l_env"):
        a, b = getattr(rec, f).cpu().numpy(), getattr(ref, f)
        ulps = np.abs(a.view(np.int32).astype(np.int64) - b.view(np.int32).astype(np.int64))
        assert np.all((ulps <= 2) | (a == b)), f

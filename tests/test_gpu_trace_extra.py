"""The tracer's extra samples, drawn in a pass of their own: sample counts and path counts around a wave and a block,
paths without a first vertex among them, a crop, and path counts that narrow the waves of the path pass.  Same
criterion as the tracer's other tests (within 2 float ulps of the host generator's)."""
from dataclasses import replace

import numpy as np
import pytest

import scenegen
from tests.test_gpu_trace import compare, traced

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,spp,M,more", [(1, 1, 1, 3, {}), (7, 9, 1, 1, {}), (13, 5, 4, 17, {}), (64, 64, 2, 4, {}),
                                            (33, 31, 3, 5, dict(vfov_deg=120.0)), (90, 91, 1, 2, dict(max_depth=1)),
                                            (21, 17, 2, 3, dict(pl_I=(1.5, 1.0, 0.5), pl_pos=(0.5, 1.1, 0.5)))])
def test_extra_samples_match_the_generator(w, h, spp, M, more):
    cfg = replace(scenegen.WORKLOADS["tiny"].scene, width=w, height=h, spp=spp, extra_samples=M, **more)
    print(f"trace {w}x{h}x{spp} with {M} extra samples {more}", flush=True)
    compare(cfg)
    ref, rec = scenegen.generate(cfg), traced(cfg)
    for f in ("fb_l_sun", "fb_dir_env", "fb_l_env"):
        a, b = getattr(rec, f).cpu().numpy(), getattr(ref, f)
        ulps = np.abs(a.view(np.int32).astype(np.int64) - b.view(np.int32).astype(np.int64))
        assert np.all((ulps <= 2) | (a == b)), f


@pytest.mark.parametrize("w,h,spp", [(64, 64, 1), (4097, 1, 1), (64, 64, 2), (241, 34, 1), (128, 128, 1), (113, 145, 1),
                                     (128, 128, 2), (149, 220, 1)])
def test_records_where_the_waves_narrow(w, h, spp):
    print(f"trace {w}x{h}x{spp}", flush=True)
    compare(replace(scenegen.WORKLOADS["tiny"].scene, width=w, height=h, spp=spp))

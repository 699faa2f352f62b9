"""pg_gather of an image whose pixels take more threads than one launch may have (2^32 at 64 lanes a pixel)."""
from types import SimpleNamespace

import pytest
import torch

import paper_2404_11894_amd as pg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height", [(8192, 8191), (8192, 8193)])
def test_gather_of_many_pixels(width, height):
    print(f"gather {width}x{height} k=64", flush=True)
    P, N, k = width * height, 200, 64
    gen = torch.Generator(device="cuda").manual_seed(width + height)
    rand = lambda *sh: torch.rand(*sh, generator=gen, device="cuda")  # noqa: E731
    pixel = torch.cat([torch.tensor([0, P // 2, P - 2, P - 1], device="cuda"),
                       torch.randint(1, P - 2, (N - 4,), generator=gen, device="cuda")]).unique()
    N = len(pixel)
    off = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    off[1:][pixel] = 1
    off = off.cumsum(0)
    d = torch.nn.functional.normalize(rand(N, 3) - 0.5, dim=1)
    sc = SimpleNamespace(width=width, height=height, spp=1, path_offsets=off, pos=rand(N, 3), dir_in=d, dir_out=d,
                         albedo=rand(N), l_sun=rand(N, 3), dir_env=d, l_env=rand(N, 3), l_phase=rand(N, 3),
                         e_cam=rand(P, 3))
    paths = pg.DevicePaths(sc)
    row_ptr = torch.arange(N + 1, device="cuda") * k
    col = torch.randint(0, N, (N, k), generator=gen, device="cuda").int()
    w, d_pt, lplus = rand(N, k), rand(N, 3), rand(N, 3)
    image = pg.pg_gather(paths, pg.params(k=k), row_ptr, col.reshape(-1), w.reshape(-1), d_pt, lplus).reshape(P, 3)
    torch.cuda.synchronize()
    inner = (w.double()[..., None] * lplus.double()[col.long()]).sum(1)
    ref = sc.e_cam[pixel].double() + sc.albedo.double()[:, None] * (d_pt.double() + inner)
    assert ((image[pixel].double() - ref).abs() <= 1e-6 * ref).all()
    image[pixel] = sc.e_cam[pixel]
    assert torch.equal(image, sc.e_cam)   # one sample: its camera term as it is

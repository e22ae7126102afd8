"""Depth order and lists at the sizes where one workgroup's scan (6144 counts)
and sort (12,288 keys) give way to the grid's, for depths of many powers of two
(all four of the sort's passes), equal depths (none but the first), and no
visible Gaussian; from raw parameters and from a prepared scene, whose ties are
ordered after the sort.  Integers: exact."""
import numpy as np
import pytest

from gpu_helpers import gpu_frame
from oracle_helpers import identity_camera, opts
from test_gpu_sort_edges import check_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depths", ["wide", "equal", "culled"])
@pytest.mark.parametrize("P", [6143, 6144, 6145, 12287, 12288, 12289, 16385])
def test_small_sort_and_scan(P, depths):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    print(f"[sort limits] P {P} {depths}", flush=True)
    g = torch.Generator().manual_seed(P)
    W, H = 300, 200
    z = {"wide": torch.exp(torch.rand(P, generator=g) * np.log(1e4 / 0.3)) * 0.3,
         "equal": torch.full((P,), 3.0), "culled": torch.full((P,), -1.0)}[depths]
    if depths == "wide":
        z[P // 2: P // 2 + 300] = z[0]  # a long run of equal depths
    x = (torch.rand(P, generator=g) - 0.5) * 0.9 * z * W / 200.0
    y = (torch.rand(P, generator=g) - 0.5) * 0.9 * z * H / 200.0
    ls = torch.log(z.abs() * 0.01).repeat(3, 1)
    sc = GaussianScene(torch.stack([x, y, z]).cuda(), ls.cuda(),
                       torch.tensor([1.0, 0, 0, 0])[:, None].repeat(1, P).cuda(), torch.zeros(1, P).cuda(),
                       torch.zeros(3, P).cuda(), 0)
    cam, o = identity_camera(W, H, 200.0), opts()
    R = Renderer()
    h = R.prepare(sc, o)
    raw, prep = (gpu_frame(R, sc, cam, W, H, o, prepared=p) for p in (None, h))
    R.release_prepared(h)
    R.close()
    assert np.count_nonzero(raw["count"]) == (0 if depths == "culled" else P)
    check_lists(raw, P)
    for f in ("order", "values", "tiles", "count", "ranges", "rgb", "T", "last"):
        assert np.array_equal(raw[f], prep[f]), f

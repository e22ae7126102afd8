"""Sorts at the sizes where their split changes: one tile of 1024 keys per
workgroup up to 2^20 keys, then tiles of 2048, 3072 and 4096 keys, and several
4096-key tiles per workgroup beyond 2^22.  Depth order and the tiles' lists are
integers and have to be exact: order = stable by (depth bits, index), every
tile's list in depth order, every Gaussian in as many lists as its count."""
import numpy as np
import pytest

from gpu_helpers import gpu_frame
from oracle_helpers import identity_camera, opts

pytestmark = pytest.mark.gpu

M = 1 << 20


@pytest.mark.parametrize("P", [1, 255, 1023, 1024, 1025, 4095, 4097, 65537, M - 1, M, M + 1, 2 * M + 1, 3 * M + 1,
                               4 * M, 4 * M + 1])
def test_order_and_lists(P):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    print(f"[sort] P {P}", flush=True)
    g = torch.Generator().manual_seed(P)
    z = 2.0 + 6.0 * torch.rand(P, generator=g)
    z[: P // 3] = z[0]  # one long run of equal depths
    W, H = 1000, 700
    x = (torch.rand(P, generator=g) - 0.5) * 0.9 * z * W / 800.0
    y = (torch.rand(P, generator=g) - 0.5) * 0.9 * z * H / 800.0
    sc = GaussianScene(torch.stack([x, y, z]).cuda(), torch.full((3, P), -7.0).cuda(),
                       torch.tensor([1.0, 0, 0, 0])[:, None].repeat(1, P).cuda(), torch.zeros(1, P).cuda(),
                       torch.zeros(3, P).cuda(), 0)
    R = Renderer()
    r = gpu_frame(R, sc, identity_camera(W, H, 800.0), W, H, opts())
    R.close()
    assert np.count_nonzero(r["count"]) >= 0.99 * P
    check_lists(r, P)


def check_lists(r, P):
    vis = np.nonzero(r["count"])[0]
    bits = r["gauss"][vis, 10].view(np.uint32)
    want = vis[np.lexsort((vis, bits))].astype(np.uint32)
    got = r["order"]
    assert np.array_equal(got[np.isin(got, vis)], want)
    rank = np.full(P, -1, np.int64)
    rank[got] = np.arange(got.size)
    tiles, values = r["tiles"].astype(np.int64), r["values"]
    assert np.array_equal(np.bincount(values, minlength=P), r["count"])
    key = tiles * (P + 1) + rank[values]
    assert np.all(key[1:] > key[:-1])


@pytest.mark.parametrize("log_scale", [-7.0, -3.2, -2.9, -2.5, -2.1, -1.7, -0.5, 1.0])
@pytest.mark.parametrize("P", [3, 300, 3000])
def test_lists_of_wide_gaussians(log_scale, P):
    """From one tile per Gaussian to every tile of a super-tile: the pairs of
    256 entries fill the list writer's buffer whole, by halves, by 64 and by 32
    entries."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    print(f"[lists] P {P} log scale {log_scale}", flush=True)
    g = torch.Generator().manual_seed(P)
    W, H = 300, 270  # 3 x 3 super-tiles, the last row and column cut
    z = 2.0 + torch.rand(P, generator=g)
    x = (torch.rand(P, generator=g) - 0.5) * z * W / 200.0
    y = (torch.rand(P, generator=g) - 0.5) * z * H / 200.0
    sc = GaussianScene(torch.stack([x, y, z]).cuda(), torch.full((3, P), log_scale).cuda(),
                       torch.tensor([1.0, 0, 0, 0])[:, None].repeat(1, P).cuda(), torch.zeros(1, P).cuda(),
                       torch.zeros(3, P).cuda(), 0)
    R = Renderer()
    r = gpu_frame(R, sc, identity_camera(W, H, 200.0), W, H, opts())
    R.close()
    check_lists(r, P)
    print(f"[lists] pairs {r['stats']['pairs']} entries {r['stats']['entries']}", flush=True)

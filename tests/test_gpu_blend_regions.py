"""The blend's region tests at the ends of their range, in both forms of the
blend (one and two pixels per lane, chosen by the number of tiles): footprints
whose terms leave binary32's range, where the image has to be that of the
prefetch variant, which tests no regions, bit for bit."""
import numpy as np
import pytest

from oracle_helpers import identity_camera, opts, scene_from

pytestmark = pytest.mark.gpu
SIZES = [(200, 136), (2064, 1280)]  # one and two pixels per lane


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import Renderer
    r = Renderer()
    yield r
    r.close()


def both_variants(R, sc, cam, W, H):
    import torch
    from paper_2408_07967_amd import binding as B
    from paper_2408_07967_amd.render import GaussianScene
    gsc, o = GaussianScene.from_numpy(sc), opts(bg=[0.3, 0.1, 0.2])
    out = R.render(gsc, cam, W, H, o, want_T=True, want_last=True)
    R.set_blend_variant(B.BLEND_PREFETCH)
    pre = R.render(gsc, cam, W, H, o, want_T=True, want_last=True)
    R.set_blend_variant(B.BLEND_LDS_BATCHES)
    torch.cuda.synchronize()
    return out, pre


@pytest.mark.parametrize("W,H", SIZES)
@pytest.mark.parametrize("log_scale", [14.0, 18.0, 18.5, 19.5, 22.0])
def test_footprints_of_billions_of_pixels(orc, R, log_scale, W, H):
    """The product of the conic's entries underflows from about 19 on."""
    import torch
    print(f"[regions] log scale {log_scale} {W}x{H}", flush=True)
    P = 5
    sc = scene_from([[0.05, 0.02, 2.0 + 0.1 * i] for i in range(P)], np.full((P, 3), log_scale),
                    np.tile([1.0, 0, 0, 0], (P, 1)), np.linspace(-2.0, 0.0, P), dc_rgb=[0.6, 0.4, 0.2])
    cam = identity_camera(W, H, 100.0)
    out, pre = both_variants(R, sc, cam, W, H)
    for k in ("rgb", "T", "last"):
        assert torch.equal(out[k], pre[k]), k
    assert torch.all(out["last"] == P)  # every Gaussian reaches every pixel
    ref = orc.render(sc.astype(np.float64), cam, W, H, opts(bg=[0.3, 0.1, 0.2]), "f64")
    assert np.abs(out["rgb"].cpu().numpy() - ref["rgb"]).max() <= 1e-5

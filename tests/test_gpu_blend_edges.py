"""The blend's two forms (one and two pixels per lane, chosen by the number of
tiles) where they can go wrong: lists around a batch and around a pair,
pixels that saturate at the first or the second Gaussian of a pair, images
that cut the regions, and both sides of the line between the forms.  Images,
transmittance and last contributor against the oracle's binary64 blend, and
the prefetch variant's image bit for bit."""
import numpy as np
import pytest

from gpu_helpers import IMG_FRAC, IMG_MAX, IMG_MEAN
from oracle_helpers import identity_camera, opts, random_scene, scene_from

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import Renderer
    r = Renderer()
    yield r
    r.close()


def check(orc, R, sc, cam, W, H, o, tag):
    import torch
    from paper_2408_07967_amd import binding as B
    from paper_2408_07967_amd.render import GaussianScene
    print(f"[blend] {tag} {W}x{H}", flush=True)
    gsc = GaussianScene.from_numpy(sc)
    out = R.render(gsc, cam, W, H, o, want_T=True, want_last=True)
    R.set_blend_variant(B.BLEND_PREFETCH)
    pre = R.render(gsc, cam, W, H, o, want_T=True, want_last=True)
    R.set_blend_variant(B.BLEND_LDS_BATCHES)
    torch.cuda.synchronize()
    for k in ("rgb", "T", "last"):
        assert torch.equal(out[k], pre[k]), f"{tag}: {k} differs from the prefetch variant"
    ref = orc.render(sc.astype(np.float64), cam, W, H, o, "f64")
    d = np.abs(out["rgb"].cpu().numpy() - ref["rgb"]).max(0)
    dT = np.abs(out["T"].cpu().numpy() - ref["T"])
    assert (d <= IMG_MAX).mean() >= IMG_FRAC and d.mean() <= IMG_MEAN, (tag, d.max(), d.mean())
    assert (dT <= IMG_MAX).mean() >= IMG_FRAC and dT.mean() <= IMG_MEAN, (tag, dT.max(), dT.mean())
    same = out["last"].cpu().numpy().view(np.uint32) == ref["last"]
    assert same.mean() >= 0.995, (tag, same.mean())


@pytest.mark.parametrize("P", [1, 2, 3, 63, 64, 65, 127, 128, 129, 255, 256, 257, 513])
@pytest.mark.parametrize("W,H", [(16, 16), (17, 9), (7, 1)])
def test_list_lengths(orc, R, P, W, H):
    rng = np.random.default_rng(2000 + P)
    sc = scene_from(np.stack([rng.uniform(-0.3, 0.3, P), rng.uniform(-0.3, 0.3, P), rng.uniform(3.0, 6.0, P)], 1),
                    rng.normal(0.0, 0.2, (P, 3)), rng.normal(0.0, 1.0, (P, 4)), rng.uniform(-4.5, -4.0, P),
                    dc_rgb=[0.6, 0.4, 0.2])
    check(orc, R, sc, identity_camera(W, H, 18.0), W, H, opts(bg=[0.2, 0.1, 0.4]), f"list {P}")


@pytest.mark.parametrize("clear", [0, 1, 2, 3])
def test_saturation_within_a_pair(orc, R, clear):
    """Opaque Gaussians behind `clear` faint ones: T passes the threshold at
    the first or at the second Gaussian of a pair."""
    P = clear + 6
    z = 3.0 + 0.5 * np.arange(P)
    sc = scene_from(np.stack([np.zeros(P), np.zeros(P), z], 1), np.full((P, 3), 0.7), np.tile([1.0, 0, 0, 0], (P, 1)),
                    [-4.0] * clear + [6.0] * 6, dc_rgb=[0.6, 0.4, 0.2])
    check(orc, R, sc, identity_camera(16, 16, 18.0), 16, 16, opts(), f"saturate {clear}")


@pytest.mark.parametrize("W,H", [(2048, 1280), (2064, 1280)])  # 10240 tiles and 10320
def test_both_sides_of_the_line(orc, R, W, H):
    sc = random_scene(np.random.default_rng(5), 20000, ls_mu=-3.5, sh_degree=1)
    check(orc, R, sc, identity_camera(W, H, 0.9 * W), W, H, opts(), "line")

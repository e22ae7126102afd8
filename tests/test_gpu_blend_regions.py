"""The blend's region tests at the ends of their range, in both forms of the
blend (one and two pixels per lane, chosen by the number of tiles): footprints
whose terms leave binary32's range, where the image has to be that of the
prefetch variant, which tests no regions, bit for bit; and footprints thousands
of times longer than wide, where the adjoint has to replay what the forward
blended."""
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


def needle(rng, W, H, f=500.0, z=2.0):
    """One Gaussian in a random direction of the image plane, 1000 to 6000
    pixels (standard deviation) long and as narrow as the low-pass leaves it."""
    th, s1 = rng.uniform(0.0, np.pi), np.exp(rng.uniform(np.log(1000.0), np.log(6000.0)))
    t = rng.uniform(-2.0, 2.0) * s1
    x, y = rng.uniform(-0.4, 0.4) * W + t * np.cos(th), rng.uniform(-0.4, 0.4) * H + t * np.sin(th)
    return scene_from([[x * z / f, y * z / f, z]], [[np.log(s1 * z / f), -9.0, -9.0]],
                      [[np.cos(th / 2), 0, 0, np.sin(th / 2)]], [rng.uniform(0.0, 4.0)], dc_rgb=[0.6, 0.4, 0.2])


@pytest.mark.parametrize("W,H", SIZES)
def test_needle_adjoint_replays_the_forward(R, W, H):
    """For one Gaussian and dL/dR = 1 the colour's gradient is the sum over the
    pixels of its weights, which is the sum of 1 - T of the forward.  Each
    weight carries a few binary32 roundings, as does 1 - T (at least 1/255
    where it is not 0: 1.5e-5 relative at worst)."""
    import torch
    from paper_2408_07967_amd.render import GaussianScene
    rng = np.random.default_rng(4)
    cam = identity_camera(W, H, 500.0)
    o = opts()
    dL = torch.zeros(3, H, W, device="cuda")
    dL[0] = 1.0
    bad = []
    for k in range(300 if W < 1000 else 60):
        gsc = GaussianScene.from_numpy(needle(rng, W, H))
        out = R.render(gsc, cam, W, H, o, want_T=True, save=True)
        g = R.backward(out["frame"], gsc, cam, W, H, o, dL)
        got = float(g[4][0, 0]) / 0.28209479177387814
        want = float((1.0 - out["T"].double()).sum())
        R.release(out["frame"])
        if abs(got - want) > 3e-5 * want:
            bad.append((k, got, want))
    print(f"[regions] adjoint {W}x{H}: {len(bad)} differ {bad[:8]}", flush=True)
    assert not bad

"""A prepared scene built in the block that a released one left: frames from it
equal the raw-parameter frames bit for bit, for sizes around a workgroup,
every SH degree (record strides 4, 12, 28 and 48 floats) and blocks that fit,
that are too small and that are too large to take."""
import numpy as np
import pytest

from oracle_helpers import identity_camera, opts, random_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
def test_frames_after_release_and_prepare(deg):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    R = Renderer()
    W, H = 97, 61
    cam, o = identity_camera(W, H, 80.0), opts(bg=[0.1, 0.2, 0.3])
    for k, P in enumerate((5000, 4000, 257, 256, 255, 1, 30000, 20000, 64, 0, 12000)):
        print(f"[prepare] degree {deg} P {P}", flush=True)
        sc = random_scene(np.random.default_rng(100 * deg + k), P, ls_mu=-2.5, sh_degree=deg)
        gsc = GaussianScene.from_numpy(sc)
        h = R.prepare(gsc, o)
        a = R.render(gsc, cam, W, H, o, want_T=True, want_last=True, prepared=h)
        b = R.render(gsc, cam, W, H, o, want_T=True, want_last=True)
        torch.cuda.synchronize()
        for f in ("rgb", "T", "last"):
            assert torch.equal(a[f], b[f]), (P, f)
        assert a["stats"]["pairs"] == b["stats"]["pairs"]
        R.release_prepared(h)
    R.close()

"""GPU parity of the blend adjoint where its batches and matrix products have
edges: lists of one more and one less than a product's eight Gaussians and
than a batch's 128, images that cut the tile's quadrants, and footprints whose
centre lies far outside the image (the sums are taken about the tile's centre
and moved to the Gaussian's).  Reference: the oracle's binary64 adjoint, with
the backward tests' bar (1e-3 relative with a floor of 1e-5 of the group's
largest entry)."""
import numpy as np
import pytest

from oracle_helpers import identity_camera, opts, random_scene, scene_from
from test_gpu_backward import R, compare, gpu_grads  # noqa: F401  (R: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 7, 8, 9, 127, 128, 129, 257])
@pytest.mark.parametrize("W,H", [(16, 16), (9, 7), (1, 1)])
def test_one_tile_list_lengths(orc, R, P, W, H):  # noqa: F811
    """Every Gaussian covers the tile; low opacities keep every pixel open."""
    print(f"[bwd] list {P} {W}x{H}", flush=True)
    rng = np.random.default_rng(1000 + P)
    sc = scene_from(np.stack([rng.uniform(-0.3, 0.3, P), rng.uniform(-0.3, 0.3, P), rng.uniform(3.0, 6.0, P)], 1),
                    rng.normal(0.0, 0.2, (P, 3)), rng.normal(0.0, 1.0, (P, 4)), rng.uniform(-4.0, -3.0, P),
                    dc_rgb=[0.6, 0.4, 0.2])
    cam = identity_camera(W, H, 18.0)
    o = opts(bg=[0.2, 0.1, 0.4])
    w = np.random.default_rng(7).uniform(-1, 1, (3, H, W))
    g, _, dL = gpu_grads(R, sc, cam, W, H, o, dL=w)
    ref = orc.backward(orc.render(sc.astype(np.float64), cam, W, H, o, "f64"), dL)
    compare(g, ref, f"list{P}")


@pytest.mark.parametrize("seed,W,H", [(31, 48, 32), (32, 33, 17)])
def test_centres_far_outside(orc, R, seed, W, H):  # noqa: F811
    """Wide footprints centred up to several image widths away."""
    print(f"[bwd] far {seed} {W}x{H}", flush=True)
    rng = np.random.default_rng(seed)
    P = 150
    sc = random_scene(rng, P, ls_mu=-0.2, sh_degree=1)
    sc.means[0] = rng.uniform(-6.0, 6.0, P).astype(np.float32)
    cam = identity_camera(W, H, 0.9 * W)
    o = opts()
    w = np.random.default_rng(seed + 100).uniform(-1, 1, (3, H, W))
    g, _, dL = gpu_grads(R, sc, cam, W, H, o, dL=w)
    ref = orc.backward(orc.render(sc.astype(np.float64), cam, W, H, o, "f64"), dL)
    compare(g, ref, f"far{seed}", min_frac=0.99)


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("P", [1, 63, 65, 300])
def test_culled_among_seen(orc, R, deg, P):  # noqa: F811
    """Every third Gaussian is behind the camera: exact zeros there, in the
    lines of the seen ones' gradients."""
    print(f"[bwd] culled degree {deg} P {P}", flush=True)
    rng = np.random.default_rng(100 * deg + P)
    W, H = 40, 30
    sc = random_scene(rng, P, ls_mu=-2.5, sh_degree=deg)
    sc.means[2, 1::3] = -3.0
    cam = identity_camera(W, H, 0.9 * W)
    o = opts()
    w = np.random.default_rng(8).uniform(-1, 1, (3, H, W))
    g, _, dL = gpu_grads(R, sc, cam, W, H, o, dL=w)
    for name in g:
        assert np.all(g[name][:, 1::3] == 0.0), name
    ref = orc.backward(orc.render(sc.astype(np.float64), cam, W, H, o, "f64"), dL)
    compare(g, ref, f"culled{deg}-{P}")

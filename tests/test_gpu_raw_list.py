"""Raw frames of more Gaussians than one per lane of the grid list the possibly
visible ones first and pack their outputs: the same frame as the one-pass path
renders, bit for bit.  A small scene (one pass) is spread over a large one whose
other Gaussians cannot be seen, in the same order, with parameters at the edges
of the list's keep test: beyond the image's borders, at the near plane, faint,
huge, degenerate, non-finite and equally deep."""
import dataclasses

import numpy as np
import pytest

from oracle_helpers import identity_camera, opts, random_scene

pytestmark = pytest.mark.gpu


def edge_scene(rng, P, deg):
    sc = random_scene(rng, P, box=3.0, ls_mu=-3.0, ls_sigma=1.2, sh_degree=deg, z0=3.0)
    m, ls, q, lg, sh = (np.array(a, np.float32) for a in (sc.means, sc.log_scales, sc.quats, sc.logits, sc.sh))
    lg = lg.reshape(1, P)
    k = rng.permutation(P)
    part = [k[i::16] for i in range(16)]
    m[2, part[0]] = 0.2 + rng.uniform(-1e-6, 1e-6, part[0].size)     # at the near plane
    m[0, part[1]] = m[2, part[1]] * rng.uniform(0.9, 1.1, part[1].size)  # at the border (f = W / 2)
    lg[0, part[2]] = np.log(1 / 254.0) + rng.uniform(-2e-2, 2e-2, part[2].size)  # at the opacity limit
    ls[:, part[3]] += 4.0
    ls[0, part[4]] += 9.0                                            # needles across the image
    q[:, part[5]] *= 1e-22                                           # squared norm without precision
    q[:, part[6]] *= 1e15
    m[2, part[7]] = 2.5                                              # equal depths
    m[0, part[8][:4]] = [np.nan, np.inf, -np.inf, 3e38]
    lg[0, part[8][4:7]] = [np.nan, np.inf, -np.inf]
    ls[1, part[8][7:11]] = [np.nan, np.inf, -np.inf, 80.0]
    q[:, part[8][11]] = 0.0
    sh[0, part[8][12:14]] = [np.nan, np.inf]
    return dataclasses.replace(sc, means=m, log_scales=ls, quats=q, logits=lg, sh=sh)


def spread(sc, rng, total):
    P = sc.means.shape[1]
    at = np.sort(rng.choice(total, P, replace=False))

    def grow(a, fill):
        a = np.asarray(a, np.float32).reshape(-1, P)
        out = np.empty((a.shape[0], total), np.float32)
        out[:] = fill
        out[:, at] = a
        return out

    means = grow(sc.means, 0.0)
    hidden = np.ones(total, bool)
    hidden[at] = False
    means[2, hidden] = rng.choice([-5.0, 0.1, 4.0], hidden.sum())
    means[0, hidden & (means[2] == 4.0)] = 60.0  # off the image
    return dataclasses.replace(sc, means=means, log_scales=grow(sc.log_scales, -2.0), quats=grow(sc.quats, 0.5),
                               logits=grow(sc.logits, 1.0), sh=grow(sc.sh, 0.1))


@pytest.mark.parametrize("deg,options,total", [
    (0, {}, 262_145), (1, dict(binning=1), 300_000), (2, dict(binning=2), 400_001),
    (3, dict(cap_3sigma=0), 1_000_000), (3, dict(alpha_min=0.3), 524_288), (3, dict(jac_clip=1.0, dilation=0.0), 700_003)])
def test_listed_equals_one_pass(deg, options, total):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    rng = np.random.default_rng(total)
    W, H = 333, 250
    cam, o = identity_camera(W, H, W / 2.0), opts(**options)
    small = edge_scene(rng, 20_000, deg)
    large = spread(small, rng, total)
    R = Renderer()
    print(f"[raw list] degree {deg} {options} {total}", flush=True)
    a = R.render(GaussianScene.from_numpy(small), cam, W, H, o, want_T=True, want_last=True)
    gl = GaussianScene.from_numpy(large)
    b = R.render(gl, cam, W, H, o, want_T=True, want_last=True)
    c = R.render(gl, cam, W, H, o, want_T=True, want_last=True, save=True)  # kept: outputs by Gaussian
    torch.cuda.synchronize()
    assert a["stats"]["visible"] > 1000
    for x in (b, c):
        for f in ("visible", "pairs", "entries"):
            assert a["stats"][f] == x["stats"][f], f
        for f in ("rgb", "T", "last"):
            assert torch.equal(a[f].view(torch.int32), x[f].view(torch.int32)), f
    R.release(c["frame"])
    R.close()

"""Row intervals of the large rectangles' tile tests.

CPU: no tile that the oracle's exact test hits lies outside a row's interval,
and every tile that the interval calls certain is hit, on random and
adversarial ellipses (aligned, diagonal and needle-like ones, centres on tile
and sample boundaries and far outside, ragged images).

GPU: pairs and states against the binary32 oracle, bit for bit, on scenes of
rectangles around a chunk (64 and 256 tiles), of needles too thin for
intervals, and of both together, in the exact and the box binning."""
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from gpu_helpers import check_gauss_state, check_pairs, gpu_frame
from oracle_helpers import identity_camera, opts, scene_from

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang not installed")
def test_intervals_against_the_exact_test():
    td = tempfile.mkdtemp(prefix="fgs_rows_")
    try:
        orc = os.path.join(ROOT, "oracle")
        for src, defs, o in (("orc_core.c", ["-DORC_FP32"], "core.o"), ("orc_math.c", [], "math.o")):
            subprocess.run(["gcc", "-std=c11", "-O2", "-ffp-contract=off", "-I", orc, *defs, "-c",
                            os.path.join(orc, src), "-o", os.path.join(td, o)], check=True)
        exe = os.path.join(td, "tile_rows")
        subprocess.run([CLANG, "-std=c++17", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2408_07967_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "tile_rows_driver.cpp"), os.path.join(td, "core.o"),
                        os.path.join(td, "math.o"), "-lm", "-o", exe], check=True)
        r = subprocess.run([exe, "15000", "1"], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0 and " bad 0" in r.stdout, r.stdout
    finally:
        shutil.rmtree(td, ignore_errors=True)


def _scene(rng, P, axes, f, W, H):
    """P Gaussians at depth 4 whose footprints have the given pixel axes
    (standard deviations), at random angles and centres in and around the image."""
    z = 4.0
    x = rng.uniform(-0.2, 1.2, P) * W - W / 2
    y = rng.uniform(-0.2, 1.2, P) * H - H / 2
    means = np.stack([x * z / f, y * z / f, z + rng.uniform(0, 0.5, P)], 1)
    s = np.stack([axes[0] * z / f * np.exp(rng.normal(0, 0.3, P)), axes[1] * z / f * np.exp(rng.normal(0, 0.3, P)),
                  np.full(P, 0.01)], 1)
    th = rng.choice([0.0, np.pi / 2, np.pi / 4, -1.0], P) + rng.normal(0, 1e-3, P)
    th = np.where(rng.random(P) < 0.5, th, rng.uniform(0, np.pi, P))
    q = np.stack([np.cos(th / 2), np.zeros(P), np.zeros(P), np.sin(th / 2)], 1)
    return scene_from(means, np.log(s), q, rng.normal(0, 1.5, P), dc_rgb=[0.6, 0.4, 0.2])


@pytest.mark.gpu
@pytest.mark.parametrize("binning", [0, 1])
@pytest.mark.parametrize("tag,axes,W,H", [
    ("64 tiles", (21.0, 21.0), 1021, 777),
    ("256 tiles", (43.0, 41.0), 1021, 777),
    ("wide", (300.0, 30.0), 2049, 333),
    ("needles", (400.0, 0.02), 1280, 720),
    ("thin", (200.0, 1.0), 1280, 720),
    ("screen", (1500.0, 900.0), 641, 359),
])
def test_pairs_of_large_rectangles(orc, tag, axes, W, H, binning):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    print(f"[rows] {tag} {W}x{H} binning {binning}", flush=True)
    R = Renderer()
    f = 0.8 * W
    sc = _scene(np.random.default_rng(17), 700, axes, f, W, H)
    cam, o = identity_camera(W, H, f), opts(binning=binning)
    g = gpu_frame(R, GaussianScene.from_numpy(sc), cam, W, H, o)
    o32 = orc.render(sc, cam, W, H, o, mode="f32")
    assert g["stats"]["big_chunks"] > 0
    check_gauss_state(orc, g, o32)
    check_pairs(g, o32)
    R.close()

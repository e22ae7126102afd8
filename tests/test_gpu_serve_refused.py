"""Refused and admitted requests of mixed sizes share a server's four slots: a
refused request frees its slot while its depth order may still run, and the
slot's next request may start in a first half that other slots share.  Every
admitted image equals the plain render bit for bit."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [400_000, 9_000])
def test_refused_requests_leave_the_others_images_alone(P):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_07967_amd import binding as B
    from paper_2408_07967_amd import scenes
    from paper_2408_07967_amd.render import GaussianScene, Renderer
    from paper_2408_07967_amd.serve import RenderServer
    sc = scenes.make_scene("serve", P=P)
    if P < 10_000:
        sc.log_scales += 1.5  # (the least budget holds about 58,000 pairs)
    gsc = GaussianScene.from_numpy(sc)
    R = Renderer()
    rng = np.random.default_rng(21)

    def pose(W, H, fov):
        th, h = rng.uniform(0.0, 2.0 * math.pi), rng.uniform(50.0, 150.0)
        return scenes.look_at((200.0 * math.cos(th), h, 200.0 * math.sin(th)), (0.0, 0.0, 0.0), W, H, fov)

    # every third request sees the whole scene, the others a few degrees of it
    reqs, alone = [], {}
    for rid in range(48):
        W, H, fov = (2560, 1440, 70.0) if rid % 3 == 1 else ((320, 180, 6.0), (200, 333, 9.0))[rid % 2]
        cam = pose(W, H, fov)
        out = R.render(gsc, cam, W, H)
        reqs.append((rid, cam, W, H))
        alone[rid] = (out["rgb"].clone(), out["stats"])
    large = min(s["pairs"] for r, (_, s) in alone.items() if r % 3 == 1)
    small = max(max(s["pairs"], 3 * s["entries"] + 4096) for r, (_, s) in alone.items() if r % 3 != 1)
    budget = max(16 * large - 4096, 1 << 20)
    print(f"[refused] P {P} budget {budget} large {large} small {small}", flush=True)
    assert 18 * (large + 4096) > budget > 18 * (small + 4096)  # the scene's own pairs separate the two kinds
    torch.cuda.synchronize()
    srv = RenderServer(gsc, budget_bytes=budget, max_inflight=4, max_width=2560, max_height=1440)
    outs = {rid: torch.empty(3 * W * H, device="cuda") for rid, _, W, H in reqs}
    got = {}
    try:
        # a few at a time: slots are refused and taken again all along
        for k in range(0, len(reqs), 6):
            for rid, cam, W, H in reqs[k:k + 6]:
                srv.submit(rid, cam, W, H, out=outs[rid])
            while len(got) < k + 3:
                for r in srv.poll(wait_s=0.5):
                    got[r["id"]] = r
                    if r["status"] == 0:
                        srv.release(r["id"])
        while len(got) < len(reqs):
            for r in srv.poll(wait_s=0.5):
                got[r["id"]] = r
                if r["status"] == 0:
                    srv.release(r["id"])
        st = srv.stats()
    finally:
        srv.close()
    torch.cuda.synchronize()
    R.close()
    print(f"[refused] {st}", flush=True)
    assert st["batched_fronts"] >= 1
    for rid, cam, W, H in reqs:
        if rid % 3 == 1:
            assert got[rid]["status"] == B.FGS_ERR_CAPACITY, got[rid]
        else:
            assert got[rid]["status"] == 0, got[rid]
            assert got[rid]["pairs"] == alone[rid][1]["pairs"]
            assert torch.equal(outs[rid].view(3, H, W), alone[rid][0]), f"request {rid} ({W}x{H})"

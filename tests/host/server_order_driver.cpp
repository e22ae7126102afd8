// Ordering of the render server's device work, checked on the host with
// stand-ins for the device (fake_device.hpp).  The scenario: slots 0 and 1 hold
// finished images, slot 2's request can never fit the budget and is refused.  The
// images are released, a request occupies slot 0, and two more that start
// together share one preprocess on slot 1's stream, which writes slot 2's
// buffers: its refused request's depth order must be behind it.
#include "fake_device.hpp"

namespace {

int g_failures = 0;
void check(bool ok, const char *what) {
    if (!ok) {
        std::fprintf(stderr, "FAILED: %s\n", what);
        ++g_failures;
    }
}

fgs_server_result wait_one(fgs_server *srv) {
    fgs_server_result r{};
    for (int k = 0; k < 1000; ++k)
        if (fgs_server_poll(srv, &r, 1, 20'000'000) == 1) return r;
    std::fprintf(stderr, "no request completed\n");
    std::exit(1);
}

}  // namespace

int main(int argc, char **argv) {
    const int P = argc > 1 ? std::atoi(argv[1]) : 100000;  // at most 16384: the depth order of one workgroup
    std::vector<float> planes(16, 0.0f);
    fgs_scene sc{};
    sc.num_gaussians = sc.plane_stride = P;
    sc.means = sc.log_scales = sc.quats = sc.opacity_logits = sc.sh = planes.data();
    fgs_camera cam{};
    cam.R[0] = cam.R[4] = cam.R[8] = 1.0f;
    cam.fx = cam.fy = 100.0f;
    cam.near_z = 0.2f;
    fgs_server_config cfg{};
    cfg.budget_bytes = 64 << 20;
    cfg.max_inflight = 4;
    cfg.max_width = cfg.max_height = 128;
    cfg.max_bypass = 1;
    cfg.use_graphs = 0;
    cfg.share_queue = 0;
    cfg.batch_fronts = 1;
    fgs_server *srv = nullptr;
    check(fgs_server_create(0, &sc, nullptr, &cfg, &srv) == FGS_OK, "server created");
    auto submit = [&](uint64_t id, int W) {
        check(fgs_server_submit(srv, id, &cam, W, 64, 0, nullptr) == FGS_OK, "request accepted");
    };
    for (uint64_t id = 0; id < 2; ++id) {  // one after the other: slots 0 and 1
        submit(id, 64);
        const fgs_server_result r = wait_one(srv);
        check(r.status == FGS_OK && r.slot == (int)id, "an image held in slots 0 and 1");
    }
    submit(2, kRefusedWidth);
    const fgs_server_result bad = wait_one(srv);
    check(bad.status == FGS_ERR_CAPACITY && bad.slot == 2, "slot 2's request is refused");
    check(g_refused_orders == 1, "its first half ran");
    for (uint64_t id = 0; id < 2; ++id) check(fgs_server_release(srv, id) == FGS_OK, "image released");
    // the worker takes this one alone and stops in its launch until the two
    // that are to start together are queued
    submit(3, kGateWidth);
    {
        std::unique_lock<std::mutex> lk(g_gate_mu);
        g_gate_cv.wait(lk, [] { return g_gate_reached; });
    }
    submit(4, 64);
    submit(5, 64);
    {
        std::lock_guard<std::mutex> lk(g_gate_mu);
        g_gate_open = true;
    }
    g_gate_cv.notify_all();
    bool reused = false;
    for (int k = 0; k < 3; ++k) {
        const fgs_server_result r = wait_one(srv);
        check(r.status == FGS_OK, "the later requests complete");
        reused |= r.id == 5 && r.slot == 2;
    }
    check(reused, "slot 2 was the second member of a shared first half");
    fgs_server_stats st{};
    check(fgs_server_get_stats(srv, &st) == FGS_OK, "stats");
    check(st.batched_fronts == 1 && st.batched_requests == 2, "one shared first half");
    fgs_server_destroy(srv);
    check(g_races == 0, "every access of a slot's buffers is ordered");
    check(g_bad_pointers == 0, "every launch has its buffers");
    if (g_failures) return 1;
    std::printf("order ok\n");
    return 0;
}

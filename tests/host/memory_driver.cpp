// The runtime at the end of device memory, checked on the host with stand-ins
// for the device (fake_device.hpp).
//   growth  every allocation of a large frame fails in turn; the call reports it
//           (or succeeds without), and a small frame after it gets all its
//           buffers: a launch with a null or freed one would fault a device.
//   spare   a released scene's block that a context keeps for the next one is
//           given back when another context, or a server, needs the memory, and
//           is not kept at all where memory is short.
//   threads contexts of several threads prepare and release scenes while the
//           memory holds two of three.
#include <thread>

#include "fake_device.hpp"

namespace {

int g_failures = 0;
void check(bool ok, const std::string &what) {
    if (!ok) {
        std::fprintf(stderr, "FAILED: %s\n", what.c_str());
        ++g_failures;
    }
}

float g_planes[16];
fgs_scene scene(int64_t P) {
    fgs_scene s{};
    s.num_gaussians = s.plane_stride = P;
    s.means = s.log_scales = s.quats = s.opacity_logits = s.sh = g_planes;
    return s;
}
fgs_camera camera() {
    fgs_camera c{};
    c.R[0] = c.R[4] = c.R[8] = 1.0f;
    c.fx = c.fy = 100.0f;
    c.near_z = 0.2f;
    return c;
}
fgs_context *context() {
    fgs_context *ctx = nullptr;
    check(fgs_create(0, &ctx) == FGS_OK, "context");
    return ctx;
}

enum Mode { RAW, KEPT, PREPARED, BATCH, ADJOINT, MODES };
fgs_status frame(fgs_context *ctx, Mode mode, int64_t P, int W, uint32_t pairs) {
    const fgs_scene sc = scene(P);
    const fgs_camera cams[3] = {camera(), camera(), camera()};
    g_pairs = pairs;
    g_entries = pairs / 2;
    float out[4];
    float *outs[3] = {out, out, out};
    fgs_status st = FGS_OK;
    if (mode == RAW) return fgs_render(ctx, &sc, cams, W, W, nullptr, out, nullptr, nullptr, nullptr, nullptr, nullptr);
    if (mode == KEPT || mode == ADJOINT) {
        fgs_frame *f = nullptr;
        g_kept = true;
        st = fgs_render(ctx, &sc, cams, W, W, nullptr, out, nullptr, nullptr, &f, nullptr, nullptr);
        g_kept = false;
        if (st == FGS_OK && mode == ADJOINT) {
            const fgs_scene_grad g{P, out, out, out, out, out};
            st = fgs_render_backward(ctx, f, &sc, nullptr, nullptr, out, &g, nullptr);
        }
        check(fgs_frame_release(ctx, f) == FGS_OK, "frame released");
        return st;
    }
    fgs_prepared *p = nullptr;
    st = fgs_prepare_scene(ctx, &sc, nullptr, &p, nullptr);
    if (st != FGS_OK) return st;
    st = mode == PREPARED
             ? fgs_render_prepared(ctx, p, cams, W, W, nullptr, out, nullptr, nullptr, nullptr, nullptr, nullptr)
             : fgs_render_prepared_batch(ctx, p, cams, 3, W, W, nullptr, outs, nullptr, nullptr, nullptr, nullptr);
    check(fgs_prepared_release(ctx, p) == FGS_OK, "scene released");
    return st;
}

void growth() {
    for (int mode = 0; mode < MODES; ++mode) {
        int failed = 0;
        for (int k = 0; k < 80; ++k) {
            fgs_context *ctx = context();
            const std::string tag = "mode " + std::to_string(mode) + ", allocation " + std::to_string(k);
            check(frame(ctx, (Mode)mode, 20'000, 64, 1000) == FGS_OK, tag + ": a small frame");
            g_fail_in = k;
            const fgs_status st = frame(ctx, (Mode)mode, 2'000'000, 512, 40'000'000);
            const bool hit = g_fail_in == -1;
            g_fail_in = -1;
            failed += hit;
            check(st == FGS_OK || (hit && st == FGS_ERR_OUT_OF_MEMORY), tag + ": reported");
            check(frame(ctx, (Mode)mode, 20'000, 64, 1000) == FGS_OK, tag + ": a small frame after it");
            check(frame(ctx, (Mode)mode, 20'000, 512, 1000) == FGS_OK, tag + ": a wider one");
            check(frame(ctx, (Mode)mode, 2'000'000, 512, 40'000'000) == FGS_OK, tag + ": the large one");
            fgs_destroy(ctx);
            if (!hit) break;  // past the last allocation
        }
        check(failed > 3, "mode " + std::to_string(mode) + ": allocations failed");
    }
    check(g_bad_pointers == 0, "every launch has its buffers");
}

void spare() {
    const int64_t P = 400'000;
    fgs_context *a = context();
    check(frame(a, PREPARED, P, 64, 1000) == FGS_OK, "a scene in the first context");
    const size_t with = g_used;
    check(frame(a, PREPARED, P / 3, 64, 1000) == FGS_OK && g_used <= with, "a smaller scene holds no more");
    size_t block = 0;
    for (auto &x : g_alloc) block = x.second > block ? x.second : block;
    // room for a second context's frame and precompute only without the block
    const size_t roomy = g_limit;
    for (int round = 0; round < 3; ++round) {
        check(frame(a, PREPARED, P, 64, 1000) == FGS_OK, "the first context again");
        fgs_context *b = nullptr;
        fgs_server *srv = nullptr;
        const size_t held = g_used;
        g_limit = held + block - 1;
        if (round < 2) {
            b = context();
            // (needs more than the rest, less than the rest and the block)
            check(frame(b, round == 0 ? PREPARED : BATCH, round == 0 ? P / 4 : P / 8, 64, 1000) == FGS_OK,
                  "a second context gets the memory that the first one keeps");
        } else {
            fgs_server_config cfg{};
            cfg.budget_bytes = (int64_t)block;
            cfg.max_inflight = 1;
            cfg.max_width = cfg.max_height = 64;
            const fgs_scene sc = scene(1000);
            check(fgs_server_create(0, &sc, nullptr, &cfg, &srv) == FGS_OK,
                  "a server gets the memory that a context keeps");
        }
        check(g_used <= g_limit, "within the memory");
        fgs_destroy(b);
        fgs_server_destroy(srv);
        g_limit = roomy;
    }
    // memory is short: a released scene's block is freed at once
    check(frame(a, PREPARED, P, 64, 1000) == FGS_OK, "the first context again");
    const size_t before = g_used;
    g_limit = before + block / 2;
    const fgs_scene sc = scene(P);
    fgs_prepared *p = nullptr;
    check(fgs_prepare_scene(a, &sc, nullptr, &p, nullptr) == FGS_OK, "the kept block serves");
    check(fgs_prepared_release(a, p) == FGS_OK && g_used <= before - block, "freed where memory is short");
    g_limit = roomy;
    fgs_destroy(a);
    check(g_used == 0, "all memory given back");
}

void threads() {
    const int64_t P = 100'000;
    fgs_context *probe = context();
    check(frame(probe, PREPARED, P, 64, 1000) == FGS_OK, "a scene");
    const size_t one = g_used;
    fgs_destroy(probe);
    const size_t roomy = g_limit;
    g_limit = 3 * one;  // (a scene being prepared takes temporary memory too)
    std::vector<std::thread> ts;
    for (int t = 0; t < 3; ++t)
        ts.emplace_back([&] {
            fgs_context *ctx = nullptr;
            if (fgs_create(0, &ctx) != FGS_OK) return;
            const fgs_scene sc = scene(P);
            for (int k = 0; k < 300; ++k) {
                fgs_prepared *p = nullptr;
                const fgs_status st = fgs_prepare_scene(ctx, &sc, nullptr, &p, nullptr);
                if (st != FGS_OK && st != FGS_ERR_OUT_OF_MEMORY) std::abort();
                if (fgs_prepared_release(ctx, p) != FGS_OK) std::abort();
            }
            fgs_destroy(ctx);
        });
    for (std::thread &t : ts) t.join();
    g_limit = roomy;
    check(g_used == 0, "all memory given back after the threads");
    check(g_bad_pointers == 0, "every launch has its buffers");
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "growth") growth();
    else if (what == "spare") spare();
    else if (what == "threads") threads();
    else return 2;
    if (g_failures) return 1;
    std::printf("memory ok\n");
    return 0;
}

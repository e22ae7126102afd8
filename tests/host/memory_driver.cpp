// The runtime at the end of device memory, checked on the host with stand-ins
// for the device (fake_device.hpp).
//   growth  every allocation of a large frame fails in turn; the call reports it
//           (or succeeds without), and a small frame after it gets all its
//           buffers: a launch with a null or freed one would fault a device.
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

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "growth") growth();
    else return 2;
    if (g_failures) return 1;
    std::printf("memory ok\n");
    return 0;
}

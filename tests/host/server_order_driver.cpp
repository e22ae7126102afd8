// Ordering of the render server's device work, checked on the host.  The HIP
// runtime and the kernel launchers are stand-ins: nothing runs, every stream,
// event and buffer carries vector clocks, and two accesses of one buffer, at
// least one a write, that no stream order, event or host wait orders are
// reported as a race.  An event looks complete to the host as soon as it is
// recorded, the earliest that a device could report it.
//
// The scenario: slots 0 and 1 hold finished images, slot 2's request can never
// fit the budget and is refused.  The images are released, a request occupies
// slot 0, and two more that start together share one preprocess on slot 1's
// stream, which writes slot 2's buffers: its refused request's depth order
// must be behind it.
#include <hip/hip_runtime.h>

#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "fgs.h"
#include "fgs_internal.hpp"

namespace {

constexpr int kRefusedWidth = 96;  // the request of this width has too many pairs
constexpr int kGateWidth = 80;     // the launch of this one waits for the gate

using Clock = std::map<int, long>;  // execution lane -> steps
void merge(Clock &a, const Clock &b) {
    for (auto &kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}

struct FakeStream {
    int id;
    Clock now;
};
struct FakeEvent {
    Clock at;
};
struct Access {
    int lane;
    long step;
    std::string what;
    bool write;
};

std::recursive_mutex g_mu;
int g_next_id = 1;
Clock g_host;
std::vector<FakeStream *> g_streams;
FakeStream g_null{0, {}};
std::map<const void *, std::vector<Access>> g_accesses;
std::map<const void *, int> g_width;  // counters -> width of the frame they count
int g_races = 0, g_refused_orders = 0;

std::mutex g_gate_mu;
std::condition_variable g_gate_cv;
bool g_gate_open = false, g_gate_reached = false;

FakeStream *stream_of(hipStream_t s) { return s ? reinterpret_cast<FakeStream *>(s) : &g_null; }

// one kernel on a stream: everything the host has seen is before it
void work(hipStream_t sv, const char *what, std::vector<const void *> reads, std::vector<const void *> writes) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    FakeStream *s = stream_of(sv);
    merge(s->now, g_host);
    const long step = ++s->now[s->id];
    auto touch = [&](const void *p, bool write) {
        if (!p) return;
        std::vector<Access> &v = g_accesses[p];
        for (const Access &a : v)
            if ((a.write || write) && s->now[a.lane] < a.step) {
                std::fprintf(stderr, "race: %s on stream %d is not ordered after %s on stream %d\n", what, s->id,
                             a.what.c_str(), a.lane);
                ++g_races;
            }
        v.push_back(Access{s->id, step, what, write});
    };
    for (const void *p : reads) touch(p, false);
    for (const void *p : writes) touch(p, true);
}

void counters(const void *fc, int W) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    g_width[fc] = W;
    if (W == kRefusedWidth) ++g_refused_orders;
}

void wait_at_gate(int W) {
    if (W != kGateWidth) return;
    std::unique_lock<std::mutex> lk(g_gate_mu);
    g_gate_reached = true;
    g_gate_cv.notify_all();
    g_gate_cv.wait(lk, [] { return g_gate_open; });
}

[[noreturn]] void unexpected(const char *what) {
    std::fprintf(stderr, "%s is not expected here\n", what);
    std::abort();
}

}  // namespace

// ---- the HIP runtime --------------------------------------------------------------
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    // (device memory that nothing here reads or writes)
    *p = std::malloc(n < 256 ? 256 : 256);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *f = *t = (size_t)1 << 40;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *, int) { unexpected("hipGetDeviceProperties"); }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    FakeStream *f = new FakeStream{g_next_id++, {}};
    g_streams.push_back(f);
    *s = reinterpret_cast<hipStream_t>(f);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    merge(g_host, stream_of(s)->now);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    for (FakeStream *f : g_streams) merge(g_host, f->now);
    merge(g_host, g_null.now);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned int) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    merge(stream_of(s)->now, reinterpret_cast<FakeEvent *>(e)->at);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new FakeEvent{});
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    delete reinterpret_cast<FakeEvent *>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    reinterpret_cast<FakeEvent *>(e)->at = stream_of(s)->now;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    merge(g_host, reinterpret_cast<FakeEvent *>(e)->at);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return hipEventQuery(e); }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { unexpected("hipEventElapsedTime"); }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { unexpected("hipMemcpy"); }
hipError_t hipMemset(void *, int, size_t) { unexpected("hipMemset"); }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { unexpected("hipMemsetAsync"); }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t, hipMemcpyKind kind, hipStream_t s) {
    if (kind != hipMemcpyDeviceToHost) unexpected("a copy that is not the counters'");
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    work(s, "the counters' copy", {src}, {});
    fgs::FrameCounters h{};
    h.visible = 10;
    h.pairs = g_width[src] == kRefusedWidth ? 100u << 20 : 64u;
    h.entries = 32;
    std::memcpy(dst, &h, sizeof h);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { unexpected("capture"); }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { unexpected("capture"); }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { unexpected("graph"); }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { unexpected("graph"); }
hipError_t hipGraphDestroy(hipGraph_t) { unexpected("graph"); }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { unexpected("graph"); }
}

// ---- the kernel launchers ---------------------------------------------------------
namespace fgs {

void launch_fill_u32(uint32_t *p, uint32_t, size_t, hipStream_t s) { work(s, "fill", {}, {p}); }
hipError_t noalloc_scratch(int, unsigned char **) { unexpected("noalloc_scratch"); }
void launch_peak_fma(int, int, float *, hipStream_t) { unexpected("peak_fma"); }
void launch_peak_exp(int, int, float *, hipStream_t) { unexpected("peak_exp"); }
void launch_peak_copy(const void *, void *, size_t, hipStream_t) { unexpected("peak_copy"); }
unsigned preprocess_grid(int64_t) { return 1; }
unsigned emit_grid(uint32_t) { return 1; }
void launch_preprocess(const DevScene &, const DevPrepared *, const DevCamera &, const DevCam64 &, const DevOptions &,
                       int W, int, GaussState *gs, float4 *conic, uint4 *, uint32_t *count, uint8_t *count8,
                       uint4 *erec, uint32_t *dkey, uint32_t *cand, uint32_t *seg_count, uint32_t *gmap, uint2 *chunks,
                       uint32_t, FrameCounters *fc, uint32_t *gsum_clear, bool, hipStream_t s) {
    wait_at_gate(W);
    counters(fc, W);
    work(s, "preprocess", {cand, seg_count},
         {gs, conic, count, count8, erec, dkey, gmap, chunks, fc, &fc->nlong, gsum_clear});
}
void launch_cull(const DevScene &, const DevPrepared &, const DevCamera &, const DevOptions &, int, int,
                 uint32_t *cand, uint32_t *seg_count, FrameCounters *fc, hipStream_t s) {
    work(s, "cull", {}, {cand, seg_count, fc, &fc->nlong});
}
void launch_preprocess_multi(const DevScene &, const DevPrepared &, const MultiOut &mo, const DevOptions &,
                             uint32_t *cand, uint32_t *seg_count, uint32_t *gmap, hipStream_t s) {
    work(s, "shared cull", {}, {cand, seg_count});
    std::vector<const void *> w = {gmap};
    for (int c = 0; c < mo.n; ++c) {
        const CamOut &o = mo.c[c];
        counters(o.fc, o.W);
        for (const void *p : {(const void *)o.gs, (const void *)o.conic, (const void *)o.count, (const void *)o.count8,
                              (const void *)o.erec, (const void *)o.dkey, (const void *)o.gmap, (const void *)o.chunks,
                              (const void *)o.fc, (const void *)&o.fc->nlong, (const void *)o.gsum_clear})
            w.push_back(p);
    }
    work(s, "shared preprocess", {cand, seg_count}, w);
}
void launch_prepare(const DevScene &, const DevOptions &, const uint32_t *, float4 *, float4 *, float *, float2 *,
                    uint32_t *, int, hipStream_t) {}
void launch_spatial_keys(const DevScene &, uint32_t *, uint32_t *, hipStream_t) {}
void launch_block_bounds(const float4 *, const float2 *, int64_t, float4 *, hipStream_t) {}
void launch_depth_ties(const uint32_t *keys, uint32_t *vals, const uint32_t *gmap, uint32_t, const uint32_t *,
                       uint32_t *long_list, FrameCounters *fc, uint32_t *tmp_v, hipStream_t s) {
    // (its own counter: the host never reads that word of the counters' copy)
    work(s, "depth ties", {keys, gmap}, {vals, long_list, &fc->nlong, tmp_v});
}
void launch_big_count(int, int, int, const GaussState *gs, const float4 *conic, const uint4 *erec, const uint2 *chunks,
                      uint32_t, uint32_t *chunk_mask, uint32_t *count, FrameCounters *, hipStream_t s) {
    // (its counters' words are its own)
    work(s, "large rectangles' tests", {gs, conic, erec, chunks}, {chunk_mask, count});
}
void launch_super_emit(int, int, const uint32_t *order, uint32_t, const uint32_t *, const uint32_t *offsets,
                       const uint4 *erec, uint32_t, const uint2 *, uint2 *big, const uint32_t *chunk_mask, uint32_t,
                       const FrameCounters *, uint16_t *skey, uint32_t *, uint64_t *, uint32_t, uint2 *sranges,
                       uint32_t, uint32_t *gsum_clear, hipStream_t s) {
    work(s, "emission", {order, offsets, erec, chunk_mask}, {big, skey, sranges, gsum_clear});
}
void launch_tile_lists(int, int, const uint2 *sranges, const uint32_t *, const uint64_t *, uint32_t, uint32_t *,
                       uint2 *ranges, uint32_t *values, uint32_t, hipStream_t s) {
    work(s, "tile lists", {sranges}, {ranges, values});
}
void launch_radix_pass(const void *keys_in, const uint32_t *vals_in, void *keys_out, uint32_t *vals_out, uint32_t,
                       const uint32_t *n_dev, int, int bits, bool, bool write_keys, uint32_t *hist, uint32_t *,
                       uint32_t *, hipStream_t s, uint2 *, uint32_t, int, const uint64_t *, uint64_t *, bool) {
    (void)n_dev;  // (read-only words of the counters that the counters' copy may read too)
    const bool in_place = bits == 32 && keys_in == keys_out;
    work(s, "radix pass", {in_place ? nullptr : keys_in, vals_in}, {write_keys ? keys_out : nullptr, vals_out, hist});
}
void launch_count_scan(const uint32_t *order, const uint8_t *count8, const uint4 *erec, uint32_t, const uint32_t *,
                       uint32_t *cs, uint32_t *sums, uint32_t *offsets, uint32_t *, hipStream_t s) {
    work(s, "entry scan", {order, count8, erec}, {cs, sums, offsets});
}
void launch_single_range(uint2 *ranges, uint32_t, const uint32_t *, hipStream_t s) {
    work(s, "single range", {}, {ranges});
}
void launch_blend(const GaussState *gs, const uint32_t *values, const uint2 *ranges, int, int, const DevOptions &,
                  float *rgb, float *, uint32_t *, unsigned long long *, int, uint32_t, uint32_t, hipStream_t s) {
    work(s, "blend", {gs, values, ranges}, {rgb});
}
void launch_blend_backward(const GaussState *, const uint32_t *, const uint2 *, const float *, const uint32_t *,
                           const float *, int, int, const DevOptions &, float *, int64_t, hipStream_t) {
    unexpected("blend_backward");
}
void launch_preprocess_backward(const DevScene &, const DevCamera &, const DevOptions &, int, int, const GaussState *,
                                const float *, int64_t, float *, float *, float *, float *, float *, int64_t,
                                hipStream_t) {
    unexpected("preprocess_backward");
}

}  // namespace fgs

// ---- the scenario -------------------------------------------------------------------
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
    if (g_failures) return 1;
    std::printf("order ok\n");
    return 0;
}

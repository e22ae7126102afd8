// Stand-ins for the HIP runtime and the kernel launchers, for host tests of the
// runtime's own logic (linked with runtime.cpp, pipeline.cpp and server.cpp, no
// kernel file and no HIP library).  Nothing runs; what is checked:
//   order   every stream, event and buffer carries vector clocks, and two
//           accesses of one buffer, at least one a write, that no stream order,
//           event or host wait orders are reported as a race.  An event looks
//           complete to the host as soon as it is recorded, the earliest that a
//           device could report it.
//   memory  allocations are counted against g_limit; a launch that is given a
//           null pointer, or a buffer that has been freed, is reported.
// The signatures are those of fgs_internal.hpp, so any drift fails to link.
#pragma once

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

constexpr int kRefusedWidth = 96;  // a frame of this width has too many pairs for a small budget
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
int g_fail_in = -1;  // the allocation after that many fails (-1: none)
int g_races = 0, g_bad_pointers = 0, g_refused_orders = 0;
size_t g_limit = (size_t)1 << 40, g_used = 0;  // device memory
std::map<const void *, size_t> g_alloc;
bool g_kept = false;  // the frames are kept: their blend has a last contributor to write
uint32_t g_pairs = 64, g_entries = 32;  // counters of a frame

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
        auto a = g_alloc.upper_bound(p);  // (a part of an allocation)
        if (!p || a == g_alloc.begin() || (const char *)p >= (const char *)(--a)->first + a->second) {
            std::fprintf(stderr, "%s: %s\n", what, p ? "not an allocation" : "null");
            ++g_bad_pointers;
            return;
        }
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
// (addresses only: no one reads or writes device memory here)
hipError_t hipMalloc(void **p, size_t n) {
    static uintptr_t next = (uintptr_t)1 << 44;
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    *p = nullptr;
    if (n > g_limit - g_used || g_fail_in == 0) {
        if (g_fail_in == 0) g_fail_in = -1;
        return hipErrorOutOfMemory;
    }
    if (g_fail_in > 0) --g_fail_in;
    *p = reinterpret_cast<void *>(next);
    next += (n + 4096) / 4096 * 4096;
    g_alloc[*p] = n;
    g_used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    if (!p) return hipSuccess;
    auto it = g_alloc.find(p);
    if (it == g_alloc.end()) unexpected("a second free");
    (void)hipDeviceSynchronize();
    g_used -= it->second;
    g_alloc.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    *f = g_limit - g_used;
    *t = g_limit;
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
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
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
    h.pairs = g_width[src] == kRefusedWidth ? 100u << 20 : g_pairs;
    h.entries = g_entries;
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
hipError_t noalloc_scratch(int, unsigned char **base) {
    static unsigned char scratch[256];
    *base = scratch;
    return hipSuccess;
}
void launch_peak_fma(int, int, float *, hipStream_t) { unexpected("peak_fma"); }
void launch_peak_exp(int, int, float *, hipStream_t) { unexpected("peak_exp"); }
void launch_peak_copy(const void *, void *, size_t, hipStream_t) { unexpected("peak_copy"); }
unsigned preprocess_grid(int64_t) { return 1; }
unsigned emit_grid(uint32_t) { return 1; }
void launch_preprocess(const DevScene &, const DevPrepared *pp, const DevCamera &, const DevCam64 &, const DevOptions &,
                       int W, int, GaussState *gs, float4 *conic, uint4 *, uint32_t *count, uint8_t *count8,
                       uint4 *erec, uint32_t *dkey, uint32_t *cand, uint32_t *seg_count, uint32_t *gmap, uint2 *chunks,
                       uint32_t, FrameCounters *fc, uint32_t *gsum_clear, bool, hipStream_t s) {
    wait_at_gate(W);
    counters(fc, W);
    if (pp) work(s, "preprocess", {pp->pos_o, pp->cov, pp->sh, pp->orig}, {});
    work(s, "preprocess", {cand, seg_count},
         {gs, conic, count, count8, erec, dkey, gmap, chunks, fc, &fc->nlong, gsum_clear});
}
void launch_cull(const DevScene &, const DevPrepared &pp, const DevCamera &, const DevOptions &, int, int,
                 uint32_t *cand, uint32_t *seg_count, FrameCounters *fc, hipStream_t s) {
    work(s, "cull", {pp.pos_o, pp.bnd, pp.blk}, {cand, seg_count, fc, &fc->nlong});
}
void launch_preprocess_multi(const DevScene &, const DevPrepared &pp, const MultiOut &mo, const DevOptions &,
                             uint32_t *cand, uint32_t *seg_count, uint32_t *gmap, hipStream_t s) {
    work(s, "shared cull", {pp.pos_o, pp.bnd, pp.blk}, {cand, seg_count});
    std::vector<const void *> w = {gmap};
    for (int c = 0; c < mo.n; ++c) {
        const CamOut &o = mo.c[c];
        counters(o.fc, o.W);
        for (const void *p : {(const void *)o.gs, (const void *)o.conic, (const void *)o.count, (const void *)o.count8,
                              (const void *)o.erec, (const void *)o.dkey, (const void *)o.gmap, (const void *)o.chunks,
                              (const void *)o.fc, (const void *)&o.fc->nlong, (const void *)o.gsum_clear})
            w.push_back(p);
    }
    work(s, "shared preprocess", {cand, seg_count, pp.pos_o, pp.cov, pp.sh, pp.orig}, w);
}
void launch_prepare(const DevScene &, const DevOptions &, const uint32_t *perm, float4 *pos_o, float4 *cov, float *sh,
                    float2 *bnd, uint32_t *orig, int, hipStream_t s) {
    work(s, "prepare", {perm}, {pos_o, cov, sh, bnd, orig});
}
void launch_spatial_keys(const DevScene &, uint32_t *bounds, uint32_t *keys, hipStream_t s) {
    work(s, "spatial keys", {}, {bounds, keys});
}
void launch_block_bounds(const float4 *pos_o, const float2 *bnd, int64_t, float4 *blk, hipStream_t s) {
    work(s, "block bounds", {pos_o, bnd}, {blk});
}
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
                       const uint4 *erec, uint32_t, const uint2 *chunks, uint2 *big, const uint32_t *chunk_mask,
                       uint32_t, const FrameCounters *, uint16_t *skey, uint32_t *gidx, uint64_t *smask, uint32_t,
                       uint2 *sranges, uint32_t, uint32_t *gsum_clear, hipStream_t s) {
    if (order) {
        work(s, "emission", {order, offsets, erec}, {big, skey, gidx, smask});
        if (sranges) work(s, "emission", {}, {sranges});
        if (gsum_clear) work(s, "emission", {}, {gsum_clear});
    }
    if (chunk_mask) work(s, "large rectangles' entries", {big, erec, chunks, chunk_mask}, {skey, gidx, smask});
}
void launch_tile_lists(int, int, const uint2 *sranges, const uint32_t *, const uint64_t *, uint32_t, uint32_t *,
                       uint2 *ranges, uint32_t *values, uint32_t, hipStream_t s) {
    work(s, "tile lists", {sranges}, {ranges, values});
}
void launch_radix_pass(const void *keys_in, const uint32_t *vals_in, void *keys_out, uint32_t *vals_out, uint32_t,
                       const uint32_t *, int, int bits, bool, bool write_keys, uint32_t *hist, uint32_t *,
                       uint32_t *, hipStream_t s, uint2 *, uint32_t, int, const uint64_t *, uint64_t *, bool) {
    // (the counters that n_dev reads are words that the counters' copy reads too)
    std::vector<const void *> r = {keys_in}, w = {vals_out};
    if (vals_in) r.push_back(vals_in);
    if (write_keys && keys_out != keys_in) w.push_back(keys_out);
    if (bits != 32) w.push_back(hist);
    if (write_keys && keys_out == keys_in) {
        r.clear();
        w.push_back(keys_out);
    }
    work(s, "radix pass", r, w);
}
void launch_count_scan(const uint32_t *order, const uint8_t *count8, const uint4 *erec, uint32_t, const uint32_t *,
                       uint32_t *cs, uint32_t *sums, uint32_t *offsets, uint32_t *, hipStream_t s) {
    work(s, "entry scan", {order, count8, erec}, {cs, sums, offsets});
}
void launch_single_range(uint2 *ranges, uint32_t, const uint32_t *, hipStream_t s) {
    work(s, "single range", {}, {ranges});
}
void launch_blend(const GaussState *gs, const uint32_t *values, const uint2 *ranges, int, int, const DevOptions &,
                  float *, float *, uint32_t *last, unsigned long long *, int, uint32_t, uint32_t, hipStream_t s) {
    // (the outputs may be the caller's own memory)
    work(s, "blend", {gs, values, ranges}, {});
    if (g_kept && !last) work(s, "blend", {}, {last});
}
void launch_blend_backward(const GaussState *gs, const uint32_t *values, const uint2 *ranges, const float *Tfin,
                           const uint32_t *last, const float *, int, int, const DevOptions &, float *acc, int64_t,
                           hipStream_t s) {
    work(s, "blend adjoint", {gs, values, ranges, Tfin, last}, {acc});
}
void launch_preprocess_backward(const DevScene &, const DevCamera &, const DevOptions &, int, int, const GaussState *gs,
                                const float *acc, int64_t, float *, float *, float *, float *, float *, int64_t,
                                hipStream_t s) {
    work(s, "preprocess adjoint", {gs, acc}, {});
}

}  // namespace fgs

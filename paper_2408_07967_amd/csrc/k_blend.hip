// Per-tile front-to-back alpha blending with early termination (Sec. 2.2
// rendering stage; Sec. 5.2 early stop on saturated transmittance, opacity
// checks moved out of the per-pixel loop; Sec. 5.3.2 exponent in log form).
//
// One workgroup per 16 x 16 tile, in two forms (launch_blend picks one by the
// number of tiles): two wavefronts, each owning a 16 x 8 half with two
// horizontally adjacent pixels per lane, so that the row terms of the
// quadratic form, the LDS reads and the loop control are shared by two
// pixels; or four, each owning an 8 x 8 quadrant with one pixel per lane,
// which walk shorter lists and fill the device when the tiles are few.  The
// tile's sorted list is walked in batches of one Gaussian per thread (eight
// wavefronts per SIMD fit):
// every thread stages one Gaussian (the coefficients of the exponent,
// opacity threshold and colour) in LDS and tests each ellipse against the
// regions (the exact tile test with a slightly inflated extent; what it can
// drop stands at test_extent); a wavefront walks only the entries that meet its
// region, two at a time: their evaluations overlap, and the saturation check
// of both is one (T only falls; when a pixel saturates within the pair, the
// pair is resolved entry by entry).  Bound by FP32 issue when the tiles are
// many (4K city 10M: 24 slots per step and two pixels) and by the serial chain
// of a wavefront when they are few.  One entry at a time in halves took 346 us
// at 4K and 97 / 106 / 149 us at 256 / 3600 / 8160 tiles; now 324 and 46 / 71 /
// 115 us.  (The colour accumulated by v_mfma_f32_4x4x1_f32, which leaves 18
// slots, was slower: 380 us at 4K.)
// Per pixel and Gaussian:
//   E = log2 o - q log2(e) / 2; contributes iff E >= log2 o - k^2 log2(e) / 2;
//   alpha = min(alpha_max, 2^E);
//   T' = T (1 - alpha); if T' < T_stop the pixel stops before blending it;
//   C += colour alpha T; T = T'.
// A stopped pixel moves its sample point to +1e30 so that E becomes -inf and
// the Gaussian never contributes again: the hot loop carries no done-flag.
#include "fgs_internal.hpp"
#include "blend_common.hpp"

namespace fgs {
namespace {

constexpr int kWave = 64;
constexpr int kThreads = 128;        // two wavefronts per tile (the prefetch variant)
constexpr float kFar = 1e30f;

struct Pixel {
    float x;        // sample x, or kFar once stopped
    float T, c0, c1, c2;
    uint32_t last;
    uint32_t examined;
    bool done;
};

// Alpha of one pixel for one Gaussian, and whether it contributes.
struct Alpha {
    float a;
    bool in;
};

__device__ __forceinline__ Alpha alpha_at(float e, float thr, float amax) {
    Alpha r;
    r.in = e >= thr;
    // min(2^E, amax), 0 outside the extent: the clamp's upper end is selected
    // beside the exponential (2^E >= 0), one v_med3_f32 with no per-iteration
    // canonicalisation of amax that a minimum would bring
    r.a = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(e), 0.0f, r.in ? amax : 0.0f);
    return r;
}

// kPx: horizontally adjacent pixels per lane (2: two wavefronts per tile, a
// 16 x 8 half each; 1: four, an 8 x 8 quadrant each).
template <int kPx, bool kCountWork, bool kLast>
__global__ __launch_bounds__(256 / kPx) __attribute__((amdgpu_waves_per_eu(8))) void k_blend(const GaussState *__restrict__ gs,
                                                     const uint32_t *__restrict__ values,
                                                     const uint2 *__restrict__ ranges, int W, int H, int tiles_x,
                                                     DevOptions op, float *__restrict__ rgb, float *__restrict__ Tout,
                                                     uint32_t *__restrict__ last_out, unsigned long long *work) {
    constexpr int kThreads = 256 / kPx, kBatch = kThreads;  // each thread stages one Gaussian of a batch
    constexpr int kRegions = kThreads / kWave, kWords = kBatch / kWave;
    // one float4 stride for all three arrays: a single LDS address per
    // Gaussian.  Entry kBatch contributes nowhere (its threshold is +inf).
    __shared__ float4 s_f0[kBatch + 1], s_f1[kBatch + 1], s_f2[kBatch + 1];
    // kPx == 1: bit h of s_hit: the entry meets region h; s_list: the entries
    // that meet region h, in list order, as byte offsets into s_f0 (padded to
    // whole pairs with entry kBatch).  kPx == 2: s_rel[h][w]: bit i set iff
    // entry 64 w + i meets region h; its set bits are walked in scalar code.
    constexpr bool kList = kPx == 1;
    static_assert(!kList || !kCountWork, "work is counted on the halves");
    __shared__ uint8_t s_hit[kList ? kBatch : 1];
    __shared__ alignas(4) uint16_t s_list[kList ? kRegions : 1][kList ? kBatch + 2 : 2];
    __shared__ uint32_t s_rel[kList ? 1 : kRegions][kWords][2];
    static_assert((kBatch + 1) * sizeof(float4) <= 65536, "16-bit offsets");

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform
    const int tile = blockIdx.x;
    const int tx = tile % tiles_x, ty = tile / tiles_x;
    const int rx = kPx == 2 ? 0 : wave & 1, ry = kPx == 2 ? wave : wave >> 1;
    const int pi0 = tx * kTile + rx * 8 + kPx * (lane & 7);
    const int pj = ty * kTile + ry * 8 + (lane >> 3);
    const float py = (float)pj + 0.5f;

    const uint2 rg = ranges[tile];
    const uint32_t start = rg.x, end = rg.y > rg.x ? rg.y : rg.x;  // an empty tile may hold start > end
    Pixel p[kPx];
    auto all_done = [&]() {
        bool d = p[0].done;
        if constexpr (kPx == 2) d = d && p[1].done;
        return d;
    };
#pragma unroll
    for (int i = 0; i < kPx; ++i) {
        const bool in = pi0 + i < W && pj < H;
        p[i] = Pixel{in ? (float)(pi0 + i) + 0.5f : kFar, 1.0f, 0.0f, 0.0f, 0.0f, 0u, in ? end - start : 0u, !in};
    }
    bool wave_done = __ballot(!all_done()) == 0;
    // loop-invariant clamp as the result of an arithmetic op (a canonical
    // value, so the minimum needs no per-iteration canonicalisation)
    const float amax = op.alpha_max + 0.0f;
    const float tstop = op.T_stop;
    uint32_t wsteps = 0;  // kCountWork: entries this wavefront evaluates (uniform)
    if (tid == 0) {
        s_f0[kBatch] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        s_f1[kBatch] = make_float4(0.0f, INFINITY, 0.0f, 0.0f);
        s_f2[kBatch] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    // kPx == 1 (few tiles, so little else hides it): the next batch's state is
    // loaded while this one is blended
    constexpr bool kAhead = kPx == 1;
    GaussState ahead;
    if (kAhead && start + tid < end) ahead = gs[values[start + tid]];

    for (uint32_t b0 = start; b0 < end; b0 += kBatch) {
        const uint32_t nb = (end - b0) < (uint32_t)kBatch ? (end - b0) : (uint32_t)kBatch;
        {
            uint32_t hm = 0;
            if ((uint32_t)tid < nb) {
                const GaussState s = kAhead ? ahead : gs[values[b0 + tid]];
                // (a quadrant counts only where its half is met, so that both
                // forms blend the same entries)
                const float k2i = test_extent(s), k2t = kPx == 1 ? test_extent_thin(s) : 0.0f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int X0 = tx * kTile, Y0 = ty * kTile + 8 * h;
                    const bool half = region_hit(s, k2i, X0, kTile, Y0, W, H);
                    if constexpr (kPx == 2) {
                        hm |= (uint32_t)half << h;
                    } else {
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            hm |= (uint32_t)(half & region_hit(s, k2t, X0 + 8 * q, 8, Y0, W, H)) << (2 * h + q);
                    }
                }
                float4 f0, f1;
                float2 f2;
                stage_gauss(s, f0, f1, f2);
                s_f0[tid] = f0;
                s_f1[tid] = f1;
                s_f2[tid] = make_float4(f2.x, f2.y, 0.0f, 0.0f);
            }
            if constexpr (kList) {
                s_hit[tid] = (uint8_t)hm;
            } else {
#pragma unroll
                for (int h = 0; h < kRegions; ++h) {
                    const uint64_t bq = __ballot((hm >> h) & 1u);
                    if (lane == 0) {
                        s_rel[h][wave][0] = (uint32_t)bq;
                        s_rel[h][wave][1] = (uint32_t)(bq >> 32);
                    }
                }
            }
        }
        __syncthreads();
        if (kAhead && b0 + kBatch + tid < end) ahead = gs[values[b0 + kBatch + tid]];
        if (!wave_done) {
            const uint32_t pos1 = b0 - start + 1u;
            // two staged Gaussians (byte offsets into s_f0) for the lane's
            // pixels: their chains overlap, and one termination check covers
            // both; true once every pixel of the wavefront has stopped
            auto blend_two = [&](uint32_t offa, uint32_t offb) {
                const uint32_t off[2] = {offa, offb};
                float4 f0[2], f1[2];
                float2 f2[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    f0[k] = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_f0) + off[k]);
                    f1[k] = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_f1) + off[k]);
                    f2[k] = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(s_f2) + off[k]);
                }
                Alpha a[2][kPx];
                float T[3][kPx];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const RowTerms rt = row_terms(f0[k], f1[k], py);
#pragma unroll
                    for (int i = 0; i < kPx; ++i) a[k][i] = alpha_at(exponent_at(f0[k], rt, p[i].x), f1[k].y, amax);
                }
                bool low = false;
#pragma unroll
                for (int i = 0; i < kPx; ++i) {
                    T[0][i] = p[i].T;
#pragma unroll
                    for (int k = 0; k < 2; ++k) T[k + 1][i] = fmaf(-a[k][i].a, T[k][i], T[k][i]);
                    low = low || T[2][i] < tstop;
                }
                // (T only falls, so the first of them cannot pass the
                // threshold unseen)
                if (__ballot(low) != 0) {
#pragma unroll
                    for (int i = 0; i < kPx; ++i) {
                        // the pixel saturates: it stops before the first
                        // Gaussian that would pass the threshold (rare path)
                        bool stopped = false;
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            if (!stopped && T[k + 1][i] < tstop) {
                                stopped = true;
                                if (kCountWork) p[i].examined = pos1 + off[k] / (uint32_t)sizeof(float4);
                                p[i].x = kFar;
                                p[i].done = true;
                            }
                            if (stopped) {
                                a[k][i].a = 0.0f;
                                a[k][i].in = false;
                                T[k + 1][i] = T[k][i];
                            }
                        }
                    }
                    wave_done = __ballot(!all_done()) == 0;
                }
#pragma unroll
                for (int i = 0; i < kPx; ++i) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const float w = a[k][i].a * T[k][i];
                        p[i].c0 = fmaf(w, f1[k].w, p[i].c0);
                        p[i].c1 = fmaf(w, f2[k].x, p[i].c1);
                        p[i].c2 = fmaf(w, f2[k].y, p[i].c2);
                        if (kLast) p[i].last = a[k][i].in ? pos1 + off[k] / (uint32_t)sizeof(float4) : p[i].last;
                    }
                    p[i].T = T[2][i];
                }
                return wave_done;
            };
            constexpr uint32_t kNone = kBatch * sizeof(float4);
            if constexpr (kList) {
                uint32_t n = 0;  // uniform
                uint16_t *const list = s_list[wave];
#pragma unroll
                for (int w = 0; w < kWords; ++w) {
                    const uint64_t bal = __ballot(((s_hit[w * kWave + lane] >> wave) & 1u) != 0u);
                    const uint32_t at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                    if ((bal >> lane) & 1u) list[at] = (uint16_t)((w * kWave + lane) * (int)sizeof(float4));
                    n += (uint32_t)__popcll(bal);
                }
                if (lane == 0) list[n] = (uint16_t)kNone;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                for (uint32_t q = 0; q < n; q += 2) {
                    const uint32_t pair = *reinterpret_cast<const uint32_t *>(list + q);
                    if (blend_two(pair & 0xffffu, pair >> 16)) break;
                }
            } else {
                for (int w = 0; w < kWords && !wave_done; ++w) {
                    uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)s_rel[wave][w][0]) |
                                 ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)s_rel[wave][w][1]) << 32);
                    while (m) {
                        const uint32_t ja = (uint32_t)(w * kWave + __builtin_ctzll(m));
                        m &= m - 1;
                        const uint32_t jb = m ? (uint32_t)(w * kWave + __builtin_ctzll(m)) : (uint32_t)kBatch;
                        m &= m - 1;  // (0 stays 0)
                        if (kCountWork) wsteps += jb < (uint32_t)kBatch ? 2u : 1u;
                        if (blend_two(ja * (uint32_t)sizeof(float4), jb * (uint32_t)sizeof(float4))) break;
                    }
                }
            }
        }
        // all 256 pixels finished: stop walking the list (also the barrier
        // that protects the staging buffers)
        if (__syncthreads_count(all_done() ? 1 : 0) == kThreads) break;
    }

    if (kCountWork) {
        // a wave that skipped a Gaussian whose ellipse misses its region still
        // counts it: the count is the method's, not this kernel's
        unsigned long long v = 0;
#pragma unroll
        for (int i = 0; i < kPx; ++i) v += p[i].examined;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) v += __shfl_xor(v, d, kWave);
        if (lane == 0) {
            atomicAdd(work, v);
            atomicAdd(work + 1, (unsigned long long)wsteps);
        }
    }
    const size_t hw = (size_t)W * H;
    const size_t q = (size_t)pj * W + pi0;
#pragma unroll
    for (int i = 0; i < kPx; ++i)
        if (pi0 + i < W && pj < H) {
            rgb[q + i] = p[i].c0 + p[i].T * op.bg[0];
            rgb[hw + q + i] = p[i].c1 + p[i].T * op.bg[1];
            rgb[2 * hw + q + i] = p[i].c2 + p[i].T * op.bg[2];
            if (Tout) Tout[q + i] = p[i].T;
            if (kLast && last_out) last_out[q + i] = p[i].last;
        }
}

// ---- the variant's pixel: colour in plain registers ------------------------
struct PixelV {
    float x;        // sample x, or kFar once stopped
    float T, c0, c1, c2;
    uint32_t last;
    uint32_t examined;
    bool done;
};

// Alpha and transmittance of one pixel for one Gaussian, before the
// termination check.
struct Step {
    float a, Tn;
    bool in, stop;
};

__device__ __forceinline__ Step step(const PixelV &p, float e, float thr, float amax, float tstop) {
    Step st;
    st.in = e >= thr;
    // min(2^E, amax) as a clamp to [0, amax] (2^E >= 0): one v_med3_f32, with
    // no per-iteration canonicalisation of amax that a minimum would bring
    st.a = st.in ? __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(e), 0.0f, amax) : 0.0f;
    st.Tn = fmaf(-st.a, p.T, p.T);
    st.stop = st.Tn < tstop;
    return st;
}

// The pixel saturates: it stops before this Gaussian (rare path).
template <bool kCountWork>
__device__ __forceinline__ void stop_before(PixelV &p, Step &st, uint32_t pos) {
    st.a = 0.0f;
    st.Tn = p.T;
    st.in = false;
    p.x = kFar;
    p.done = true;
    if (kCountWork) p.examined = pos + 1u;
}

template <bool kLast>
__device__ __forceinline__ void apply(PixelV &p, const Step &st, const float4 &f1, const float2 &f2, uint32_t pos) {
    const float w = st.a * p.T;
    p.c0 = fmaf(w, f1.w, p.c0);
    p.c1 = fmaf(w, f2.x, p.c1);
    p.c2 = fmaf(w, f2.y, p.c2);
    p.T = st.Tn;
    if (kLast) p.last = st.in ? pos + 1u : p.last;
}

// Variant of the blend (selected per context): each wavefront walks its
// tile's whole list on its own with a software prefetch pipeline, the form
// of the paper's render loop (Sec. 5.3.2): while entry i is blended, the
// state of entry i + 1 and the index of entry i + 2 are in flight (vector
// buffer loads, which complete in order, so the wait for entry i's state
// leaves the later loads outstanding).  Nothing is staged in LDS and no half
// mask is kept: every entry is evaluated for the wavefront's 128 pixels; an
// entry whose ellipse misses a pixel gives it alpha 0, which leaves colour,
// transmittance and last contributor exactly as they were, so the image is
// bit for bit the one of k_blend.
template <bool kLast>
__global__ __launch_bounds__(kThreads) void k_blend_prefetch(const GaussState *__restrict__ gs,
                                                             const uint32_t *__restrict__ values,
                                                             const uint2 *__restrict__ ranges, int W, int H,
                                                             int tiles_x, uint32_t nvalues, uint32_t ngs,
                                                             DevOptions op, float *__restrict__ rgb,
                                                             float *__restrict__ Tout, uint32_t *__restrict__ last_out) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform
    const int tile = blockIdx.x;
    const int tx = tile % tiles_x, ty = tile / tiles_x;
    const int pi0 = tx * kTile + 2 * (lane & 7);
    const int pj = ty * kTile + wave * 8 + (lane >> 3);
    const bool in0 = pi0 < W && pj < H, in1 = pi0 + 1 < W && pj < H;
    const float py = (float)pj + 0.5f;

    const uint2 rg = ranges[tile];
    const uint32_t start = rg.x, end = rg.y > rg.x ? rg.y : rg.x;  // an empty tile may hold start > end
    PixelV p0{in0 ? (float)pi0 + 0.5f : kFar, 1.0f, 0.0f, 0.0f, 0.0f, 0u, 0u, !in0};
    PixelV p1{in1 ? (float)pi0 + 1.5f : kFar, 1.0f, 0.0f, 0.0f, 0.0f, 0u, 0u, !in1};
    bool wave_done = __ballot(!(p0.done && p1.done)) == 0;
    const float amax = op.alpha_max + 0.0f;
    const float tstop = op.T_stop;

    if (!wave_done && start < end) {
        // bounds-checked buffer loads with a wave-uniform offset
        const __amdgpu_buffer_rsrc_t vrs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(values), (short)0, (int)(nvalues * 4u), 0x00020000);
        const __amdgpu_buffer_rsrc_t grs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<GaussState *>(gs), (short)0, (int)(ngs * (uint32_t)sizeof(GaussState)), 0x00020000);
        auto index = [&](uint32_t i) -> uint32_t {  // entry i's Gaussian (past the list: entry start's)
            return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(vrs, (i < end ? i : start) * 4u, 0, 0);
        };
        auto state = [&](uint32_t g) -> GaussState {
            GaussState st;
            const uint32_t o = g * (uint32_t)sizeof(GaussState);
            const auto v0 = __builtin_amdgcn_raw_buffer_load_b128(grs, o, 0, 0);
            const auto v1 = __builtin_amdgcn_raw_buffer_load_b128(grs, o + 16u, 0, 0);
            const auto v2 = __builtin_amdgcn_raw_buffer_load_b128(grs, o + 32u, 0, 0);
            st.f0 = make_float4(__uint_as_float(v0[0]), __uint_as_float(v0[1]), __uint_as_float(v0[2]),
                                __uint_as_float(v0[3]));
            st.f1 = make_float4(__uint_as_float(v1[0]), __uint_as_float(v1[1]), __uint_as_float(v1[2]),
                                __uint_as_float(v1[3]));
            st.f2 = make_float4(__uint_as_float(v2[0]), __uint_as_float(v2[1]), __uint_as_float(v2[2]),
                                __uint_as_float(v2[3]));
            return st;
        };
        // one entry for both pixels of the lane; true once every pixel of the
        // wavefront has stopped
        auto blend_one = [&](const GaussState &gsx, uint32_t pos) {
            float4 f0, f1;
            float2 f2;
            stage_gauss(gsx, f0, f1, f2);
            const RowTerms rt = row_terms(f0, f1, py);
            const float e0 = exponent_at(f0, rt, p0.x);
            const float e1 = exponent_at(f0, rt, p1.x);
            Step s0 = step(p0, e0, f1.y, amax, tstop);
            Step s1 = step(p1, e1, f1.y, amax, tstop);
            if (__ballot(s0.stop || s1.stop) != 0) {
                if (s0.stop) stop_before<false>(p0, s0, pos);
                if (s1.stop) stop_before<false>(p1, s1, pos);
                wave_done = __ballot(!(p0.done && p1.done)) == 0;
            }
            apply<kLast>(p0, s0, f1, f2, pos);
            apply<kLast>(p1, s1, f1, f2, pos);
            return wave_done;
        };
        // two entries per trip, so that the prefetched values alternate
        // between two register sets instead of being copied
        uint32_t i = start;
        uint32_t inext = index(i + 1);
        GaussState sa = state(index(i)), sb;
        for (;;) {
            sb = state(inext);                // entry i + 1
            const uint32_t inn = index(i + 2);
            if (blend_one(sa, i - start) || ++i >= end) break;
            sa = state(inn);                  // entry i + 1
            const uint32_t in3 = index(i + 2);
            if (blend_one(sb, i - start) || ++i >= end) break;
            inext = in3;
        }
    }

    const size_t hw = (size_t)W * H;
    const size_t q = (size_t)pj * W + pi0;
    if (in0) {
        rgb[q] = p0.c0 + p0.T * op.bg[0];
        rgb[hw + q] = p0.c1 + p0.T * op.bg[1];
        rgb[2 * hw + q] = p0.c2 + p0.T * op.bg[2];
        if (Tout) Tout[q] = p0.T;
        if (kLast && last_out) last_out[q] = p0.last;
    }
    if (in1) {
        rgb[q + 1] = p1.c0 + p1.T * op.bg[0];
        rgb[hw + q + 1] = p1.c1 + p1.T * op.bg[1];
        rgb[2 * hw + q + 1] = p1.c2 + p1.T * op.bg[2];
        if (Tout) Tout[q + 1] = p1.T;
        if (kLast && last_out) last_out[q + 1] = p1.last;
    }
}

}  // namespace

void launch_blend(const GaussState *gs, const uint32_t *values, const uint2 *ranges, int W, int H,
                  const DevOptions &op, float *rgb, float *T, uint32_t *last, unsigned long long *work,
                  int variant, uint32_t nvalues, uint32_t ngs, hipStream_t s) {
    const int tiles_x = (W + kTile - 1) / kTile, tiles_y = (H + kTile - 1) / kTile;
    const dim3 grid((unsigned)(tiles_x * tiles_y)), block(kThreads);
    if (variant == 1 && !work && nvalues > 0 && ngs > 0) {
        if (last)
            hipLaunchKernelGGL((k_blend_prefetch<true>), grid, block, 0, s, gs, values, ranges, W, H, tiles_x, nvalues,
                               ngs, op, rgb, T, last);
        else
            hipLaunchKernelGGL((k_blend_prefetch<false>), grid, block, 0, s, gs, values, ranges, W, H, tiles_x,
                               nvalues, ngs, op, rgb, T, last);
        return;
    }
    // One pixel per lane (four wavefronts per tile) while the tiles leave the
    // device short of wavefronts or with a long tail, two per lane (about 15 %
    // fewer instructions per pixel) above.  Blend, us, one / two per lane, 1M
    // Gaussians in a box and 10M city: 920 tiles 96 / 123 and 136 / 244, 3600
    // tiles 101 / 130 and 93 / 144, 8160 tiles 114 / 136 and 138 / 133, 14400
    // tiles 173 / 179 and 202 / 183, 32400 tiles 273 / 235 and 381 / 311.
    constexpr int kOnePixelTiles = 10240;
    const bool one = tiles_x * tiles_y <= kOnePixelTiles;
#define FGS_BLEND(PX, CW, KL)                                                                                     \
    hipLaunchKernelGGL((k_blend<PX, CW, KL>), grid, dim3(256 / PX), 0, s, gs, values, ranges, W, H, tiles_x, op, \
                       rgb, T, last, work)
    if (work) FGS_BLEND(2, true, true);
    else if (one && last) FGS_BLEND(1, false, true);
    else if (one) FGS_BLEND(1, false, false);
    else if (last) FGS_BLEND(2, false, true);
    else FGS_BLEND(2, false, false);
#undef FGS_BLEND
}

}  // namespace fgs

// Per-pixel evaluation shared by the blend and its adjoint.  Both must take
// the same contribution and clamp decisions bit for bit, so the staged
// coefficients and the exponent are written once, with explicit multiply-adds.
#pragma once

#include <hip/hip_runtime.h>

#include "fgs_internal.hpp"

namespace fgs {

constexpr float kHalfLog2e = 0.72134752044448170f;  // log2(e) / 2

// Conservative ellipse / rectangle test used only to skip work: the
// rectangle [X0, X1] x [Y0, Y1] in pixel-sample coordinates (Alg. 3 with the
// chord-overlap condition of Eq. 7).  Callers inflate k2 slightly, against the
// test's roundings.
// (Straight-line, and with its roundings written out: the tests of a tile's
// regions share their lines' terms, and the blend and its adjoint take the same
// decisions.)
__device__ __forceinline__ bool rect_hit(float u, float v, float A, float B, float C, float k2, float X0, float X1,
                                         float Y0, float Y1) {
#pragma clang fp contract(off)
    const float x0 = X0 - u, x1 = X1 - u, y0 = Y0 - v, y1 = Y1 - v;
    bool hit = (x0 <= 0.0f) & (0.0f <= x1) & (y0 <= 0.0f) & (0.0f <= y1);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float y = e ? y1 : y0;
        const float bq = 2.0f * B * y;
        const float cq = fmaf(y, C * y, -k2);
        const float delta = fmaf(bq, bq, -(4.0f * A * cq));
        const float e1 = 2.0f * A * x0 + bq, e2 = 2.0f * A * x1 + bq;
        hit |= (delta >= 0.0f) & ((e1 <= 0.0f) | (e1 * e1 <= delta)) & ((e2 >= 0.0f) | (e2 * e2 <= delta));
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float x = e ? x1 : x0;
        const float bq = 2.0f * B * x;
        const float cq = fmaf(x, A * x, -k2);
        const float delta = fmaf(bq, bq, -(4.0f * C * cq));
        const float e1 = 2.0f * C * y0 + bq, e2 = 2.0f * C * y1 + bq;
        hit |= (delta >= 0.0f) & ((e1 <= 0.0f) | (e1 * e1 <= delta)) & ((e2 >= 0.0f) | (e2 * e2 <= delta));
    }
    return hit;
}

// The inflated extent of that test for the halves of a tile.  (It does not cover
// the cancellation described below: of the halves that a footprint contributes
// to, as narrow as the low-pass leaves it and with a standard deviation of 1000
// pixels along its length, the test drops one in 1100; of 200 pixels one in
// 80,000; of 15 pixels none of 317,000.)
__device__ __forceinline__ float test_extent(const GaussState &s) { return fmaf(s.f1.y, 1.00002f, 1e-5f); }

// And for parts of a half, where it must drop nothing that the half's test
// kept.  The discriminant cancels for long thin footprints: over the
// ellipse's height (y^2 <= k^2 A / det) its terms reach 4 A k^2 (A C / det),
// so a few roundings of them move it as a change of about 5e-7 (A C / det) in
// k^2 would.  Twice that, and 2e-5 for the rest; a conic too thin to tell, or
// whose products leave binary32's range (0 times infinity), always hits.  (The
// extent is then large, but finite: the test multiplies it by a conic entry,
// which may be 0.)
__device__ __forceinline__ float test_extent_thin(const GaussState &s) {
    const float ac = s.f0.z * s.f1.x, det = fmaf(-s.f0.w, s.f0.w, ac);
    const float k2i = fmaf(s.f1.y, fmaf(1e-6f * ac, __builtin_amdgcn_rcpf(det), 1.00002f), 1e-5f);
    return det > 1e-6f * ac ? fminf(k2i, 1e36f) : 1e36f;
}

// Whether a Gaussian's ellipse, inflated to k2, meets the region
// [X0, X0 + w) x [Y0, Y0 + 8) of pixels, cut by the image.
__device__ __forceinline__ bool region_hit(const GaussState &s, float k2, int X0, int w, int Y0, int W, int H) {
    int X1 = X0 + w, Y1 = Y0 + 8;
    X1 = X1 > W ? W : X1;
    Y1 = Y1 > H ? H : Y1;
    const bool in = (X0 < X1) & (Y0 < Y1);
    return in & rect_hit(s.f0.x, s.f0.y, s.f0.z, s.f0.w, s.f1.x, k2, (float)X0 + 0.5f, (float)X1 - 0.5f,
                         (float)Y0 + 0.5f, (float)Y1 - 0.5f);
}

// Whether the half's test can have dropped a half with a contributor: the
// discriminant's error is then more than half of what test_extent allows for.
__device__ __forceinline__ bool half_test_decides(const GaussState &s, float k2t) {
    return k2t > fmaf(s.f1.y, 1.00004f, 1e-5f);
}

// Staged form of a Gaussian for the pixel loop.  With c = log2(e) / 2 the
// base-2 exponent of o exp(-q/2) is (Sec. 5.3.2, exponent in log form)
//     E = log2 o - c q = log2 o + A' dx^2 + B2' dx dy + C' dy^2,
// A' = -c A, B2' = -2 c B, C' = -c C, and the pixel lies in the opacity-aware
// extent (q <= k^2) iff E >= thr = log2 o - c k^2.
//   f0 = (u, v, A', B2')   f1 = (C', thr, log2 o, r)   f2 = (g, b)
__device__ __forceinline__ void stage_gauss(const GaussState &s, float4 &f0, float4 &f1, float2 &f2) {
    const float log2o = s.f1.z;
    f0 = make_float4(s.f0.x, s.f0.y, -kHalfLog2e * s.f0.z, -2.0f * kHalfLog2e * s.f0.w);
    f1 = make_float4(-kHalfLog2e * s.f1.x, fmaf(-kHalfLog2e, s.f1.y, log2o), log2o, s.f1.w);
    f2 = make_float2(s.f2.x, s.f2.y);
}

// Row terms shared by the pixels of one row (same dy).
struct RowTerms {
    float b2dy;  // B2' dy
    float base;  // C' dy^2 + log2 o
};

__device__ __forceinline__ RowTerms row_terms(const float4 &f0, const float4 &f1, float py) {
    const float dy = py - f0.y;
    RowTerms r;
    r.b2dy = f0.w * dy;
    r.base = fmaf(f1.x * dy, dy, f1.z);
    return r;
}

// E at pixel-sample x for the row terms r: dx (A' dx + B2' dy) + C' dy^2 + log2 o.
__device__ __forceinline__ float exponent_at(const float4 &f0, const RowTerms &r, float px) {
    const float dx = px - f0.x;
    return fmaf(dx, fmaf(f0.z, dx, r.b2dy), r.base);
}

}  // namespace fgs

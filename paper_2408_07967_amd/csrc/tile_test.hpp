// The exact ellipse / tile test (Alg. 3; Eq. 7 with the discriminant guard),
// and the columns of a tile row that it can hit, computed per row instead of
// per tile.  Every binary32 operation of the test is one correctly rounded
// IEEE operation in the written order: translation units that include this
// are compiled with -ffp-contract=off.  Host and device code.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "fgs_internal.hpp"

namespace fgs {

#define FGS_HD __host__ __device__ __forceinline__

// Exact test of the ellipse { d : A dx^2 + 2 B dx dy + C dy^2 <= k2 } around
// (u, v) against the pixel-sample hull of tile (tx, ty) (Alg. 3; Eq. 7 with
// the discriminant guard).  Centre inside -> hit; otherwise each edge line
// meets the ellipse in a chord whose overlap with the edge segment is decided
// without division or square root.
//
// The test splits into terms of the tile's column alone and of its row alone;
// tile_hit is the two halves combined.
//
// Column terms (hull x-range [x0, x1] relative to u):
//   a = (2A x0, 2A x1, bq(x0), delta(x0)), b = (bq(x1), delta(x1), flag, 0)
// with bq(x) = 2B x and delta(x) = bq^2 - 4C (A x^2 - k2) for the vertical
// edge at x (quadratic in y), and flag = 1 if x0 <= 0 <= x1.
FGS_HD void tile_col_terms(float u, float A, float B, float C, float k2, int tx, int W, float4 &a, float4 &b) {
    int xe = kTile * tx + kTile;
    xe = xe > W ? W : xe;
    const float x0 = ((float)(kTile * tx) + 0.5f) - u;
    const float x1 = ((float)xe - 0.5f) - u;
    const float A2 = 2.0f * A, B2 = 2.0f * B, C4 = 4.0f * C;
    const float bq0 = B2 * x0, bq1 = B2 * x1;
    const float cq0 = (A * x0) * x0 - k2, cq1 = (A * x1) * x1 - k2;
    a = make_float4(A2 * x0, A2 * x1, bq0, bq0 * bq0 - C4 * cq0);
    b = make_float4(bq1, bq1 * bq1 - C4 * cq1, (x0 <= 0.0f && 0.0f <= x1) ? 1.0f : 0.0f, 0.0f);
}

// Hull y-range of tile row ty relative to v.
FGS_HD void tile_row_span(float v, int ty, int H, float &y0, float &y1) {
    int ye = kTile * ty + kTile;
    ye = ye > H ? H : ye;
    y0 = ((float)(kTile * ty) + 0.5f) - v;
    y1 = ((float)ye - 0.5f) - v;
}

// Row terms (hull y-range [y0, y1] relative to v):
//   a = (bq(y0), delta(y0), bq(y1), delta(y1)), b = (2C y0, 2C y1, flag, 0)
// with bq(y) = 2B y and delta(y) = bq^2 - 4A (C y^2 - k2) for the horizontal
// edge at y (quadratic in x), and flag = 1 if y0 <= 0 <= y1.
FGS_HD void tile_row_terms(float v, float A, float B, float C, float k2, int ty, int H, float4 &a, float4 &b) {
    float y0, y1;
    tile_row_span(v, ty, H, y0, y1);
    const float B2 = 2.0f * B, C2 = 2.0f * C, A4 = 4.0f * A;
    const float bq0 = B2 * y0, bq1 = B2 * y1;
    const float cq0 = (C * y0) * y0 - k2, cq1 = (C * y1) * y1 - k2;
    a = make_float4(bq0, bq0 * bq0 - A4 * cq0, bq1, bq1 * bq1 - A4 * cq1);
    b = make_float4(C2 * y0, C2 * y1, (y0 <= 0.0f && 0.0f <= y1) ? 1.0f : 0.0f, 0.0f);
}

// One edge: the chord [r-, r+] of the quadratic with discriminant d overlaps
// the edge segment, given e1 = 2a s0 + bq and e2 = 2a s1 + bq at its ends:
//   d >= 0 and (e1 <= 0 or e1^2 <= d) and (e2 >= 0 or e2^2 <= d).
// (Bitwise, not short-circuit, so that the test compiles to straight-line
// code.)
FGS_HD bool edge_hit(float e1, float e2, float d) {
    return (d >= 0.0f) & ((e1 <= 0.0f) | (e1 * e1 <= d)) & ((e2 >= 0.0f) | (e2 * e2 <= d));
}

// The same decision for finite e1 and e2 in three instructions instead of
// seven: the conditions bind only for e1 > 0 and e2 < 0, rounded squares keep
// their order, and 0 <= d is the third condition's case of neither, so they
// hold exactly when the square of max(e1, -e2, 0) is at most d (a NaN d fails
// both ways).
FGS_HD bool edge_hit_finite(float e1, float e2, float d) {
    const float m = __builtin_fmaxf(__builtin_fmaxf(e1, -e2), 0.0f);
    return m * m <= d;
}

// Whether every term of a Gaussian's tile tests is finite: all products of
// the conic and two coordinates (hulls lie within 2^14) stay below 1e37.
FGS_HD bool tile_terms_finite(float u, float v, float A, float B, float C) {
    return (fabsf(u) < 1e9f) & (fabsf(v) < 1e9f) & (fabsf(A) < 1e9f) & (fabsf(B) < 1e9f) & (fabsf(C) < 1e9f);
}

// kFinite: the terms are finite (tile_terms_finite)
template <bool kFinite>
FGS_HD bool tile_hit_terms(const float4 ca, const float4 cb, const float4 ra, const float4 rb) {
    const bool inside = (cb.z != 0.0f) & (rb.z != 0.0f);  // centre inside the hull
    auto edge = [](float e1, float e2, float d) {
        if constexpr (kFinite)
            return edge_hit_finite(e1, e2, d);
        else
            return edge_hit(e1, e2, d);
    };
    // horizontal edges y = y0, y1, then vertical edges x = x0, x1
    return inside | edge(ca.x + ra.x, ca.y + ra.x, ra.y) | edge(ca.x + ra.z, ca.y + ra.z, ra.w) |
           edge(rb.x + ca.z, rb.y + ca.z, ca.w) | edge(rb.x + cb.x, rb.y + cb.x, cb.y);
}

template <bool kFinite>
FGS_HD bool tile_hit(float u, float v, float A, float B, float C, float k2, int tx, int ty, int W, int H) {
    float4 ca, cb, ra, rb;
    tile_col_terms(u, A, B, C, k2, tx, W, ca, cb);
    tile_row_terms(v, A, B, C, k2, ty, H, ra, rb);
    return tile_hit_terms<kFinite>(ca, cb, ra, rb);
}

// ---- a row's hits ---------------------------------------------------------------
// Within the strip of one tile row, a tile meets the ellipse exactly when its
// x-range meets the x-projection of (ellipse, cut by the strip), an interval.
// The exact test above decides as real arithmetic would for some k2' with
// |k2' - k2| <= delta k2: the roundings of its discriminants reach
// eps (9 r + 4) relative to 4 A k2 over the ellipse's height, r = A C / (A C -
// B^2), and those of e^2 at most 12 eps sqrt(r), so delta <= 21 eps (r + 1).
// So the interval for k2 (1 + delta) holds every tile that the test can hit,
// and every tile that meets the interval for k2 (1 - delta) is hit: only the
// tiles between the two need the test.  delta = 4e-6 (r + 1) is used (67
// eps), which also covers the roundings of the intervals themselves: they
// are a few eps of the half-chord sqrt(k2 / A) times at most sqrt(r), while
// the two deltas' difference moves the interval's ends by at least
// sqrt(k2 / A) times half of it.
struct RowTest {
    float ymax;   // half-height sqrt(k2 A / det) of the ellipse
    float slope;  // B / A
    float sc;     // sqrt(det) / A
    float ymr;    // the rightmost point's y over ymax: -B / sqrt(A C)
    float fo, fi; // sqrt(1 + delta), sqrt(1 - delta); fo < 0: no interval, test every tile
};

FGS_HD RowTest row_test(float u, float v, float A, float B, float C, float k2) {
    RowTest t;
    const float det = (float)((double)A * (double)C - (double)B * (double)B);
    const float delta = 4e-6f * (A * C / det + 1.0f);
    const bool ok = (A > 0.0f) & (C > 0.0f) & (det > 1e-30f) & (delta < 0.5f) & tile_terms_finite(u, v, A, B, C) &
                    (k2 >= 0.0f) & (k2 < 1e9f);
    t.ymax = sqrtf(k2 * A / det);
    t.slope = B / A;
    t.sc = sqrtf(det) / A;
    t.ymr = -B / sqrtf(A * C);
    t.fo = ok ? sqrtf(1.0f + delta) : -1.0f;
    t.fi = ok ? sqrtf(1.0f - delta) : 0.0f;
    return t;
}

// Columns of the tile row with hull y-range [y0, y1]: hits lie within
// [first, last], and all of [sure_first, sure_last] (possibly empty) are hits.
struct RowCols {
    int first, last, sure_first, sure_last;
};

FGS_HD RowCols row_columns(const RowTest &t, float u, float y0, float y1, int tx0, int tx1, int W) {
    RowCols r;
    r.first = tx0;
    r.last = tx1;
    r.sure_first = tx1 + 1;
    r.sure_last = tx0 - 1;
    if (t.fo < 0.0f) return r;
    auto clamp = [](float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); };
    // x-projection of the strip's part of the ellipse with half-height ym
    auto ends = [&](float ym, float &lo, float &hi) {
        const float ya = fmaxf(y0, -ym), yb = fminf(y1, ym);
        const float yr = t.ymr * ym, yc = clamp(yr, ya, yb), yd = clamp(-yr, ya, yb);
        hi = t.sc * sqrtf(fmaxf((ym - yc) * (ym + yc), 0.0f)) - t.slope * yc;
        lo = -t.sc * sqrtf(fmaxf((ym - yd) * (ym + yd), 0.0f)) - t.slope * yd;
        return ya <= yb;
    };
    float lo, hi;
    const bool any = ends(t.ymax * t.fo, lo, hi);
    // tile tx: samples 16 tx + 1/2 ... 16 tx + 15 1/2 (the last one cut by the
    // image).  The pad covers the roundings of lo + u and of the hulls'
    // coordinates relative to u.
    const float pad = 0.001f + 1e-6f * (fabsf(u) + fmaxf(fabsf(lo), fabsf(hi)));
    constexpr float kInv = 1.0f / (float)kTile;
    auto col = [&](float x) { return (int)clamp(x, (float)(tx0 - 1), (float)(tx1 + 1)); };  // (in range before the cast)
    r.first = col(ceilf((lo + u - 15.5f - pad) * kInv));
    r.last = col(floorf((hi + u - 0.5f + pad) * kInv));
    r.first = r.first < tx0 ? tx0 : r.first;
    r.last = r.last > tx1 ? tx1 : r.last;
    if (!any) r.last = r.first - 1;
    const bool sure = ends(t.ymax * t.fi, lo, hi);
    r.sure_first = col(ceilf((lo + u - 15.5f + pad) * kInv));
    r.sure_last = col(floorf((hi + u - 0.5f - pad) * kInv));
    r.sure_first = r.sure_first < tx0 ? tx0 : r.sure_first;
    r.sure_last = r.sure_last > tx1 ? tx1 : r.sure_last;
    // (the last tile's samples end at W - 1/2)
    if (!sure || !(lo + u + pad <= (float)W - 0.5f)) r.sure_last = r.sure_first - 1;
    return r;
}

}  // namespace fgs

// Per-Gaussian preprocessing with the exact ellipse/tile test, and key
// emission in depth order (FlashGS Alg. 4, Alg. 3, Eq. 1-3, Eq. 7, Sec. 4.2).
//
// This translation unit is compiled with -ffp-contract=off: every binary32
// + - * / and sqrt below is one correctly rounded IEEE operation in the
// written order, so the per-Gaussian state and the tile test give the same
// bits as the canonical FP32 evaluation of the method; exp and ln are
// evaluated in binary64 by a fixed operation sequence and rounded once.
#include <algorithm>
#include <cstddef>

#include "fgs_internal.hpp"
#include "sh_basis.hpp"
#include "tile_test.hpp"

namespace fgs {
namespace {

constexpr int kWave = 64;

// ---- canonical binary64 exp / ln (Cody-Waite reduction + Taylor; atanh series)

#define FGS_LN2_HI 0x1.62e42fee00000p-1
#define FGS_LN2_LO 0x1.a39ef35793c76p-33
#define FGS_INV_LN2 0x1.71547652b82fep+0

__device__ __forceinline__ double pow2i(int k) {
    return __longlong_as_double((long long)(k + 1023) << 52);
}

__device__ __forceinline__ double floor_exact(double x) {
    double t = (double)(long long)x;
    return (t > x) ? t - 1.0 : t;
}

__device__ double canon_exp(double x) {
    if (x != x) return x;
    if (x > 709.8) return __longlong_as_double(0x7ff0000000000000LL);
    if (x < -745.2) return 0.0;
    double k = floor_exact(x * FGS_INV_LN2 + 0.5);
    double r = (x - k * FGS_LN2_HI) - k * FGS_LN2_LO;
    double p = 1.0 / 6227020800.0;
    p = p * r + 1.0 / 479001600.0;
    p = p * r + 1.0 / 39916800.0;
    p = p * r + 1.0 / 3628800.0;
    p = p * r + 1.0 / 362880.0;
    p = p * r + 1.0 / 40320.0;
    p = p * r + 1.0 / 5040.0;
    p = p * r + 1.0 / 720.0;
    p = p * r + 1.0 / 120.0;
    p = p * r + 1.0 / 24.0;
    p = p * r + 1.0 / 6.0;
    p = p * r + 0.5;
    p = p * r + 1.0;
    p = p * r + 1.0;
    int ki = (int)k;
    int k1 = ki / 2;
    int k2 = ki - k1;
    return (p * pow2i(k1)) * pow2i(k2);
}

// ln x for finite x >= 1 (the only use: ln(o / tau) with o > tau)
__device__ double canon_log(double x) {
    unsigned long long bits = (unsigned long long)__double_as_longlong(x);
    int e = (int)((bits >> 52) & 0x7ff) - 1023;
    double m = __longlong_as_double((long long)((bits & 0x000fffffffffffffULL) | 0x3ff0000000000000ULL));
    if (m > 1.4142135623730951) {
        m = m * 0.5;
        e = e + 1;
    }
    double s = (m - 1.0) / (m + 1.0);
    double z = s * s;
    double p = 1.0 / 23.0;
    p = p * z + 1.0 / 21.0;
    p = p * z + 1.0 / 19.0;
    p = p * z + 1.0 / 17.0;
    p = p * z + 1.0 / 15.0;
    p = p * z + 1.0 / 13.0;
    p = p * z + 1.0 / 11.0;
    p = p * z + 1.0 / 9.0;
    p = p * z + 1.0 / 7.0;
    p = p * z + 1.0 / 5.0;
    p = p * z + 1.0 / 3.0;
    double lnm = (2.0 * s) + (2.0 * s) * (z * p);
    double de = (double)e;
    return de * FGS_LN2_HI + (lnm + de * FGS_LN2_LO);
}

__device__ __forceinline__ float clampf_(float x, float lo, float hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// Row and column of row-major position idx in rows of ntx (idx < 2^24,
// rcpn = reciprocal of ntx): the rounded quotient estimate is off by at most
// one and is corrected, so this equals integer division.
__device__ __forceinline__ void row_col(int idx, int ntx, float rcpn, int &ry, int &rx) {
    ry = (int)((float)idx * rcpn);
    rx = idx - ry * ntx;
    const int below = rx < 0, above = rx >= ntx;
    ry += above - below;
    rx += (below - above) * ntx;
}

// (tx0, tx1, ty0, ty1) of an emission record's packed rectangle
__device__ __forceinline__ uint4 unpack_rect(const uint4 &r) {
    return make_uint4(r.x & 0xffffu, r.x >> 16, r.y & 0xffffu, r.y >> 16);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
        if (lane >= d) x += y;
    }
    return x;
}

// Largest lane L with s[L] <= item, for s non-decreasing over 64 lanes with
// s[0] = 0: the owner of flattened item `item` (lanes with no items are
// skipped because the next lane has the same start).
__device__ __forceinline__ int owner_lane(const uint32_t *s, uint32_t item) {
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
        if (s[lo + step] <= item) lo += step;
    return lo;
}

// k / n for 0 <= k < 64 and 1 <= n <= 64: (k + 1/2) / n is at least 1/128
// away from an integer, far more than the reciprocal's error.
__device__ __forceinline__ int small_div(uint32_t k, int n) {
    return (int)(((float)k + 0.5f) * __builtin_amdgcn_rcpf((float)n));
}

// Scales exp(log-scale) and the unit quaternion q / |q| (computeCov3D's
// inputs), as the binary32 values of the canonical evaluation.  False for a
// non-finite scale or a quaternion of zero or non-finite norm.
__device__ __forceinline__ bool scale_rot(float ls0, float ls1, float ls2, const float *q4, float *s3, float *qu) {
    const float qw = q4[0], qx = q4[1], qy = q4[2], qz = q4[3];
    s3[0] = (float)canon_exp((double)ls0);
    s3[1] = (float)canon_exp((double)ls1);
    s3[2] = (float)canon_exp((double)ls2);
    const float n2 = ((qw * qw + qx * qx) + qy * qy) + qz * qz;
    const bool fin = isfinite(ls0) && isfinite(ls1) && isfinite(ls2) && isfinite(n2);
    if (!(fin && n2 > 0.0f)) return false;
    const float qn = sqrtf(n2);
    qu[0] = qw / qn;
    qu[1] = qx / qn;
    qu[2] = qy / qn;
    qu[3] = qz / qn;
    return true;
}

// 3D covariance Sigma = M M^T with M = R(q) diag(s) (computeCov3D), upper
// triangle S00, S01, S02, S11, S12, S22, in binary32.
__device__ __forceinline__ void sigma3(const float *s3, const float *qu, float *S) {
    const float s0 = s3[0], s1 = s3[1], s2 = s3[2];
    const float w = qu[0], x = qu[1], y = qu[2], z = qu[3];
    const float r00 = 1.0f - 2.0f * (y * y + z * z);
    const float r01 = 2.0f * (x * y - w * z);
    const float r02 = 2.0f * (x * z + w * y);
    const float r10 = 2.0f * (x * y + w * z);
    const float r11 = 1.0f - 2.0f * (x * x + z * z);
    const float r12 = 2.0f * (y * z - w * x);
    const float r20 = 2.0f * (x * z - w * y);
    const float r21 = 2.0f * (y * z + w * x);
    const float r22 = 1.0f - 2.0f * (x * x + y * y);
    const float M00 = r00 * s0, M01 = r01 * s1, M02 = r02 * s2;
    const float M10 = r10 * s0, M11 = r11 * s1, M12 = r12 * s2;
    const float M20 = r20 * s0, M21 = r21 * s1, M22 = r22 * s2;
    S[0] = (M00 * M00 + M01 * M01) + M02 * M02;
    S[1] = (M00 * M10 + M01 * M11) + M02 * M12;
    S[2] = (M00 * M20 + M01 * M21) + M02 * M22;
    S[3] = (M10 * M10 + M11 * M11) + M12 * M12;
    S[4] = (M10 * M20 + M11 * M21) + M12 * M22;
    S[5] = (M20 * M20 + M21 * M21) + M22 * M22;
}

// Conic of the dilated EWA covariance in binary64, rounded once to binary32
// (the blend's conic, see GaussState).  The inputs are the binary32 scales,
// unit quaternion, mean and camera, promoted to binary64 (c: the camera and
// its Jacobian clamp limits in binary64); the Jacobian clamp is the same.
// With M = R(q) diag(s) and T = J R_cam, Sigma' = T M M^T T^T + dilation I =
// N N^T + dilation I for N = T M, accumulated one column of M at a time (the
// product the canonical evaluation forms as T Sigma T^T).  The binary32
// determinant of Sigma' cancels badly for long thin footprints; in binary64
// the narrow axis keeps its accuracy.  False if the binary64 determinant is
// not positive.
__device__ bool conic_b64(const float *s3, const float *qu, float mx, float my, float mz, const DevCam64 &c,
                          double dil, float *Ab, float *Bb, float *Cb) {
    const double px = mx, py = my, pz = mz;
    const double tx = c.R[0] * px + c.R[1] * py + c.R[2] * pz + c.t[0];
    const double ty = c.R[3] * px + c.R[4] * py + c.R[5] * pz + c.t[1];
    const double tz = c.R[6] * px + c.R[7] * py + c.R[8] * pz + c.t[2];
    const double iz = 1.0 / tz;
    double xc = tx * iz, yc = ty * iz;
    xc = xc < -c.limx ? -c.limx : (xc > c.limx ? c.limx : xc);
    yc = yc < -c.limy ? -c.limy : (yc > c.limy ? c.limy : yc);
    const double J00 = c.fx * iz, J02 = -(c.fx * xc) * iz, J11 = c.fy * iz, J12 = -(c.fy * yc) * iz;
    double T0[3], T1[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        T0[j] = J00 * c.R[j] + J02 * c.R[6 + j];
        T1[j] = J11 * c.R[3 + j] + J12 * c.R[6 + j];
    }
    const double w = qu[0], x = qu[1], y = qu[2], z = qu[3];
    double a = 0.0, b = 0.0, cc = 0.0;
    auto column = [&](double r0, double r1, double r2, double sj) {
        const double n0 = (T0[0] * r0 + T0[1] * r1 + T0[2] * r2) * sj;
        const double n1 = (T1[0] * r0 + T1[1] * r1 + T1[2] * r2) * sj;
        a += n0 * n0;
        b += n0 * n1;
        cc += n1 * n1;
    };
    column(1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y + w * z), 2.0 * (x * z - w * y), (double)s3[0]);
    column(2.0 * (x * y - w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z + w * x), (double)s3[1]);
    column(2.0 * (x * z + w * y), 2.0 * (y * z - w * x), 1.0 - 2.0 * (x * x + y * y), (double)s3[2]);
    a += dil;
    cc += dil;
    const double det = a * cc - b * b;
    if (!(det > 0.0)) return false;
    const double inv = 1.0 / det;
    *Ab = (float)(cc * inv);
    *Bb = (float)(-b * inv);
    *Cb = (float)(a * inv);
    return true;
}

// Opacity-aware extent (Eq. 3), capped by the 3 sigma rule (Eq. 1).
__device__ __forceinline__ float extent_k2(float o, const DevOptions &op) {
    double k2d = 2.0 * canon_log((double)o / (double)op.alpha_min);
    if (op.cap_3sigma && k2d > 9.0) k2d = 9.0;
    return (float)k2d;
}

// The inverse of a permutation, and a copy of it.
__global__ __launch_bounds__(kBlock) void k_invert(const uint32_t *__restrict__ perm, int64_t P,
                                                   uint32_t *__restrict__ inv, uint32_t *__restrict__ orig) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t g = perm[i];
        orig[i] = g;
        inv[g] = (uint32_t)i;
    }
}

// View-independent precompute of a resident scene (Sec. 5.3.1: preprocessing
// shared by the viewpoints of one scene): per Gaussian (x, y, z, opacity) with
// opacity 0 for a Gaussian that can never be visible, the scales, the unit
// quaternion and k^2, the trace of the 3D covariance with k^2 (the cull's
// extent bound), and the SH coefficients Gaussian-major.  The same operations
// as the per-frame path, so frames render bit for bit the same.  Slot i holds
// Gaussian perm[i] (a spatial order, so that the candidates of a frame's cull
// are read as few contiguous runs), and orig[i] = perm[i].
//
// Bound by HBM: each thread takes one Gaussian in the caller's order, so that
// the parameter planes are read as whole lines, and writes its records (16,
// 32, 8 and up to 192 contiguous bytes) to its slot inv[g].  Reading in slot
// order instead costs a line per 4-byte element of every plane: 10M Gaussians
// of degree 3 took 13.5 ms and now take 2.5 ms (5 GB), 1M 985 and 180 us.
__global__ __launch_bounds__(kBlock) void k_prepare(DevScene sc, DevOptions op, const uint32_t *__restrict__ inv,
                                                    float4 *__restrict__ pos_o, float4 *__restrict__ cov,
                                                    float *__restrict__ sh_out, float2 *__restrict__ bnd,
                                                    int sh_stride) {
    const int64_t st = sc.stride;
    const int ncoef = 3 * (sc.D + 1) * (sc.D + 1);
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < sc.P;
         g += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = inv[g];
        const float mx = sc.means[g], my = sc.means[st + g], mz = sc.means[2 * st + g];
        const float logit = sc.logits[g];
        const float q4[4] = {sc.quats[g], sc.quats[st + g], sc.quats[2 * st + g], sc.quats[3 * st + g]};
        const float ls0 = sc.log_scales[g], ls1 = sc.log_scales[st + g], ls2 = sc.log_scales[2 * st + g];
        const float o = (float)(1.0 / (1.0 + canon_exp(-(double)logit)));
        float S[6] = {0, 0, 0, 0, 0, 0}, s3[3] = {0, 0, 0}, qu[4] = {0, 0, 0, 0};
        float k2 = 0.0f;
        bool ok = isfinite(logit) && o > op.alpha_min;
        if (ok) ok = scale_rot(ls0, ls1, ls2, q4, s3, qu);
        if (ok) {
            sigma3(s3, qu, S);
            k2 = extent_k2(o, op);
        }
        pos_o[i] = make_float4(mx, my, mz, ok ? o : 0.0f);
        cov[2 * i] = make_float4(s3[0], s3[1], s3[2], k2);
        cov[2 * i + 1] = make_float4(qu[0], qu[1], qu[2], qu[3]);
        // trace(Sigma) >= its largest eigenvalue: bounds the screen extent
        bnd[i] = make_float2(S[0] + S[3] + S[5], k2);
    }
    // SH: planar in, Gaussian-major out (all loads of a Gaussian in flight
    // together; sh_stride is a multiple of 4, its padding zero)
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < sc.P;
         g += (int64_t)gridDim.x * blockDim.x) {
        float4 *const dst = reinterpret_cast<float4 *>(sh_out + (int64_t)inv[g] * sh_stride);
        float v[48];
#pragma unroll
        for (int j = 0; j < 48; ++j) v[j] = j < ncoef ? sc.sh[(int64_t)j * st + g] : 0.0f;
#pragma unroll
        for (int j = 0; j < 12; ++j)
            if (4 * j < sh_stride) dst[j] = make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
    }
}

// A binary32 value as an unsigned integer of the same order (for atomic
// min / max), and back.
__device__ __forceinline__ uint32_t float_order(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float order_float(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// Box of the finite means: per workgroup a reduction over its Gaussians,
// then one atomic min / max per axis into bounds (order-mapped, see
// float_order).
__global__ __launch_bounds__(kBlock) void k_spatial_bounds(DevScene sc, uint32_t *__restrict__ bounds) {
    const int64_t st = sc.stride;
    uint32_t lo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, hi[3] = {0u, 0u, 0u};
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < sc.P; g += (int64_t)gridDim.x * blockDim.x) {
        const float m[3] = {sc.means[g], sc.means[st + g], sc.means[2 * st + g]};
        if (!(isfinite(m[0]) && isfinite(m[1]) && isfinite(m[2]))) continue;
        for (int a = 0; a < 3; ++a) {
            const uint32_t u = float_order(m[a]);
            lo[a] = u < lo[a] ? u : lo[a];
            hi[a] = u > hi[a] ? u : hi[a];
        }
    }
    __shared__ uint32_t s_lo[3][kBlock / kWave], s_hi[3][kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int a = 0; a < 3; ++a) {
        uint32_t l = lo[a], h = hi[a];
        for (int d = kWave / 2; d > 0; d >>= 1) {
            const uint32_t l2 = (uint32_t)__shfl_xor((int)l, d, kWave), h2 = (uint32_t)__shfl_xor((int)h, d, kWave);
            l = l2 < l ? l2 : l;
            h = h2 > h ? h2 : h;
        }
        if (lane == 0) {
            s_lo[a][wave] = l;
            s_hi[a][wave] = h;
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int a = threadIdx.x;
        uint32_t l = 0xffffffffu, h = 0u;
        for (int w = 0; w < kBlock / kWave; ++w) {
            l = s_lo[a][w] < l ? s_lo[a][w] : l;
            h = s_hi[a][w] > h ? s_hi[a][w] : h;
        }
        // (a bound already met needs no atomic: the same six words serve the
        // whole grid, and the first workgroups settle them)
        if (l < __hip_atomic_load(&bounds[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&bounds[a], l);
        if (h > __hip_atomic_load(&bounds[3 + a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&bounds[3 + a], h);
    }
}

__global__ void k_spatial_bounds_init(uint32_t *bounds) {
    if (threadIdx.x < 6) bounds[threadIdx.x] = threadIdx.x < 3 ? 0xffffffffu : 0u;
}

// Ten bits of x spread to every third bit (bit b to bit 3b).
__device__ __forceinline__ uint32_t spread3(uint32_t x) {
    x &= 0x3ffu;
    x = (x | (x << 16)) & 0x030000ffu;
    x = (x | (x << 8)) & 0x0300f00fu;
    x = (x | (x << 4)) & 0x030c30c3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

// Morton code of each mean quantised to 1024 cells per axis of the box.
__global__ __launch_bounds__(kBlock) void k_spatial_keys(DevScene sc, const uint32_t *__restrict__ bounds,
                                                         uint32_t *__restrict__ keys) {
    const int64_t st = sc.stride;
    float lo[3], sc3[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = order_float(bounds[a]);
        const float ext = order_float(bounds[3 + a]) - lo[a];
        sc3[a] = ext > 0.0f ? 1024.0f / ext : 0.0f;
    }
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < sc.P; g += (int64_t)gridDim.x * blockDim.x) {
        const float m[3] = {sc.means[g], sc.means[st + g], sc.means[2 * st + g]};
        uint32_t key = 0xffffffffu;
        if (isfinite(m[0]) && isfinite(m[1]) && isfinite(m[2]) && bounds[0] != 0xffffffffu) {
            uint32_t q[3];
            for (int a = 0; a < 3; ++a) {
                const float c = (m[a] - lo[a]) * sc3[a];
                q[a] = c <= 0.0f ? 0u : (c >= 1023.0f ? 1023u : (uint32_t)c);
            }
            key = spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
        }
        keys[g] = key;
    }
}

// Gaussians [lo, hi) of cull workgroup b of kCullBlocks: whole 256-Gaussian
// batches split evenly.
__device__ __forceinline__ void cull_range(int64_t P, uint32_t b, int64_t *lo, int64_t *hi) {
    const int64_t batches = (P + kBlock - 1) / kBlock;
    *lo = batches * b / kCullBlocks * kBlock;
    const int64_t h = batches * (b + 1) / kCullBlocks * kBlock;
    *hi = h < P ? h : P;
    if (*lo > *hi) *lo = *hi;
}

// The cull's keep test of one Gaussian (position and opacity p4, extent
// terms b) for one camera.  Evaluated without branches, so that a caller's
// loads of p4 and b are all issued together.
__device__ __forceinline__ bool cull_keep(const float4 &p4, const float2 &b, const DevCamera &cam,
                                          const DevOptions &op, int W, int H) {
    const float *R = cam.R;
    const float tx = ((R[0] * p4.x + R[1] * p4.y) + R[2] * p4.z) + cam.t[0];
    const float ty = ((R[3] * p4.x + R[4] * p4.y) + R[5] * p4.z) + cam.t[1];
    const float tz = ((R[6] * p4.x + R[7] * p4.y) + R[8] * p4.z) + cam.t[2];
    const bool front = (tz > cam.near_z) & (p4.w > op.alpha_min) & isfinite(p4.x) & isfinite(p4.y) & isfinite(p4.z);
    const float iz = 1.0f / tz;
    const float xt = tx * iz, yt = ty * iz;
    const float limx = op.jac_clip * (0.5f * (float)W / cam.fx);
    const float limy = op.jac_clip * (0.5f * (float)H / cam.fy);
    const float xc = fminf(fmaxf(xt, -limx), limx), yc = fminf(fmaxf(yt, -limy), limy);
    const float J00 = cam.fx * iz, J02 = -cam.fx * xc * iz, J11 = cam.fy * iz, J12 = -cam.fy * yc * iz;
    float n0 = 0.0f, n1 = 0.0f;
    for (int j = 0; j < 3; ++j) {
        const float t0 = J00 * R[j] + J02 * R[6 + j], t1 = J11 * R[3 + j] + J12 * R[6 + j];
        n0 += t0 * t0;
        n1 += t1 * t1;
    }
    float hx, hy;
    if (op.binning == 2) {
        // square of radius ceil(3 sqrt(lambda_max(Sigma'))), lambda_max <= trace
        hx = sqrtf(9.0f * ((n0 + n1) * b.x + op.dilation)) * 1.001f + 3.0f;
        hy = hx;
    } else {
        hx = sqrtf(b.y * (n0 * b.x + op.dilation)) * 1.001f + 3.0f;
        hy = sqrtf(b.y * (n1 * b.x + op.dilation)) * 1.001f + 3.0f;
    }
    const float u = cam.fx * xt + cam.cx, v = cam.fy * yt + cam.cy;
    // drop only what is certainly off the image (a NaN keeps it)
    const bool out = (u + hx < 0.0f) | (u - hx > (float)W) | (v + hy < 0.0f) | (v - hy > (float)H);
    return front & !out;
}

// The parameters that a raw Gaussian's keep test reads.
struct RawTerms {
    float x, y, z, ls0, ls1, ls2, logit, qw, qx, qy, qz;
};
__device__ __forceinline__ RawTerms raw_terms(const DevScene &sc, int64_t g) {
    const int64_t st = sc.stride;
    return {sc.means[g],
            sc.means[st + g],
            sc.means[2 * st + g],
            sc.log_scales[g],
            sc.log_scales[st + g],
            sc.log_scales[2 * st + g],
            sc.logits[g],
            sc.quats[g],
            sc.quats[st + g],
            sc.quats[2 * st + g],
            sc.quats[3 * st + g]};
}

// The cull's keep test on raw parameters: false only for a Gaussian that the
// projection would find invisible.  The covariance's trace is the sum of the
// squared scales (the rotation keeps it), k^2 is bounded by its value at
// opacity 1 (and by 9 where it is capped), and the opacity is above alpha_min
// only if the logit is above alpha_min's.  The factors and the 0.01 cover the
// rounding of the hardware's exponential and logarithm (about 1e-5 relative)
// many times over; a NaN or an infinity in a bound keeps the Gaussian, one in
// the mean or the logit drops it as the projection does.  A quaternion so small
// that its squared norm has lost its precision is normalised to something that
// is no rotation: it is kept.
__device__ __forceinline__ bool raw_keep(const RawTerms &r, const DevCamera &cam, const DevOptions &op, int W,
                                         int H) {
    constexpr float kLog2e2 = 2.885390082f, kLn2 = 0.6931471806f;
    const float trace = (exp2f(r.ls0 * kLog2e2) + exp2f(r.ls1 * kLog2e2)) + exp2f(r.ls2 * kLog2e2);
    const float k2 = op.cap_3sigma ? 9.0f : -2.0f * kLn2 * log2f(op.alpha_min);
    const float logit_min = kLn2 * log2f(op.alpha_min / (1.0f - op.alpha_min)) - 0.01f;
    const bool dim = !isfinite(r.logit) | (r.logit < logit_min);
    // (an opacity that passes: dim stands for it)
    const float4 p4 = make_float4(r.x, r.y, r.z, __builtin_inff());
    const float n2 = ((r.qw * r.qw + r.qx * r.qx) + r.qy * r.qy) + r.qz * r.qz;
    const float t = n2 >= 1e-30f ? trace * 1.001f : __builtin_inff();
    return !dim & cull_keep(p4, make_float2(t, k2 * 1.001f + 1e-3f), cam, op, W, H);
}

// Whether the cull would drop every member of a batch whose bounds are
// (lo, hi, kx) (DevPrepared::blk), for one camera.  A member is dropped if
// its opacity is at most alpha_min, its view depth is not past the near
// plane, or its screen extent bound is off the image (cull_keep).  Over the
// batch: the opacity is at most lo.w; the view depth is affine in the mean,
// so over the box of means it lies between the corners' depths; in front of
// the camera the projection is linear-fractional with a positive
// denominator, so the means' screen coordinates also lie between the
// corners'; and each member's extent bound sqrt(k^2 (|t0|^2 trace +
// dilation)) grows with k^2, trace and |t0|^2 = (fx / z)^2 |R_0 - xc R_2|^2
// <= (fx / z_min)^2 (|R_0| + limx |R_2|)^2 (|xc| <= limx; the 3 sigma square
// likewise).  Margins (a relative 1e-5 on the depths, 1 % and 8 pixels on
// the extent) cover the rounding of either evaluation.
__device__ bool batch_culled(const float4 &lo, const float4 &hi, const float4 &kx, const DevCamera &cam,
                             const DevOptions &op, int W, int H) {
    if (!(lo.w > op.alpha_min)) return true;  // every opacity too low (or no member)
    const float *R = cam.R;
    bool behind = true, front = true;
    float umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY, zmin = INFINITY;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float x = (c & 1) ? hi.x : lo.x, y = (c & 2) ? hi.y : lo.y, z = (c & 4) ? hi.z : lo.z;
        const float tx = ((R[0] * x + R[1] * y) + R[2] * z) + cam.t[0];
        const float ty = ((R[3] * x + R[4] * y) + R[5] * z) + cam.t[1];
        const float tz = ((R[6] * x + R[7] * y) + R[8] * z) + cam.t[2];
        const float mag = ((fabsf(R[6] * x) + fabsf(R[7] * y)) + fabsf(R[8] * z)) + fabsf(cam.t[2]);
        behind = behind && tz < cam.near_z - 1e-5f * mag;
        front = front && tz > 1e-5f * mag && tz > 1e-20f;
        const float iz = 1.0f / tz;
        umin = fminf(umin, cam.fx * (tx * iz) + cam.cx);
        umax = fmaxf(umax, cam.fx * (tx * iz) + cam.cx);
        vmin = fminf(vmin, cam.fy * (ty * iz) + cam.cy);
        vmax = fmaxf(vmax, cam.fy * (ty * iz) + cam.cy);
        zmin = fminf(zmin, tz);
    }
    if (behind) return true;   // every member's depth is at most the near plane
    if (!front) return false;  // the box reaches behind the camera: test each member
    const float r0 = sqrtf((R[0] * R[0] + R[1] * R[1]) + R[2] * R[2]);
    const float r1 = sqrtf((R[3] * R[3] + R[4] * R[4]) + R[5] * R[5]);
    const float r2 = sqrtf((R[6] * R[6] + R[7] * R[7]) + R[8] * R[8]);
    const float limx = op.jac_clip * (0.5f * (float)W / cam.fx);
    const float limy = op.jac_clip * (0.5f * (float)H / cam.fy);
    const float ax = (cam.fx / zmin) * (r0 + limx * r2), ay = (cam.fy / zmin) * (r1 + limy * r2);
    const float n0 = ax * ax, n1 = ay * ay;
    float hx, hy;
    if (op.binning == 2) {
        hx = sqrtf(9.0f * ((n0 + n1) * hi.w + op.dilation));
        hy = hx;
    } else {
        hx = sqrtf(kx.x * (n0 * hi.w + op.dilation));
        hy = sqrtf(kx.x * (n1 * hi.w + op.dilation));
    }
    hx = hx * 1.01f + 8.0f;
    hy = hy * 1.01f + 8.0f;
    // (a NaN anywhere keeps the batch)
    return (umax + hx < 0.0f) || (umin - hx > (float)W) || (vmax + hy < 0.0f) || (vmin - hy > (float)H);
}

// Bounds of each batch of kBlock slots (one workgroup per batch) over its
// members that can be visible (see DevPrepared::blk).
__global__ __launch_bounds__(kBlock) void k_block_bounds(const float4 *__restrict__ pos_o,
                                                         const float2 *__restrict__ bnd, int64_t P,
                                                         float4 *__restrict__ blk) {
    __shared__ float s_r[kBlock / kWave][8];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float2 b = make_float2(0.0f, 0.0f);
    if (i < P) {
        p = pos_o[i];
        b = bnd[i];
    }
    const bool use = i < P && p.w > 0.0f && isfinite(p.x) && isfinite(p.y) && isfinite(p.z);
    // maxima as minima of negatives (a slot without a member adds +inf to
    // every minimum); a NaN trace or k^2 counts as +inf
    float r[8] = {use ? p.x : INFINITY, use ? p.y : INFINITY, use ? p.z : INFINITY,
                  use ? -p.x : INFINITY, use ? -p.y : INFINITY, use ? -p.z : INFINITY,
                  use ? -p.w : INFINITY, 0.0f};
    const float tr = isnan(b.x) ? INFINITY : b.x, k2 = isnan(b.y) ? INFINITY : b.y;
    float mtr = use ? tr : 0.0f, mk2 = use ? k2 : 0.0f;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
#pragma unroll
        for (int q = 0; q < 7; ++q) r[q] = fminf(r[q], __shfl_xor(r[q], d, kWave));
        mtr = fmaxf(mtr, __shfl_xor(mtr, d, kWave));
        mk2 = fmaxf(mk2, __shfl_xor(mk2, d, kWave));
    }
    r[7] = mtr;
    if (lane == 0) {
        for (int q = 0; q < 7; ++q) s_r[wv][q] = r[q];
        s_r[wv][7] = mtr;
    }
    __shared__ float s_k2[kBlock / kWave];
    if (lane == 0) s_k2[wv] = mk2;
    __syncthreads();
    if (threadIdx.x == 0) {
        float o[8];
        float k2m = s_k2[0];
        for (int q = 0; q < 8; ++q) o[q] = s_r[0][q];
        for (int w = 1; w < kBlock / kWave; ++w) {
            for (int q = 0; q < 7; ++q) o[q] = fminf(o[q], s_r[w][q]);
            o[7] = fmaxf(o[7], s_r[w][7]);
            k2m = fmaxf(k2m, s_k2[w]);
        }
        blk[3 * blockIdx.x] = make_float4(o[0], o[1], o[2], -o[6]);
        blk[3 * blockIdx.x + 1] = make_float4(-o[3], -o[4], -o[5], o[7]);
        blk[3 * blockIdx.x + 2] = make_float4(k2m, 0.0f, 0.0f, 0.0f);
    }
}

// Cull of a prepared scene: reads 24 bytes per Gaussian and keeps those in
// front of the near plane, above the opacity threshold and whose extent may
// reach a pixel sample.  The extent test is conservative: Sigma'_xx =
// t0^T Sigma t0 <= |t0|^2 trace(Sigma) for the row t0 of T = J R_cam, so
// sqrt(k^2 (|t0|^2 trace + dilation)) (or the 3 sigma radius plus one for the
// square box) bounds the half-width of the box, and a 0.1 % + 3 px margin
// covers rounding.  Everything it drops the exact path would cull too.
// kMulti: the union over the cameras of mo, whose counters it clears.  Each
// workgroup owns a contiguous range of Gaussians and lists its candidates in
// index order at the start of that range (no global atomics).
template <bool kMulti>
__global__ __launch_bounds__(kBlock) void k_cull(DevScene sc, DevPrepared pp, DevCamera cam, DevOptions op, int W,
                                                 int H, uint32_t *__restrict__ cand, uint32_t *__restrict__ seg_count,
                                                 FrameCounters *fc, MultiOut mo) {
    __shared__ uint32_t s_w[kBlock / kWave];
    // the frame's counters start at zero (the preprocess, next on the
    // stream, is their first user)
    static_assert(sizeof(FrameCounters) / 4 <= kBlock, "counters cleared by one workgroup");
    if constexpr (kMulti) {
        if (blockIdx.x == 0 && threadIdx.x < sizeof(FrameCounters) / 4)
            for (int c = 0; c < mo.n; ++c) reinterpret_cast<uint32_t *>(mo.c[c].fc)[threadIdx.x] = 0;
    } else {
        if (blockIdx.x == 0 && threadIdx.x < sizeof(FrameCounters) / 4) reinterpret_cast<uint32_t *>(fc)[threadIdx.x] = 0;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int64_t lo, hi;
    cull_range(sc.P, blockIdx.x, &lo, &hi);
    uint32_t n = 0;     // candidates of this workgroup so far (uniform)
    uint32_t read = 0;  // batches read (uniform)
    // The batch bounds of the workgroup's range are tested first, one batch
    // per thread, into a mask (a batch that the test below would drop
    // entirely is not read); then the kept batches are read in turn.
    __shared__ uint32_t s_skip[kBlock / 32];
    const int64_t b_lo = lo / kBlock, b_hi = (hi + kBlock - 1) / kBlock;
    for (int64_t cb = b_lo; cb < b_hi; cb += kBlock) {
        {
            const int64_t bt = cb + threadIdx.x;
            bool skip = false;
            if (bt < b_hi) {
                const float4 *const bb = pp.blk + 3 * bt;
                const float4 blo = bb[0], bhi = bb[1], bkx = bb[2];
                skip = true;
                if constexpr (kMulti) {
                    for (int c = 0; c < mo.n && skip; ++c)
                        skip = batch_culled(blo, bhi, bkx, mo.c[c].cam, op, mo.c[c].W, mo.c[c].H);
                } else {
                    skip = batch_culled(blo, bhi, bkx, cam, op, W, H);
                }
            }
            const uint64_t bal = __ballot(skip);
            if (lane == 0) {
                s_skip[2 * wave] = (uint32_t)bal;
                s_skip[2 * wave + 1] = (uint32_t)(bal >> 32);
            }
            __syncthreads();
        }
        const int nq = (int)((cb + kBlock < b_hi ? cb + kBlock : b_hi) - cb);
        // the first kept batch of the chunk at or after q (nq if none)
        auto next_kept = [&](int q) {
            while (q < nq) {
                const uint32_t w = ~s_skip[q >> 5] >> (q & 31);
                if (w) return min(q + (int)__builtin_ctz(w), nq);
                q = (q | 31) + 1;
            }
            return nq;
        };
        // member threadIdx.x of kept batch q: its position, opacity and
        // extent terms.  The index is clamped into the range (some member's
        // data past its end or for q = nq, unused): the loads are issued
        // unconditionally, so that nothing waits on a pending one.
        auto load = [&](int q, float4 &p4, float2 &bd) {
            int64_t g = (cb + (q < nq ? q : 0)) * kBlock + threadIdx.x;
            g = g < hi ? g : hi - 1;
            p4 = pp.pos_o[g];
            bd = pp.bnd[g];
        };
        // test and compact kept batch q, members' data p4 and bd
        auto batch = [&](int q, const float4 &p4, const float2 &bd) {
            ++read;
            const int64_t g = (cb + q) * kBlock + threadIdx.x;
            bool keep;
            if constexpr (kMulti) {
                // union of the cameras' candidates: the exact path of each
                // camera culls the rest
                keep = cull_keep(p4, bd, mo.c[0].cam, op, mo.c[0].W, mo.c[0].H);
                for (int c = 1; c < mo.n && !keep; ++c) keep = cull_keep(p4, bd, mo.c[c].cam, op, mo.c[c].W, mo.c[c].H);
            } else {
                keep = cull_keep(p4, bd, cam, op, W, H);
            }
            keep = keep && g < hi;
            // ordered compaction into this workgroup's own segment
            const uint64_t bal = __ballot(keep);
            if (lane == 0) s_w[wave] = (uint32_t)__popcll(bal);
            __syncthreads();
            uint32_t before = 0, tot = 0;
#pragma unroll
            for (int w = 0; w < kBlock / kWave; ++w) {
                before += w < wave ? s_w[w] : 0u;
                tot += s_w[w];
            }
            if (keep) cand[lo + n + before + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull))] = (uint32_t)g;
            n += tot;
            __syncthreads();
        };
        // two buffers in turn: the next kept batch's loads are in flight
        // during this one's test, with no copy between them
        float4 pa, pb;
        float2 ba, bb;
        int q = next_kept(0);
        load(q, pa, ba);
        while (q < nq) {
            int qn = next_kept(q + 1);
            load(qn, pb, bb);
            batch(q, pa, ba);
            q = qn;
            if (q >= nq) break;
            qn = next_kept(q + 1);
            load(qn, pa, ba);
            batch(q, pb, bb);
            q = qn;
        }
        __syncthreads();  // every thread has read the mask before it is replaced
    }
    if (threadIdx.x == 0) {
        seg_count[blockIdx.x] = n;
        seg_count[kCullBlocks + blockIdx.x] = read;
    }
}

// kMulti (with kPrep): every camera of mo in turn over the union candidate
// list, each with its own outputs and counters (the camera and output
// arguments are then unused); the repeated reads of a Gaussian's precompute
// for the second and later cameras follow the first within the same
// wavefront and hit the caches.
//
// The arguments are one struct, read through the kernel-argument pointer,
// which every batch takes anew: held in scalar registers across the batch
// loop, the camera in both precisions and thirty pointers spill to vector
// registers' lanes (280 of them from raw parameters), and those to memory.
struct PreArgs {
    DevScene sc;
    DevPrepared pp;
    DevCamera cam;
    DevCam64 cam64;
    DevOptions op;
    int W, H;
    GaussState *gs;
    float4 *conic;
    uint4 *rect;
    uint32_t *count;
    uint8_t *count8;
    uint4 *erec;
    uint32_t *dkey;
    const uint32_t *cand, *seg_count;
    uint32_t *gmap;
    uint2 *chunks;
    uint32_t chunk_cap;
    FrameCounters *fc;
    uint32_t *gsum_clear;
    int full;
    MultiOut mo;
};
template <bool kPrep, bool kMulti = false, bool kList = false>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_preprocess(PreArgs args_in_place) {
    (void)args_in_place;
    typedef const __attribute__((address_space(4))) PreArgs *ArgPtr;
    const ArgPtr arg_ptr = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const PreArgs &args = *(const PreArgs *)arg_ptr;
    const MultiOut &mo = args.mo;
    const uint32_t *const seg_count = args.seg_count;
    uint32_t *const gsum_clear = args.gsum_clear;
    const int64_t P = args.sc.P;
    static_assert(!kMulti || kPrep, "a batch walks a union candidate list");
    static_assert(!kList || !kPrep, "a list of raw Gaussians");
    // the first depth pass's group sums start at zero
    if constexpr (kMulti) {
        for (int c = 0; c < mo.n; ++c)
            for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < (uint32_t)kGsumWords; i += gridDim.x * kBlock)
                mo.c[c].gsum_clear[i] = 0;
    } else {
        for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < (uint32_t)kGsumWords; i += gridDim.x * kBlock)
            gsum_clear[i] = 0;
    }
    // Persistent grid: each workgroup walks batches of 256 Gaussians.  Every
    // wavefront keeps its own visible count and pending chunk reservations
    // (LDS), so the batch loop has no workgroup barrier and global atomics
    // are per wavefront flush, not per batch.
    constexpr int kWaveBig = kBigList / (kBlock / kWave);  // pending large Gaussians per wavefront
    __shared__ uint32_t s_bg[kBlock / kWave][kWaveBig], s_boff[kBlock / kWave][kWaveBig],
        s_bn[kBlock / kWave][kWaveBig], s_bx[kBlock / kWave][kWaveBig], s_by[kBlock / kWave][kWaveBig];
    __shared__ uint32_t s_excl[kBlock / kWave][kWave], s_mlo[kBlock / kWave][kWave], s_mhi[kBlock / kWave][kWave];
    const int wv = threadIdx.x / kWave;  // this lane's wavefront
    uint32_t w_nbig = 0, w_nch = 0;      // wave-uniform: pending entries and their chunks
    // visible Gaussians, small-rectangle hits and super-tile entries so far (per
    // camera; in LDS: the kernel has no register to spare)
    __shared__ uint32_t s_vis[kBlock / kWave][kMulti ? kMaxCams : 1];
    __shared__ uint32_t s_pairs[kBlock / kWave][kMulti ? kMaxCams : 1];
    __shared__ uint32_t s_ents[kBlock / kWave][kMulti ? kMaxCams : 1];
    // kMulti: the pending list holds entries of every camera, each tagged
    // with its camera; chunks are counted per camera, and a flush reserves
    // each camera's share of its own chunk list
    constexpr int kMB = kMulti ? kWaveBig : 1;
    constexpr int kMC = kMulti ? kMaxCams : 1;
    __shared__ uint32_t s_bc[kBlock / kWave][kMB], s_nch[kBlock / kWave][kMC], s_cbase[kBlock / kWave][kMC];
    __shared__ uint2 *s_chunks[kMC];
    __shared__ uint4 *s_erec[kMC];
    if ((threadIdx.x & (kWave - 1)) == 0)
        for (int c = 0; c < (kMulti ? kMaxCams : 1); ++c) {
            s_vis[wv][c] = 0;
            s_pairs[wv][c] = 0;
            s_ents[wv][c] = 0;
            s_nch[wv][c] = 0;
        }
    if constexpr (kMulti) {
        if (threadIdx.x == 0)
            for (int c = 0; c < mo.n; ++c) {
                s_chunks[c] = mo.c[c].chunks;
                s_erec[c] = mo.c[c].erec;
            }
        __syncthreads();
    }

    // reserve chunk-list space for the wavefront's pending large Gaussians
    // and write their entries (g, first chunk); on overflow only flag it
    // (the host resizes the list and renders the frame again)
    auto flush_big = [&](int ln, FrameCounters *fc, uint2 *__restrict__ chunks, uint32_t chunk_cap,
                         uint4 *__restrict__ erec) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint32_t base = 0;
        if (ln == 0) base = atomicAdd(&fc->nchunks, w_nch);
        base = (uint32_t)__shfl((int)base, 0, kWave);
        const bool ok = (uint64_t)base + w_nch <= chunk_cap;
        if (!ok && ln == 0) atomicOr(&fc->error, kErrChunkOverflow);
        for (uint32_t e = (uint32_t)ln; e < w_nbig; e += kWave) {
            const uint32_t gg = s_bg[wv][e], first = base + s_boff[wv][e], n = s_bn[wv][e];
            if (ok)
                for (uint32_t c = 0; c < n; ++c) chunks[first + c] = make_uint2(gg, first);
            // (on overflow the record still marks the rectangle as chunked, so
            // that the emission of this frame reads no record of an earlier one)
            erec[gg] = make_uint4(s_bx[wv][e], s_by[wv][e], 0u, ok ? first : 0u);
        }
        // every lane has read the list before it is refilled
        __builtin_amdgcn_wave_barrier();
        w_nbig = 0;
        w_nch = 0;
    };
    constexpr uint32_t kNoBase = 0xffffffffu;
    auto flush_big_multi = [&](int ln) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (ln == 0)
            for (int c = 0; c < mo.n; ++c) {
                const uint32_t n = s_nch[wv][c];
                uint32_t base = kNoBase;
                if (n) {
                    base = atomicAdd(&mo.c[c].fc->nchunks, n);
                    if ((uint64_t)base + n > mo.c[c].chunk_cap) {
                        atomicOr(&mo.c[c].fc->error, kErrChunkOverflow);
                        base = kNoBase;
                    }
                }
                s_cbase[wv][c] = base;
                s_nch[wv][c] = 0;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t e = (uint32_t)ln; e < w_nbig; e += kWave) {
            const uint32_t c = s_bc[wv][e], base = s_cbase[wv][c];
            const uint32_t gg = s_bg[wv][e];
            if (base == kNoBase) {
                // overflow: still mark the rectangle as chunked (no stale record)
                s_erec[c][gg] = make_uint4(s_bx[wv][e], s_by[wv][e], 0u, 0u);
                continue;
            }
            const uint32_t first = base + s_boff[wv][e], n = s_bn[wv][e];
            uint2 *const ck = s_chunks[c];
            for (uint32_t k = 0; k < n; ++k) ck[first + k] = make_uint2(gg, first);
            s_erec[c][gg] = make_uint4(s_bx[wv][e], s_by[wv][e], 0u, first);
        }
        __builtin_amdgcn_wave_barrier();
        w_nbig = 0;
    };

    const int lane = threadIdx.x & (kWave - 1);
    // A prepared scene walks the cull's candidates as one list: the exclusive
    // prefix of the segment counts maps a list position to its segment, and
    // workgroups take 256-position batches in turn, so every workgroup gets
    // the same share whatever the segment sizes.  g = sc.P marks an idle lane.
    static_assert((kCullBlocks & (kCullBlocks - 1)) == 0 && kCullBlocks % kBlock == 0, "segment prefix layout");
    __shared__ uint32_t s_pref[kPrep ? kCullBlocks : 1];
    __shared__ uint32_t s_wtot[kBlock / kWave];
    uint32_t ncand = 0;
    if constexpr (kPrep) {
        constexpr int kPer = kCullBlocks / kBlock;
        uint32_t c[kPer], sum = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            c[j] = seg_count[threadIdx.x * kPer + j];
            sum += c[j];
        }
        const int wave = threadIdx.x / kWave;
        const uint32_t incl = wave_incl_scan(sum, lane);
        if (lane == kWave - 1) s_wtot[wave] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (int w = 0; w < kBlock / kWave; ++w) {
            if (w < wave) run += s_wtot[w];
            ncand += s_wtot[w];
        }
        ncand = (uint32_t)__builtin_amdgcn_readfirstlane((int)ncand);  // (the same in every lane)
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            s_pref[threadIdx.x * kPer + j] = run;
            run += c[j];
        }
        __syncthreads();
    }
    if constexpr (kPrep) {
        // the batches the cull read (its workgroups' counts), for the stats
        if (blockIdx.x == 0) {
            constexpr int kPer = kCullBlocks / kBlock;
            uint32_t r = 0;
#pragma unroll
            for (int j = 0; j < kPer; ++j) r += seg_count[kCullBlocks + threadIdx.x * kPer + j];
            const uint32_t incl = wave_incl_scan(r, lane);
            __syncthreads();  // s_wtot is free again
            if (lane == kWave - 1) s_wtot[threadIdx.x / kWave] = incl;
            __syncthreads();
            if (threadIdx.x == 0) {
                uint32_t tot = 0;
                for (int w = 0; w < kBlock / kWave; ++w) tot += s_wtot[w];
                if constexpr (kMulti) {
                    for (int c = 0; c < mo.n; ++c) {
                        mo.c[c].fc->ncand = ncand;
                        mo.c[c].fc->cull_read = tot;
                    }
                } else {
                    args.fc->ncand = ncand;
                    args.fc->cull_read = tot;
                }
            }
        }
    }
    // Raw parameters (kList): a wavefront takes a contiguous range of Gaussians,
    // drops those that are certainly not visible before the projection (raw_keep)
    // and projects the others up to 64 at a time, from a ring of two wavefronts'
    // Gaussians and their parameters in LDS.  Its outputs are packed: the range's
    // output slots from the first on, in the Gaussians' order (so equal depths
    // keep it), the rest marked invalid.
    // Bound by HBM: 10M Gaussians of degree 3, 29 % visible, in 4K: 608 us for
    // 2.4 GB read (nearly every line of every plane holds a visible Gaussian's
    // element) and 0.25 GB written.  One pass over all Gaussians took 754: every
    // wavefront ran the whole projection, and 48-byte records 29 % apart were
    // written as partial lines.  (With a group's survivors split over two
    // projections, whose lines are then read twice, it was slower than one pass.)
    constexpr uint32_t kRing = 2 * kWave;
    constexpr int kTerms = sizeof(RawTerms) / sizeof(float);
    __shared__ uint32_t s_rg[kList ? kBlock / kWave : 1][kList ? kRing : 1];
    __shared__ float s_rt[kList ? kBlock / kWave : 1][kList ? kTerms : 1][kList ? kRing : 1];
    uint32_t n_queue = 0, n_whole = 0, q_head = 0;  // wave-uniform
    uint32_t grp = 0, grp_end = 0, slot = 0;  // wave-uniform: groups left, next output slot
    if constexpr (!kPrep) {
        const uint64_t groups = (uint64_t)((P + kWave - 1) / kWave), nw = (uint64_t)gridDim.x * (kBlock / kWave);
        const uint64_t w = (uint64_t)blockIdx.x * (kBlock / kWave) + (uint32_t)__builtin_amdgcn_readfirstlane(wv);
        grp = (uint32_t)(groups * w / nw);
        grp_end = (uint32_t)(groups * (w + 1) / nw);
        slot = grp * (uint32_t)kWave;
    }
    RawTerms rt = {};
    // outputs of a prepared scene go to the candidate's list position (dense,
    // contiguous per wavefront)
    int64_t batch = blockIdx.x;  // prepared: batch of 256 list positions
    for (;;) {
    ArgPtr batch_ptr = arg_ptr;
    asm volatile("" : "+s"(batch_ptr));
    const PreArgs &ba = *(const PreArgs *)batch_ptr;
    const DevScene &sc = ba.sc;
    const DevPrepared &pp = ba.pp;
    const DevOptions &op = ba.op;
    const bool full = !kList && ba.full != 0;
    // (Gaussian indices are below 2^31; P32: an idle lane)
    const uint32_t P32 = (uint32_t)P;
    uint32_t g = P32;
    uint32_t ii = 0;  // output slot (prepared: position in the candidate list)
    if constexpr (kPrep) {
        if ((uint64_t)batch * kBlock >= ncand) break;
        ii = (uint32_t)batch * kBlock + threadIdx.x;
        if (ii < ncand) {
            // last segment whose prefix is <= ii: it holds position ii
            uint32_t sg = 0;
#pragma unroll
            for (uint32_t step = kCullBlocks / 2; step > 0; step >>= 1)
                if (s_pref[sg + step] <= ii) sg += step;
            int64_t lo, hi;
            cull_range(P, sg, &lo, &hi);
            g = ba.cand[lo + (ii - s_pref[sg])];
        }
        batch += gridDim.x;
    } else if constexpr (kList) {
        while (n_queue < (uint32_t)kWave && grp < grp_end) {
            const int64_t gi = (int64_t)grp * kWave + lane;
            const bool in = gi < P;
            const RawTerms t = raw_terms(sc, in ? gi : P - 1);
            const bool keep = in && raw_keep(t, ba.cam, op, ba.W, ba.H);
            const uint64_t km = __ballot(keep);
            if (keep) {
                const uint32_t at = (__builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)km, n_queue)) +
                                     q_head) % kRing;
                s_rg[wv][at] = (uint32_t)gi;
                const float *f = reinterpret_cast<const float *>(&t);
#pragma unroll
                for (int j = 0; j < kTerms; ++j) s_rt[wv][j][at] = f[j];
            }
            n_whole = n_queue;
            n_queue += (uint32_t)__popcll(km);
            ++grp;
        }
        if (n_queue == 0) break;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // whole groups only: a group's survivors share the lines of every
        // coefficient plane
        const uint32_t take = n_queue <= (uint32_t)kWave ? n_queue : n_whole;
        {
            const uint32_t at = (q_head + (uint32_t)lane) % kRing;
            if ((uint32_t)lane < take) g = s_rg[wv][at];
            float *f = reinterpret_cast<float *>(&rt);
#pragma unroll
            for (int j = 0; j < kTerms; ++j) f[j] = s_rt[wv][j][at];
        }
        q_head = (q_head + take) % kRing;
        n_queue -= take;
        ii = slot + (uint32_t)lane;
        slot += take;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        if (grp >= grp_end) break;
        const int64_t i = (int64_t)grp * kWave + lane;
        if (i < P) {
            g = (uint32_t)i;
            rt = raw_terms(sc, g);
        }
        ii = (uint32_t)i;
        ++grp;
        slot = grp * (uint32_t)kWave;
    }
    const int ncams = kMulti ? ba.mo.n : 1;
    for (int ci = 0; ci < ncams; ++ci) {
    // this camera, its image size and its outputs
    const DevCamera &cm = kMulti ? ba.mo.c[ci].cam : ba.cam;
    const int W = kMulti ? ba.mo.c[ci].W : ba.W, H = kMulti ? ba.mo.c[ci].H : ba.H;
    const DevCam64 &cm64 = kMulti ? ba.mo.c[ci].cam64 : ba.cam64;
    GaussState *__restrict__ const gs_c = kMulti ? ba.mo.c[ci].gs : ba.gs;
    float4 *__restrict__ const conic_c = kMulti ? ba.mo.c[ci].conic : ba.conic;
    uint4 *__restrict__ const rect_c = kMulti ? ba.mo.c[ci].rect : ba.rect;
    uint32_t *__restrict__ const count_c = kMulti ? ba.mo.c[ci].count : ba.count;
    uint8_t *__restrict__ const count8_c = kMulti ? ba.mo.c[ci].count8 : ba.count8;
    uint4 *__restrict__ const erec_c = kMulti ? ba.mo.c[ci].erec : ba.erec;
    uint32_t *__restrict__ const dkey_c = kMulti ? ba.mo.c[ci].dkey : ba.dkey;
    const int64_t st = sc.stride;
    bool valid = false;
    float u = 0, v = 0, A = 0, B = 0, C = 0, k2 = 0, o = 0, tz = 0, l2o = 0;
    float Ab = 0, Bb = 0, Cb = 0;  // the blend's conic (see GaussState)
    int tx0 = 0, tx1 = -1, ty0 = 0, ty1 = -1;
    float col[3] = {0, 0, 0};

    if (g < P32) {
        float mx, my, mz, po = 0.0f;
        if constexpr (kPrep) {
            const float4 p4 = pp.pos_o[g];
            mx = p4.x;
            my = p4.y;
            mz = p4.z;
            po = p4.w;
        } else {
            mx = rt.x;
            my = rt.y;
            mz = rt.z;
        }
        const float *R = cm.R;
        // view transform (p_view)
        const float tx = ((R[0] * mx + R[1] * my) + R[2] * mz) + cm.t[0];
        const float ty = ((R[3] * mx + R[4] * my) + R[5] * mz) + cm.t[1];
        tz = ((R[6] * mx + R[7] * my) + R[8] * mz) + cm.t[2];
        // near plane (Alg. 4: p_view.z > 0.2); the remaining attributes are
        // read only for Gaussians in front of the camera
        if (tz > cm.near_z && isfinite(mx) && isfinite(my) && isfinite(mz)) {
            bool ok = false;
            float S[6] = {0, 0, 0, 0, 0, 0}, s3[3] = {0, 0, 0}, qu[4] = {0, 0, 0, 0};
            float log2o = 0.0f;
            if constexpr (kPrep) {
                // view-independent part precomputed once (Sec. 5.3.1); an
                // invalid Gaussian has opacity 0
                o = po;
                ok = o > op.alpha_min;
                if (ok) {
                    const float4 c0 = pp.cov[2 * (int64_t)g], c1 = pp.cov[2 * (int64_t)g + 1];
                    s3[0] = c0.x; s3[1] = c0.y; s3[2] = c0.z;
                    k2 = c0.w;
                    qu[0] = c1.x; qu[1] = c1.y; qu[2] = c1.z; qu[3] = c1.w;
                }
            } else {
                const float logit = rt.logit;
                o = (float)(1.0 / (1.0 + canon_exp(-(double)logit)));
                // opacity prefilter (Alg. 4: opacity > 1/255)
                if (o > op.alpha_min && isfinite(logit)) {
                    const float q4[4] = {rt.qw, rt.qx, rt.qy, rt.qz};
                    ok = scale_rot(rt.ls0, rt.ls1, rt.ls2, q4, s3, qu);
                    if (ok) k2 = extent_k2(o, op);
                }
            }
            if (ok) {
                sigma3(s3, qu, S);
                log2o = log2f(o);
                // the blend's conic (binary64, rounded once)
                const bool have_b64 = conic_b64(s3, qu, mx, my, mz, cm64, (double)op.dilation, &Ab, &Bb, &Cb);
                const float S00 = S[0], S01 = S[1], S02 = S[2], S11 = S[3], S12 = S[4], S22 = S[5];
                {
                    // pinhole projection (project + ndc2Pix)
                    const float xt = tx / tz, yt = ty / tz;
                    u = cm.fx * xt + cm.cx;
                    v = cm.fy * yt + cm.cy;
                    // EWA Jacobian with the view-direction clamp
                    const float limx = op.jac_clip * ((0.5f * (float)W) / cm.fx);
                    const float limy = op.jac_clip * ((0.5f * (float)H) / cm.fy);
                    const float xc = clampf_(xt, -limx, limx);
                    const float yc = clampf_(yt, -limy, limy);
                    const float J00 = cm.fx / tz, J02 = -((cm.fx * xc) / tz);
                    const float J11 = cm.fy / tz, J12 = -((cm.fy * yc) / tz);
                    // 2D covariance Sigma' = T Sigma T^T, T = J R_cam
                    const float T00 = J00 * R[0] + J02 * R[6], T01 = J00 * R[1] + J02 * R[7],
                                T02 = J00 * R[2] + J02 * R[8];
                    const float T10 = J11 * R[3] + J12 * R[6], T11 = J11 * R[4] + J12 * R[7],
                                T12 = J11 * R[5] + J12 * R[8];
                    const float U00 = (T00 * S00 + T01 * S01) + T02 * S02;
                    const float U01 = (T00 * S01 + T01 * S11) + T02 * S12;
                    const float U02 = (T00 * S02 + T01 * S12) + T02 * S22;
                    const float U10 = (T10 * S00 + T11 * S01) + T12 * S02;
                    const float U11 = (T10 * S01 + T11 * S11) + T12 * S12;
                    const float U12 = (T10 * S02 + T11 * S12) + T12 * S22;
                    const float ca = ((U00 * T00 + U01 * T01) + U02 * T02) + op.dilation;
                    const float cb = (U00 * T10 + U01 * T11) + U02 * T12;
                    const float cc = ((U10 * T10 + U11 * T11) + U12 * T12) + op.dilation;
                    const float det = ca * cc - cb * cb;
                    if (det > 0.0f) {
                        A = cc / det;
                        B = (-cb) / det;
                        C = ca / det;
                        // the blend's conic: the binary32 one if the binary64
                        // determinant was not positive
                        if (!have_b64) {
                            Ab = A;
                            Bb = B;
                            Cb = C;
                        }
                        // rectangle tangent to the ellipse (Sec. 4.1), in pixel samples;
                        // binning 2: the square of the 3 sigma circle of 3DGS
                        // (Alg. 1: radius ceil(3 sqrt(lambda_max)) of Sigma')
                        float hx, hy;
                        if (op.binning == 2) {
                            const float mid = 0.5f * (ca + cc);
                            float disc = mid * mid - det;
                            disc = disc > 0.0f ? disc : 0.0f;
                            const float lam = mid + sqrtf(disc);
                            hx = ceilf(3.0f * sqrtf(lam));
                            hy = hx;
                        } else {
                            hx = sqrtf(k2 * ca);
                            hy = sqrtf(k2 * cc);
                        }
                        const float xlo = clampf_((u - hx) - 0.5f, -1.0f, (float)W);
                        const float xhi = clampf_((u + hx) - 0.5f, -1.0f, (float)W);
                        const float ylo = clampf_((v - hy) - 0.5f, -1.0f, (float)H);
                        const float yhi = clampf_((v + hy) - 0.5f, -1.0f, (float)H);
                        int i0 = (int)ceilf(xlo), i1 = (int)floorf(xhi);
                        int j0 = (int)ceilf(ylo), j1 = (int)floorf(yhi);
                        i0 = i0 < 0 ? 0 : i0;
                        j0 = j0 < 0 ? 0 : j0;
                        i1 = i1 > W - 1 ? W - 1 : i1;
                        j1 = j1 > H - 1 ? H - 1 : j1;
                        if (i0 <= i1 && j0 <= j1) {
                            tx0 = i0 / kTile;
                            tx1 = i1 / kTile;
                            ty0 = j0 / kTile;
                            ty1 = j1 / kTile;
                            // SH colour for surviving Gaussians only (Alg. 4)
                            const float dxw = mx - cm.eye[0], dyw = my - cm.eye[1], dzw = mz - cm.eye[2];
                            const float dn = sqrtf((dxw * dxw + dyw * dyw) + dzw * dzw);
                            float Y[16];
                            sh_basis(dxw / dn, dyw / dn, dzw / dn, sc.D, Y);
                            const int nk = (sc.D + 1) * (sc.D + 1);
                            float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
                            // every coefficient load is issued before the first
                            // use (one memory round trip, not one per coefficient),
                            // a degree's loads behind one branch: with a branch per
                            // load, and two registers spilled whose reload stood
                            // between them, the 4K frame's kernel took 280 us, now
                            // 250, the 1M Gaussians' 98 and 85, and 10,000 raw
                            // ones' 11.9 and 10.6
                            float shv[48];
                            if constexpr (kPrep) {
                                // Gaussian-major coefficients: one contiguous read
                                const float4 *shg = reinterpret_cast<const float4 *>(pp.sh + (int64_t)g * pp.sh_stride);
                                auto read_sh = [&](int j0, int j1) {
#pragma unroll
                                    for (int j = j0; j < j1; ++j) {
                                        const float4 q4 = shg[j];
                                        shv[4 * j] = q4.x;
                                        shv[4 * j + 1] = q4.y;
                                        shv[4 * j + 2] = q4.z;
                                        shv[4 * j + 3] = q4.w;
                                    }
                                };
                                // (1, 4, 9 or 16 coefficients of 3 channels, padded to 4 floats)
#pragma unroll
                                for (int j = 4; j < 48; ++j) shv[j] = 0.0f;
                                read_sh(0, 1);
                                if (sc.D >= 1) read_sh(1, 3);
                                if (sc.D >= 2) read_sh(3, 7);
                                if (sc.D >= 3) read_sh(7, 12);
                            } else {
                                const float *shp = sc.sh + g;
                                auto read_sh = [&](int j0, int j1) {
#pragma unroll
                                    for (int j = j0; j < j1; ++j, shp += st) shv[j] = *shp;
                                };
#pragma unroll
                                for (int j = 3; j < 48; ++j) shv[j] = 0.0f;
                                read_sh(0, 3);
                                if (sc.D >= 1) read_sh(3, 12);
                                if (sc.D >= 2) read_sh(12, 27);
                                if (sc.D >= 3) read_sh(27, 48);
                            }
#pragma unroll
                            for (int k = 0; k < 16; ++k) {
                                if (k < nk) {
                                    a0 = a0 + shv[3 * k + 0] * Y[k];
                                    a1 = a1 + shv[3 * k + 1] * Y[k];
                                    a2 = a2 + shv[3 * k + 2] * Y[k];
                                }
                            }
                            a0 = a0 + 0.5f;
                            a1 = a1 + 0.5f;
                            a2 = a2 + 0.5f;
                            // non-finite SH inputs cull the Gaussian
                            valid = isfinite(a0) && isfinite(a1) && isfinite(a2);
                            col[0] = a0 > 0.0f ? a0 : 0.0f;
                            col[1] = a1 > 0.0f ? a1 : 0.0f;
                            col[2] = a2 > 0.0f ? a2 : 0.0f;
                            l2o = log2o;
                        }
                    }
                }
            }
        }
    }

    // ---- exact tile count (Alg. 3 over the rectangle) -------------------------
    const int ntx = tx1 - tx0 + 1, nty = ty1 - ty0 + 1;
    const int nt = valid ? ntx * nty : 0;
    uint32_t cnt = 0;
    uint64_t hm = 0;
    // rectangles of more than kBigTiles tiles go to the chunk list, where
    // wavefronts across the GPU test them kChunkTiles tiles at a time
    const bool chunked = valid && nt > kBigTiles;
    {
        const uint64_t bm = __ballot(chunked);
        if (bm) {  // uniform
            const uint32_t nch = chunked ? (uint32_t)((nt + kChunkTiles - 1) / kChunkTiles) : 0u;
            const uint32_t incl = wave_incl_scan(nch, lane);
            // chunks pending before these (this camera's, kMulti)
            uint32_t cbase = w_nch;
            if constexpr (kMulti) cbase = s_nch[wv][ci];
            if (chunked) {
                const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)bm, w_nbig));
                if constexpr (kMulti) s_bc[wv][at] = (uint32_t)ci;
                s_bg[wv][at] = ii;
                s_bn[wv][at] = nch;
                s_bx[wv][at] = (uint32_t)tx0 | ((uint32_t)tx1 << 16);
                s_by[wv][at] = (uint32_t)ty0 | ((uint32_t)ty1 << 16);
                s_boff[wv][at] = cbase + incl - nch;
            }
            w_nbig += (uint32_t)__popcll(bm);
            const uint32_t tot = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
            if constexpr (kMulti) {
                if (lane == 0) s_nch[wv][ci] = cbase + tot;
            } else {
                w_nch += tot;
            }
        }
    }
    const bool small = valid && !chunked;  // rectangle of at most kBigTiles tiles
    if (op.binning != 0) {
        // every tile of the rectangle (test and comparison modes)
        if (small) {
            cnt = (uint32_t)nt;
            hm = nt >= 64 ? ~0ull : ((1ull << nt) - 1ull);
        }
    } else {
        // The wavefront flattens its (Gaussian, rectangle tile) items so that
        // every lane tests one tile per step whatever the mix of rectangle
        // sizes (Sec. 5.1.2 size-aware scheduling, balanced across wave64).
        const int wave = threadIdx.x / kWave;
        uint32_t *sx = s_excl[wave];
        const uint32_t items = small ? (uint32_t)nt : 0u;
        const uint32_t incl = wave_incl_scan(items, lane);
        const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
        sx[lane] = incl - items;
        s_mlo[wave][lane] = 0u;
        s_mhi[wave][lane] = 0u;
        // (the wavefront's Gaussians are all finite but for adversarial input)
        const bool finite = __ballot(small && !tile_terms_finite(u, v, A, B, C)) == 0;
        for (uint32_t b0 = 0; b0 < total; b0 += kWave) {
            const uint32_t item = b0 + (uint32_t)lane;
            const int L = owner_lane(sx, item < total ? item : total - 1u);
            const uint32_t k = item - sx[L];
            const float su = __shfl(u, L, kWave), sv = __shfl(v, L, kWave), sA = __shfl(A, L, kWave),
                        sB = __shfl(B, L, kWave), sC = __shfl(C, L, kWave), sk2 = __shfl(k2, L, kWave);
            const int stx0 = __shfl(tx0, L, kWave), sty0 = __shfl(ty0, L, kWave), sntx = __shfl(ntx, L, kWave);
            if (item < total) {
                const int ry = small_div(k, sntx), rx = (int)k - ry * sntx;
                if (finite ? tile_hit<true>(su, sv, sA, sB, sC, sk2, stx0 + rx, sty0 + ry, W, H)
                           : tile_hit<false>(su, sv, sA, sB, sC, sk2, stx0 + rx, sty0 + ry, W, H))
                    atomicOr(k < 32u ? &s_mlo[wave][L] : &s_mhi[wave][L], 1u << (k & 31u));
            }
        }
        hm = (uint64_t)s_mlo[wave][lane] | ((uint64_t)s_mhi[wave][lane] << 32);
        cnt = (uint32_t)__popcll(hm);
    }

    // entries: the overlapped super-tiles (at most 10 for a rectangle of at
    // most kBigTiles tiles)
    const uint32_t ents = valid ? super_span(tx0, tx1, ty0, ty1) : 0u;
    if (g < P32) {
        const uint32_t key = valid ? __float_as_uint(tz) : kInvalidKey;
        const int64_t oi = (int64_t)ii;
        if constexpr (kPrep) {
            // the Gaussian of this list position, in the caller's indexing
            uint32_t *const gmap_c = kMulti ? ba.mo.c[ci].gmap : ba.gmap;
            gmap_c[ii] = pp.orig[g];
        }
        dkey_c[oi] = key;
        count8_c[oi] = chunked ? kCount8Big : (uint8_t)ents;
        // the 4-byte count: a chunked rectangle's starts at 0 (k_big_count
        // adds its hits); the others are read from count8
        if (full || chunked) count_c[oi] = valid ? cnt : 0u;
        if (valid) {
            GaussState s;
            s.f0 = make_float4(u, v, Ab, Bb);
            s.f1 = make_float4(Cb, k2, l2o, col[0]);
            s.f2 = make_float4(col[1], col[2], tz, o);
            gs_c[oi] = s;
            // the canonical conic: the large rectangles' tile tests read it
            if (full || chunked) conic_c[oi] = make_float4(A, B, C, 0.0f);
            if (full) rect_c[oi] = make_uint4((uint32_t)tx0, (uint32_t)tx1, (uint32_t)ty0, (uint32_t)ty1);
            // emission record: rectangle (4 x 16 bits) and hit mask in one
            // 16-byte gather (a chunked one's is written at its flush)
            if (!chunked)
                erec_c[oi] = make_uint4((uint32_t)tx0 | ((uint32_t)tx1 << 16), (uint32_t)ty0 | ((uint32_t)ty1 << 16),
                                      (uint32_t)hm, (uint32_t)(hm >> 32));
        } else if (kPrep && full) {
            // a list slot is reused every frame: clear a culled candidate's
            // introspected state
            gs_c[oi] = GaussState{};
            conic_c[oi] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            rect_c[oi] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    {
        const uint32_t nv = (uint32_t)__popcll(__ballot(valid));
        uint32_t np = small ? cnt : 0u, ne = ents;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            np += (uint32_t)__shfl_xor((int)np, d, kWave);
            ne += (uint32_t)__shfl_xor((int)ne, d, kWave);
        }
        if (lane == 0) {
            s_vis[wv][ci] += nv;
            s_pairs[wv][ci] += np;
            s_ents[wv][ci] += ne;
        }
        if (w_nbig > (uint32_t)(kWaveBig - kWave)) {  // room for the next batch (or camera)
            if constexpr (kMulti)
                flush_big_multi(lane);
            else
                flush_big(lane, args.fc, args.chunks, args.chunk_cap, args.erec);
        }
    }
    }  // camera loop
    }  // batch loop
    if constexpr (kList) {
        // the range's slots without a projected Gaussian
        const int64_t end = (int64_t)grp_end * kWave < P ? (int64_t)grp_end * kWave : P;
        for (int64_t i = (int64_t)slot + lane; i < end; i += kWave) args.dkey[i] = kInvalidKey;
    }
    // The workgroup's visible and pair counts (of each camera) in one 64-bit
    // atomic: atomics on one line take about 8 ns each, one after the other,
    // and the wavefronts of a frame all end at about the same time.  With two
    // per wavefront the kernel took 87 us for 200k Gaussians (27 now), 162 for
    // 1M (98 with this alone, 85 now) and 344 for the 3M candidates of the 10M
    // city (275, 250 now).
    static_assert(offsetof(FrameCounters, pairs) == offsetof(FrameCounters, visible) + 4 &&
                      offsetof(FrameCounters, visible) % 8 == 0,
                  "one 64-bit counter");
    auto add_counts = [&](FrameCounters *f, int c) {
        uint32_t vis = 0, prs = 0, ents = 0;
        for (int w = 0; w < kBlock / kWave; ++w) {
            vis += s_vis[w][c];
            prs += s_pairs[w][c];
            ents += s_ents[w][c];
        }
        if (vis | prs)
            atomicAdd(reinterpret_cast<unsigned long long *>(&f->visible),
                      (unsigned long long)vis | ((unsigned long long)prs << 32));
        if (ents) atomicAdd(&f->entries, ents);
    };
    if (w_nbig) {
        if constexpr (kMulti)
            flush_big_multi(lane);
        else
            flush_big(lane, args.fc, args.chunks, args.chunk_cap, args.erec);
    }
    __syncthreads();
    if constexpr (kMulti) {
        if ((int)threadIdx.x < mo.n) add_counts(mo.c[threadIdx.x].fc, (int)threadIdx.x);
    } else {
        if (threadIdx.x == 0) add_counts(args.fc, 0);
    }
}

// Hit mask of a small rectangle (bit rx + ntx ry of its emission record)
// restricted to super-tile (sx, sy), in the super-tile's own layout (bit
// lx + kSuper ly): the rectangle's rows in the super-tile, each cut to the
// super-tile's columns and moved to its place.
__device__ __forceinline__ uint64_t super_mask(uint64_t hm, int tx0, int ty0, int ntx, int nty, int sx, int sy) {
    const int xs = sx * kSuper, ys = sy * kSuper;
    const int a = xs - tx0 > 0 ? xs - tx0 : 0, b = xs + kSuper - tx0 < ntx ? xs + kSuper - tx0 : ntx;
    const int c = ys - ty0 > 0 ? ys - ty0 : 0, d = ys + kSuper - ty0 < nty ? ys + kSuper - ty0 : nty;
    const uint64_t wm = (1ull << (b - a)) - 1ull;  // b - a <= kSuper
    const int lx0 = tx0 + a - xs;
    uint64_t m = 0;
    for (int ry = c; ry < d; ++ry)
        m |= ((hm >> (ry * ntx + a)) & wm) << ((ty0 + ry - ys) * kSuper + lx0);
    return m;
}

// Key emission at super-tile granularity (Alg. 2 with the offsets of a
// prefix scan, the pair (tile, Gaussian) replaced by (super-tile, Gaussian,
// hit mask); the tile test is reused from the preprocess through the hit
// mask).  The visible Gaussians are taken 64 at a time in (depth, index)
// order; the wavefront flattens the small rectangles' entries so that every
// lane builds one entry per step, written at its Gaussian's scanned offset
// plus its index among the Gaussian's entries (row-major over the
// overlapped super-tiles).  A chunked Gaussian only leaves (its output slot,
// its offset) at its first chunk's slot of `big` for k_big_entries.
__global__ __launch_bounds__(kBlock) void k_super_emit(int W, const uint32_t *__restrict__ order, uint32_t visible,
                                                       const uint32_t *__restrict__ visible_dev,
                                                       const uint32_t *__restrict__ offsets,
                                                       const uint4 *__restrict__ erec, uint2 *__restrict__ big,
                                                       uint32_t chunk_cap, uint16_t *__restrict__ skey,
                                                       uint32_t *__restrict__ gidx, uint64_t *__restrict__ smask,
                                                       uint32_t ecap, uint2 *__restrict__ sranges, uint32_t nsuper,
                                                       uint32_t *__restrict__ gsum_clear,
                                                       const FrameCounters *__restrict__ fc) {
    __shared__ uint32_t s_excl[kBlock / kWave][kWave];
    // an overflowed chunk list left the large rectangles untested: their
    // entries (k_big_entries writes them otherwise) are filled here with
    // super-tile 0, the Gaussian and an empty mask, so that the second half
    // of this frame, which the host discards and renders again, reads only
    // entries it wrote (every list value a valid Gaussian)
    const bool overflow = (fc->error & kErrChunkOverflow) != 0;
    // every super-tile's range starts empty, (0xffffffff, 0), for the last
    // sort pass to narrow (sranges NULL: no pass records them)
    if (sranges)
        for (uint32_t t = blockIdx.x * kBlock + threadIdx.x; t < nsuper; t += gridDim.x * kBlock)
            sranges[t] = make_uint2(0xffffffffu, 0u);
    // and the first sort pass's group sums start at zero
    if (gsum_clear)
        for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < (uint32_t)kGsumWords; i += gridDim.x * kBlock)
            gsum_clear[i] = 0;
    // the visible count comes from the device when the launch is sized by a
    // bound (graph-captured frames); it never exceeds the bound
    if (visible_dev) visible = min(visible, *visible_dev);
    const int tiles_x = (W + kTile - 1) / kTile;
    const uint32_t stx = (uint32_t)((tiles_x + kSuper - 1) >> kSuperShift);
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t *sx = s_excl[threadIdx.x / kWave];
    for (uint32_t r0 = blockIdx.x * kBlock; r0 < visible; r0 += gridDim.x * kBlock) {
        const uint32_t r = r0 + threadIdx.x;
        const bool act = r < visible;
        uint32_t g = 0, base = 0;
        uint4 er = make_uint4(0u, 0u, 0u, 0u);
        if (act) {
            g = order[r];
            base = offsets[r];
            er = erec[g];
        }
        const uint4 rc = unpack_rect(er);
        const int tx0 = (int)rc.x, ty0 = (int)rc.z;
        const int ntx = (int)rc.y - tx0 + 1, nty = (int)rc.w - ty0 + 1;
        const bool chunked = act && ntx * nty > kBigTiles;
        if (chunked && er.w < chunk_cap) big[er.w] = make_uint2(g, base);
        if (chunked && overflow) {  // (rare: one lane per Gaussian is enough)
            const uint32_t n = super_span(tx0, (int)rc.y, ty0, (int)rc.w);
            for (uint32_t k = 0; k < n && base + k < ecap; ++k) {
                skey[base + k] = 0;
                gidx[base + k] = g;
                smask[base + k] = 0ull;
            }
        }
        // flattened (Gaussian, super-tile) items of the small rectangles
        const uint32_t items = act && !chunked ? super_span(tx0, (int)rc.y, ty0, (int)rc.w) : 0u;
        const uint32_t incl = wave_incl_scan(items, lane);
        const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
        sx[lane] = incl - items;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t prect = (uint32_t)tx0 | ((uint32_t)ty0 << 16), psize = (uint32_t)ntx | ((uint32_t)nty << 8);
        for (uint32_t i0 = 0; i0 < total; i0 += kWave) {
            const uint32_t item = i0 + (uint32_t)lane;
            const int L = owner_lane(sx, item < total ? item : total - 1u);
            const uint32_t k = item < total ? item - sx[L] : 0u;  // (a spare lane redoes entry 0)
            const uint32_t gL = (uint32_t)__shfl((int)g, L, kWave), bL = (uint32_t)__shfl((int)base, L, kWave);
            const uint32_t pr = (uint32_t)__shfl((int)prect, L, kWave), ps = (uint32_t)__shfl((int)psize, L, kWave);
            const uint32_t hlo = (uint32_t)__shfl((int)er.z, L, kWave), hhi = (uint32_t)__shfl((int)er.w, L, kWave);
            const int ltx0 = (int)(pr & 0xffffu), lty0 = (int)(pr >> 16);
            const int lntx = (int)(ps & 0xffu), lnty = (int)(ps >> 8);
            const int sx0 = ltx0 >> kSuperShift, sy0 = lty0 >> kSuperShift;
            const int nsx = ((ltx0 + lntx - 1) >> kSuperShift) - sx0 + 1;  // at most 9 (k < 16)
            const int ey = small_div(k, nsx), ex = (int)k - ey * nsx;
            const uint64_t m = super_mask((uint64_t)hlo | ((uint64_t)hhi << 32), ltx0, lty0, lntx, lnty, sx0 + ex,
                                          sy0 + ey);
            const uint32_t at = bL + k;
            if (item < total && at < ecap) {  // never leave the entry buffers
                skey[at] = (uint16_t)((uint32_t)(sy0 + ey) * stx + (uint32_t)(sx0 + ex));
                gidx[at] = gL;
                smask[at] = m;
            }
        }
        // every lane has read the item starts before they are replaced
        __builtin_amdgcn_wave_barrier();
    }
}

// Entries of the chunked Gaussians.  Each wavefront takes up to 64 chunk
// slots, one per lane; the slot of a Gaussian's first chunk holds, in `big`,
// its output slot and entry offset, and each of its chunks takes an even share
// of its entries.  The wavefront flattens the entries of its chunks so
// that every lane builds one entry per step: entry k of a Gaussian is
// super-tile k of its rectangle's overlap in row-major order.  The chunk
// masks of a Gaussian are one bit stream over its rectangle in row-major
// order, so each of the super-tile's (at most kSuper) rows is a run of at
// most kSuper consecutive bits, read from two words.
//
// Bound by its writes, short runs at depth-ordered places in three arrays (an
// 8K frame's 844,000 chunks: 83 us; with all of a Gaussian's entries at its
// first chunk, and so in one wavefront, 109; 4K, 200,000 chunks: 23, was 27).
__global__ __launch_bounds__(kBlock) void k_big_entries(int W, const uint4 *__restrict__ erec, uint32_t ng,
                                                        const uint2 *__restrict__ chunks,
                                                        const uint2 *__restrict__ big, uint32_t chunk_cap,
                                                        const uint32_t *__restrict__ chunk_mask,
                                                        const FrameCounters *__restrict__ fc,
                                                        uint16_t *__restrict__ skey, uint32_t *__restrict__ gidx,
                                                        uint64_t *__restrict__ smask, uint32_t ecap) {
    __shared__ uint32_t s_excl[kBlock / kWave][kWave];
    // an overflowed list has entries this frame never wrote (the frame is
    // rendered again, or reported, by the host)
    if (fc->error & kErrChunkOverflow) return;
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t *sx = s_excl[threadIdx.x / kWave];
    const int tiles_x = (W + kTile - 1) / kTile;
    const uint32_t stx = (uint32_t)((tiles_x + kSuper - 1) >> kSuperShift);
    const uint32_t n = fc->nchunks < chunk_cap ? fc->nchunks : chunk_cap;
    const uint32_t nwaves = gridDim.x * (kBlock / kWave);
    constexpr uint32_t kWordsPerChunk = kChunkTiles / 32;
    const size_t wlast = (size_t)chunk_cap * kWordsPerChunk - 1;
    // an even share of at most 64 chunk slots per wavefront and round
    const uint32_t rounds = n / (nwaves * kWave) + 1u, per = (n + nwaves * rounds - 1u) / (nwaves * rounds);
    const uint32_t w0 = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    for (uint32_t c0 = w0 * per; c0 < n; c0 += nwaves * per) {
        const uint32_t c = (uint32_t)lane < per ? c0 + (uint32_t)lane : n;
        uint32_t first = 0, k0 = 0, items = 0;
        uint2 gb = make_uint2(0u, 0u);
        uint4 rc = make_uint4(0u, 0u, 0u, 0u);
        if (c < n) {
            first = chunks[c].y;
            gb = big[first];
            if (gb.x < ng) {
                rc = unpack_rect(erec[gb.x]);
                const uint32_t nt = (rc.y - rc.x + 1u) * (rc.w - rc.z + 1u);
                const uint32_t nch = (nt + kChunkTiles - 1) / kChunkTiles;
                const uint32_t span = super_span((int)rc.x, (int)rc.y, (int)rc.z, (int)rc.w);
                const uint32_t j = c - first;
                if (j < nch) {
                    k0 = (uint32_t)((uint64_t)span * j / nch);
                    items = (uint32_t)((uint64_t)span * (j + 1u) / nch) - k0;
                }
            }
        }
        const uint32_t incl = wave_incl_scan(items, lane);
        const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
        sx[lane] = incl - items;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t px = rc.x | (rc.y << 16), py = rc.z | (rc.w << 16);
        for (uint32_t i0 = 0; i0 < total; i0 += kWave) {
            const uint32_t item = i0 + (uint32_t)lane;
            const int L = owner_lane(sx, item < total ? item : total - 1u);
            const uint32_t k = (uint32_t)__shfl((int)k0, L, kWave) + (item < total ? item - sx[L] : 0u);
            const uint32_t fc0 = (uint32_t)__shfl((int)first, L, kWave);
            const uint32_t g = (uint32_t)__shfl((int)gb.x, L, kWave), base = (uint32_t)__shfl((int)gb.y, L, kWave);
            const uint32_t lx = (uint32_t)__shfl((int)px, L, kWave), ly = (uint32_t)__shfl((int)py, L, kWave);
            const int bx0 = (int)(lx & 0xffffu), bx1 = (int)(lx >> 16), by0 = (int)(ly & 0xffffu), by1 = (int)(ly >> 16);
            const int bntx = bx1 - bx0 + 1;
            const int sx0 = bx0 >> kSuperShift, sy0 = by0 >> kSuperShift;
            const int nsx = (bx1 >> kSuperShift) - sx0 + 1;
            int ey, ex;
            row_col((int)k, nsx, __builtin_amdgcn_rcpf((float)nsx), ey, ex);
            const int xs = (sx0 + ex) << kSuperShift, ys = (sy0 + ey) << kSuperShift;
            const int xa = xs > bx0 ? xs : bx0, xb = xs + kSuper - 1 < bx1 ? xs + kSuper - 1 : bx1;
            const int ya = ys > by0 ? ys : by0, yb = ys + kSuper - 1 < by1 ? ys + kSuper - 1 : by1;
            const uint64_t lmask = (1ull << (xb - xa + 1)) - 1ull;  // xb - xa + 1 <= kSuper
            const size_t wbase = (size_t)fc0 * kWordsPerChunk;
            // every row's two words are loaded (rows past yb repeat row yb)
            // before any is used: one memory round trip
            uint32_t lo[kSuper], hi[kSuper], sh[kSuper];
#pragma unroll
            for (int rr = 0; rr < kSuper; ++rr) {
                const int ty = ya + rr < yb ? ya + rr : yb;
                const uint32_t idx = (uint32_t)((ty - by0) * bntx + (xa - bx0));
                const size_t wlo = wbase + idx / 32 < wlast ? wbase + idx / 32 : wlast;
                const size_t whi = wlo + 1 < wlast ? wlo + 1 : wlast;
                lo[rr] = chunk_mask[wlo];
                hi[rr] = chunk_mask[whi];
                sh[rr] = idx % 32;
            }
            uint64_t m = 0;
#pragma unroll
            for (int rr = 0; rr < kSuper; ++rr) {
                const uint64_t bits = (((uint64_t)lo[rr] | ((uint64_t)hi[rr] << 32)) >> sh[rr]) & lmask;
                const int place = (ya + rr - ys) * kSuper + (xa - xs);
                m |= ya + rr <= yb ? bits << place : 0ull;
            }
            const uint32_t at = base + k;
            if (item < total && at < ecap) {
                skey[at] = (uint16_t)((uint32_t)(ys >> kSuperShift) * stx + (uint32_t)(xs >> kSuperShift));
                gidx[at] = g;
                smask[at] = m;
            }
        }
        // every lane has read the item starts before they are replaced
        __builtin_amdgcn_wave_barrier();
    }
}

// LDS visibility of this wavefront's own writes to its own later reads
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exact tile tests of the chunked Gaussians, row by row.  A wavefront takes up
// to 64 consecutive chunk slots: every lane loads one slot's descriptor and
// then its Gaussian's rectangle, centre, conic and k^2, so that they cost two
// memory round trips together, and leaves them with the row intervals' terms
// in LDS.  The rows of all its chunks are then flattened over the lanes, one
// (chunk, row) each: the row's columns that can be hit and those that
// certainly are follow from two intervals (tile_test.hpp); the few between
// them take the exact test, and the hits are runs of bits set in the chunk's
// mask in LDS.  The masks are written out together, and the hits of a
// Gaussian's consecutive chunks are summed across the lanes before one atomic
// per Gaussian and wavefront; a workgroup adds its hits to the frame's pair
// count once.
// Bound by VALU and LDS latency (about 300 instructions per step of 64 rows).
// One exact test per tile (60 instructions each) took 182 us beside the depth
// sort for the 10M city at 4K (205k chunks) and 440 us at 8K (873k), and held
// the sort's wavefronts back; the rows take 72 and 164 us, and a list of 83
// chunks 11 us instead of 73.
__global__ __launch_bounds__(kBlock) void k_big_count(int W, int H, int binning, const GaussState *__restrict__ gs,
                                                      const float4 *__restrict__ conic,
                                                      const uint4 *__restrict__ erec,
                                                      const uint2 *__restrict__ chunks, uint32_t chunk_cap,
                                                      uint32_t *__restrict__ chunk_mask, uint32_t *count,
                                                      FrameCounters *fc) {
    constexpr int kWords = kChunkTiles / 32;  // mask words of a chunk
    static_assert(kWords == 8, "a chunk's mask is two 16-byte words");
    __shared__ uint32_t s_hits[kBlock / kWave];
    struct alignas(16) Slot {
        float u, v, A, B, C, k2;
        RowTest rt;
        uint32_t cols, rows, first, i0;  // tx0 | ntx << 16, ty0 | (last tile - i0) << 16, first row, first tile
    };
    static_assert(sizeof(Slot) == 64, "four 16-byte reads");
    __shared__ Slot s_slot[kBlock / kWave][kWave];
    __shared__ alignas(16) uint32_t s_mask[kBlock / kWave][kWave * kWords];
    __shared__ uint32_t s_excl[kBlock / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    uint32_t whits = 0;  // wave-uniform
    // an overflowed list has entries this frame never wrote (the frame is
    // rendered again, or reported, by the host)
    if (!(fc->error & kErrChunkOverflow)) {
        const uint32_t n = fc->nchunks < chunk_cap ? fc->nchunks : chunk_cap;
        const uint32_t nwaves = gridDim.x * (kBlock / kWave);
        // chunks per wavefront: as many as spread the list over the grid
        // (which is resident at once), one per lane at most
        const uint32_t share = (n + nwaves - 1u) / nwaves, per = share < (uint32_t)kWave ? share : (uint32_t)kWave;
        uint32_t *const sx = s_excl[wv];
        uint32_t *const sm = s_mask[wv];
        for (uint32_t c0 = (blockIdx.x * (kBlock / kWave) + (uint32_t)wv) * per; c0 < n; c0 += nwaves * per) {
            const uint32_t c = c0 + (uint32_t)lane;
            uint2 e = make_uint2(kNoChunk, 0u);
            if ((uint32_t)lane < per && c < n) e = chunks[c];
            const bool have = e.x != kNoChunk;
            uint32_t items = 0;
            bool slow = false;  // no intervals (a needle, or terms that may overflow): every tile is tested
            if (have) {
                const uint4 rr = erec[e.x];
                Slot sl;
                float4 f0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), f1 = f0, cn = f0;
                if (binning == 0) {
                    const float4 *sp = reinterpret_cast<const float4 *>(gs + e.x);
                    f0 = sp[0];
                    f1 = sp[1];
                    cn = conic[e.x];
                }
                sl.u = f0.x;
                sl.v = f0.y;
                sl.A = cn.x;
                sl.B = cn.y;
                sl.C = cn.z;
                sl.k2 = f1.y;
                sl.rt = row_test(sl.u, sl.v, sl.A, sl.B, sl.C, sl.k2);
                const int tx0 = (int)(rr.x & 0xffffu), ntx = (int)(rr.x >> 16) - tx0 + 1;
                const int ty0 = (int)(rr.y & 0xffffu), nt = ntx * ((int)(rr.y >> 16) - ty0 + 1);
                const int i0 = (int)(c - e.y) * kChunkTiles;
                const int i1 = (i0 + kChunkTiles < nt ? i0 + kChunkTiles : nt) - 1;
                const float rcpn = __builtin_amdgcn_rcpf((float)ntx);
                int ra, rb, x;
                row_col(i0, ntx, rcpn, ra, x);
                row_col(i1, ntx, rcpn, rb, x);
                items = binning != 0 || sl.rt.fo > 0.0f ? (uint32_t)(rb - ra + 1) : 0u;
                slow = items == 0;
                sl.cols = (uint32_t)tx0 | ((uint32_t)ntx << 16);
                sl.rows = (uint32_t)ty0 | ((uint32_t)(i1 - i0) << 16);
                sl.first = (uint32_t)ra;
                sl.i0 = (uint32_t)i0;
                s_slot[wv][lane] = sl;
            }
#pragma unroll
            for (int k = 0; k < kWords / 4; ++k)
                reinterpret_cast<uint4 *>(sm)[lane * (kWords / 4) + k] = make_uint4(0u, 0u, 0u, 0u);
            const uint32_t incl_i = wave_incl_scan(items, lane);
            const uint32_t total = (uint32_t)__shfl((int)incl_i, kWave - 1, kWave);
            sx[lane] = incl_i - items;
            wave_sync();
            for (uint32_t t0 = 0; t0 < total; t0 += kWave) {
                const uint32_t item = t0 + (uint32_t)lane;
                if (item >= total) continue;
                const int L = owner_lane(sx, item);
                const Slot sl = s_slot[wv][L];
                const int row = (int)(sl.first + (item - sx[L]));
                const int tx0 = (int)(sl.cols & 0xffffu), ntx = (int)(sl.cols >> 16);
                const int ty = (int)(sl.rows & 0xffffu) + row;
                // the chunk's tiles of this row, as columns
                const int base = row * ntx - (int)sl.i0;  // bit of the row's column 0 in the chunk
                const int last = (int)(sl.rows >> 16);
                const int ca = base < 0 ? -base : 0, cb = base + ntx - 1 > last ? last - base : ntx - 1;
                RowCols rc{tx0 + ca, tx0 + cb, tx0 + ca, tx0 + cb};
                if (binning == 0) {
                    float y0, y1;
                    tile_row_span(sl.v, ty, H, y0, y1);
                    rc = row_columns(sl.rt, sl.u, y0, y1, tx0 + ca, tx0 + cb, W);
                }
                uint32_t *const m = sm + L * kWords;
                auto set_run = [&](int a, int b) {  // bits a..b of the chunk
                    for (int w = a >> 5; w <= b >> 5; ++w) {
                        const int lo = a - 32 * w > 0 ? a - 32 * w : 0, hi = b - 32 * w < 31 ? b - 32 * w : 31;
                        atomicOr(&m[w], (~0u << lo) & (~0u >> (31 - hi)));
                    }
                };
                const bool sure = rc.sure_first <= rc.sure_last;
                if (sure) set_run(base + rc.sure_first - tx0, base + rc.sure_last - tx0);
                // undecided columns: before the certain run and after it (all
                // that can be hit if there is none)
                const int before = (sure ? rc.sure_first : rc.last + 1) - rc.first;
                const int after = sure ? rc.last - rc.sure_last : 0;
                for (int k = 0; k < before + after; ++k) {
                    const int tx = k < before ? rc.first + k : rc.sure_last + 1 + (k - before);
                    if (tile_hit<true>(sl.u, sl.v, sl.A, sl.B, sl.C, sl.k2, tx, ty, W, H)) {
                        const int b = base + tx - tx0;
                        atomicOr(&m[b >> 5], 1u << (b & 31));
                    }
                }
            }
            // chunks without intervals: their tiles over the lanes
            for (uint64_t todo = __ballot(slow); todo; todo &= todo - 1ull) {
                const int L = __builtin_ctzll(todo);
                const Slot sl = s_slot[wv][L];
                const int tx0 = (int)(sl.cols & 0xffffu), ntx = (int)(sl.cols >> 16), ty0 = (int)(sl.rows & 0xffffu);
                const int n_tiles = (int)(sl.rows >> 16) + 1;
                const float rcpn = __builtin_amdgcn_rcpf((float)ntx);
#pragma unroll
                for (int q = 0; q < kChunkTiles / kWave; ++q) {
                    bool h = false;
                    if (q * kWave + lane < n_tiles) {
                        int ry, rx;
                        row_col((int)sl.i0 + q * kWave + lane, ntx, rcpn, ry, rx);
                        h = tile_hit<false>(sl.u, sl.v, sl.A, sl.B, sl.C, sl.k2, tx0 + rx, ty0 + ry, W, H);
                    }
                    const uint64_t bal = __ballot(h);
                    if (lane < 2) sm[L * kWords + 2 * q + lane] = lane ? (uint32_t)(bal >> 32) : (uint32_t)bal;
                }
            }
            wave_sync();
            // this lane's chunk: its mask's hits, and the mask
            const uint4 m0 = reinterpret_cast<const uint4 *>(sm)[lane * 2], m1 = reinterpret_cast<const uint4 *>(sm)[lane * 2 + 1];
            const uint32_t my_hits =
                (uint32_t)(__popc(m0.x) + __popc(m0.y) + __popc(m0.z) + __popc(m0.w) + __popc(m1.x) + __popc(m1.y) +
                           __popc(m1.z) + __popc(m1.w));
            if (have) {
                uint4 *const dst = reinterpret_cast<uint4 *>(chunk_mask + (size_t)c * kWords);
                dst[0] = m0;
                dst[1] = m1;
            }
            // one atomic per run of lanes holding chunks of the same Gaussian
            // (a Gaussian's chunks are consecutive slots)
            const uint32_t incl = wave_incl_scan(my_hits, lane);
            whits += (uint32_t)__shfl((int)incl, kWave - 1, kWave);
            const uint32_t gprev = (uint32_t)__shfl_up((int)e.x, 1, kWave);
            const uint32_t gnext = (uint32_t)__shfl_down((int)e.x, 1, kWave);
            const bool head = lane == 0 || gprev != e.x;
            const bool tail = lane == kWave - 1 || gnext != e.x;
            const uint64_t heads = __ballot(head);
            // the run's first lane: the highest head at or below this lane
            const int first = 63 - __builtin_clzll(heads & (lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1ull)));
            const uint32_t before = (uint32_t)__shfl((int)incl, first > 0 ? first - 1 : 0, kWave);
            const uint32_t run = incl - (first > 0 ? before : 0u);
            if (have && tail && run) atomicAdd(&count[e.x], run);
            wave_sync();  // every lane has read the masks before they are cleared
        }
    }
    if (lane == 0) s_hits[wv] = whits;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
#pragma unroll
        for (int w = 0; w < kBlock / kWave; ++w) t += s_hits[w];
        if (t) atomicAdd(&fc->pairs, t);
    }
}

}  // namespace

// Workgroups that fit on the device at once for a kernel (its register and
// LDS use decide the occupancy): a persistent grid of exactly that size
// keeps every CU busy without a tail of late workgroups.
template <class K>
static unsigned resident_blocks(K kernel) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess || per_cu <= 0 ||
        cus <= 0)
        return kPersistentBlocks;
    const unsigned n = (unsigned)(per_cu * cus);
    return n < (unsigned)kPersistentBlocks ? n : (unsigned)kPersistentBlocks;
}

unsigned preprocess_grid(int64_t P) {
    static const unsigned cap = resident_blocks(k_preprocess<false>);
    const int64_t b = (P + kBlock - 1) / kBlock;
    return (unsigned)(b < (int64_t)cap ? (b > 0 ? b : 1) : cap);
}

unsigned emit_grid(uint32_t visible) {
    static const unsigned cap = resident_blocks(k_super_emit);
    const uint32_t b = (visible + kBlock - 1) / kBlock;
    return b < cap ? (b > 0 ? b : 1u) : cap;
}

void launch_preprocess(const DevScene &sc, const DevPrepared *pp, const DevCamera &cam, const DevCam64 &cam64,
                       const DevOptions &op, int W, int H, GaussState *gs, float4 *conic, uint4 *rect, uint32_t *count,
                       uint8_t *count8, uint4 *erec, uint32_t *dkey, uint32_t *cand, uint32_t *seg_count,
                       uint32_t *gmap, uint2 *chunks, uint32_t chunk_cap, FrameCounters *fc, uint32_t *gsum_clear,
                       bool full, hipStream_t s) {
    if (sc.P <= 0) return;
    const PreArgs a{sc,   pp ? *pp : DevPrepared{}, cam,  cam64, op,        W,    H,      gs,        conic, rect, count,
                    count8, erec, dkey, cand, seg_count, gmap, chunks, chunk_cap, fc,    gsum_clear, (int)full,
                    MultiOut{}};
    if (pp)
        hipLaunchKernelGGL(k_preprocess<true>, dim3(preprocess_grid(sc.P)), dim3(kBlock), 0, s, a);
    else if (!full && (int64_t)preprocess_grid(sc.P) * kBlock < sc.P)
        hipLaunchKernelGGL((k_preprocess<false, false, true>), dim3(preprocess_grid(sc.P)), dim3(kBlock), 0, s, a);
    else
        // every wavefront has one group of 64: there is nothing to merge, and
        // the list's test and its code would only add their latency (10,000
        // Gaussians: 12.7 us with both forms in one kernel, 11.7 with this one);
        // or a kept frame, whose outputs go to the Gaussians' own slots, so that
        // a list has nothing to pack and gains nothing (listed / this one, us, at
        // 1080p: 300,000 Gaussians, 93 % visible, 50 / 46; 1M of them 107 / 102;
        // the city, 29 % visible, 2M 186 / 188, 6M 560 / 554, 10M 934 / 933; 3M
        // Gaussians of which none is visible 40 / 42)
        hipLaunchKernelGGL(k_preprocess<false>, dim3(preprocess_grid(sc.P)), dim3(kBlock), 0, s, a);
}

void launch_cull(const DevScene &sc, const DevPrepared &pp, const DevCamera &cam, const DevOptions &op, int W, int H,
                 uint32_t *cand, uint32_t *seg_count, FrameCounters *fc, hipStream_t s) {
    if (sc.P <= 0) return;
    hipLaunchKernelGGL(k_cull<false>, dim3(kCullBlocks), dim3(kBlock), 0, s, sc, pp, cam, op, W, H, cand, seg_count,
                       fc, MultiOut{});
}

void launch_preprocess_multi(const DevScene &sc, const DevPrepared &pp, const MultiOut &mo, const DevOptions &op,
                             uint32_t *cand, uint32_t *seg_count, uint32_t *gmap, hipStream_t s) {
    if (sc.P <= 0 || mo.n < 1 || mo.n > kMaxCams) return;
    const CamOut &c0 = mo.c[0];
    hipLaunchKernelGGL(k_cull<true>, dim3(kCullBlocks), dim3(kBlock), 0, s, sc, pp, c0.cam, op, c0.W, c0.H, cand,
                       seg_count, c0.fc, mo);
    const PreArgs a{sc,        pp,      c0.cam,  c0.cam64, op,        c0.W,      c0.H,         c0.gs, c0.conic,
                    c0.rect,   c0.count, c0.count8, c0.erec, c0.dkey,   cand,      seg_count,    gmap,  c0.chunks,
                    c0.chunk_cap, c0.fc, c0.gsum_clear, 0,   mo};
    hipLaunchKernelGGL((k_preprocess<true, true>), dim3(preprocess_grid(sc.P)), dim3(kBlock), 0, s, a);
}

void launch_prepare(const DevScene &sc, const DevOptions &op, const uint32_t *perm, float4 *pos_o, float4 *cov,
                    float *sh, float2 *bnd, uint32_t *orig, int sh_stride, hipStream_t s) {
    if (sc.P <= 0) return;
    const int64_t blocks = (sc.P + kBlock - 1) / kBlock;
    const dim3 grid((unsigned)(blocks < 8192 ? blocks : 8192));
    uint32_t *const inv = const_cast<uint32_t *>(perm) + sc.P;
    hipLaunchKernelGGL(k_invert, grid, dim3(kBlock), 0, s, perm, sc.P, inv, orig);
    hipLaunchKernelGGL(k_prepare, grid, dim3(kBlock), 0, s, sc, op, inv, pos_o, cov, sh, bnd, sh_stride);
}

void launch_block_bounds(const float4 *pos_o, const float2 *bnd, int64_t P, float4 *blk, hipStream_t s) {
    if (P <= 0) return;
    hipLaunchKernelGGL(k_block_bounds, dim3((unsigned)((P + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, pos_o, bnd, P,
                       blk);
}

void launch_spatial_keys(const DevScene &sc, uint32_t *bounds, uint32_t *keys, hipStream_t s) {
    hipLaunchKernelGGL(k_spatial_bounds_init, dim3(1), dim3(64), 0, s, bounds);
    if (sc.P <= 0) return;
    const int64_t blocks = (sc.P + kBlock - 1) / kBlock;
    const unsigned grid = (unsigned)(blocks < 4096 ? blocks : 4096);
    hipLaunchKernelGGL(k_spatial_bounds, dim3(grid < 1024 ? grid : 1024), dim3(kBlock), 0, s, sc, bounds);
    hipLaunchKernelGGL(k_spatial_keys, dim3(grid), dim3(kBlock), 0, s, sc, bounds, keys);
}

// (asked for by the first half already: the second one may be under capture)
static unsigned big_entries_grid() {
    static const unsigned grid = resident_blocks(k_big_entries);
    return grid;
}

void launch_big_count(int W, int H, int binning, const GaussState *gs, const float4 *conic, const uint4 *erec,
                      const uint2 *chunks, uint32_t chunk_cap, uint32_t *chunk_mask, uint32_t *count,
                      FrameCounters *fc, hipStream_t s) {
    (void)big_entries_grid();
    if (chunk_cap == 0) return;
    static const unsigned grid = resident_blocks(k_big_count);
    hipLaunchKernelGGL(k_big_count, dim3(grid), dim3(kBlock), 0, s, W, H, binning, gs, conic, erec,
                       chunks, chunk_cap, chunk_mask, count, fc);
}

void launch_super_emit(int W, int H, const uint32_t *order, uint32_t visible, const uint32_t *visible_dev,
                       const uint32_t *offsets, const uint4 *erec, uint32_t ng, const uint2 *chunks, uint2 *big,
                       const uint32_t *chunk_mask, uint32_t chunk_cap, const FrameCounters *fc, uint16_t *skey,
                       uint32_t *gidx, uint64_t *smask, uint32_t ecap, uint2 *sranges, uint32_t nsuper,
                       uint32_t *gsum_clear, hipStream_t s) {
    (void)H;
    if (visible == 0 && (!sranges || nsuper == 0) && !gsum_clear) return;
    if (order) {
        unsigned grid = emit_grid(visible);
        if (sranges) grid = std::max(grid, std::min<unsigned>((nsuper + kBlock - 1) / kBlock, kPersistentBlocks));
        hipLaunchKernelGGL(k_super_emit, dim3(grid), dim3(kBlock), 0, s, W, order, visible, visible_dev, offsets, erec,
                           big, chunk_cap, skey, gidx, smask, ecap, sranges, nsuper, gsum_clear, fc);
    }
    if (chunk_cap == 0 || visible == 0 || !chunk_mask) return;
    hipLaunchKernelGGL(k_big_entries, dim3(big_entries_grid()), dim3(kBlock), 0, s, W, erec, ng, chunks, big,
                       chunk_cap, chunk_mask, fc, skey, gidx, smask, ecap);
}

}  // namespace fgs

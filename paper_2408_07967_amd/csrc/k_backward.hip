// Adjoint of the rasterizer: gradients of a scalar loss with respect to the
// raw Gaussian parameters, given dL/dRGB.  The paper calls its rasterizer
// differentiable without giving the adjoint; this follows the usual
// replay of the blend from the saved per-pixel final transmittance and last
// contributor, with wavefront-reduced atomics (the DISTWAR approach the paper
// cites among related work).
//
// k_blend_bwd: one 256-thread workgroup per tile and one wavefront per 8 x 8
// quadrant, with the forward's staged coefficients and exponent (so both take
// the same contribution and clamp decisions).  Each pixel walks its tile list
// back to front from its last contributor:
//     T_n = T_{n+1} / (1 - a_n)
//     dL/dc_n     = g . a_n T_n                        (g = dL/dRGB of the pixel)
//     dL/da_n     = T_n (g . c_n - r_n),   r_{n-1} = r_n + a_n (g . c_n - r_n),  r_last = g . bg
//     dL/dq_n     = -a_n / 2 dL/da_n     (0 where a_n is clamped at alpha_max)
// What a Gaussian needs from a tile are nine sums over its pixels: of
// w = a_n dL/da_n with the six monomials 1, x^2, xy, y^2, x, y of the pixel's
// position, and of a_n T_n with the pixel's three dL/dRGB.  Both are
// contractions over the pixels with factors that no Gaussian changes, so they
// run on the matrix cores: a wavefront leaves the w and a T of eight Gaussians
// as the rows of a 16 x 64 matrix in LDS, whose product with the 64 x 9 matrix
// of the quadrant's monomials and dL/dRGB (kept in registers) gives the sums
// of all eight.  The monomials are taken about the quadrant's centre (at most
// 3.5 pixels away, so that moving the sums to the Gaussian's centre, done on
// the product's lanes, cancels little).  (Summing the
// nine terms over the lanes with DPP adds took 54 of about 130 VALU
// instructions per step; with one plane per accumulator each of a Gaussian's
// nine atomics was a request of its own.  1M Gaussians at 1920 x 1080: 897 ->
// 390 us, 10k at 256 x 256: 278 -> 113 us, the errors of the gradients against
// binary64 unchanged.)
// Accumulators per Gaussian (kAccStride floats, one 64-byte line):
//     0: sum dL/dq            1..3: sum dL/dq dx^2, dx dy, dy^2
//     4..5: sum dL/dq dx, dy  6..8: sum dL/dcolour
// They go to HBM with one atomic per term, 16 lanes to a Gaussian, so that a
// Gaussian's nine atomics are one request to its line.
// From these, dL/dA, dL/dB, dL/dC, dL/du, dL/dv and dL/do (= -2 sum dL/dq / o,
// since da/do = a / o) follow per Gaussian.
//
// k_preprocess_bwd: one lane per Gaussian; recomputes the preprocessing
// steps in binary32 and applies the chain rule in reverse: conic = inverse
// of Sigma', Sigma' = T Sigma T^T + dilation I, T = J R_cam, Sigma = M M^T,
// M = R(q / |q|) diag(exp(log-scale)), (u, v) and J from the camera-space
// mean, opacity = sigmoid(logit), colour = max(0, SH . Y(d) + 1/2).
// Bound by HBM: 1M Gaussians of degree 3 (94 % with gradients), 0.6 GB: 108 us.
// It took 193 with the culled Gaussians' zeros in a branch of their own, so
// that nearly every line of the 59 gradient planes was written twice, in parts,
// and with the coefficients read one basis function at a time between the
// stores (on gfx950 a wait for a load also waits for every earlier store); with
// the coefficients read together 172.
#include <type_traits>

#include "fgs_internal.hpp"
#include "blend_common.hpp"
#include "sh_basis.hpp"

namespace fgs {
namespace {

constexpr int kWave = 64;
constexpr int kAcc = 9;
constexpr int kBwdBatch = 128;            // list entries staged at a time
constexpr int kSlots = 8;                 // Gaussians reduced by one matrix product
constexpr int kRowPitch = kWave + 4;      // LDS pitch of a row of 64 pixels (rows start four banks apart)
constexpr int kBwdWaves = kBlock / kWave; // one per quadrant

typedef float float4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)v, d, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// Lane kLane of each row of 16 lanes, in all lanes of the row
template <int kLane>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + kLane, 0xf, 0xf, false));  // row_newbcast
}

// LDS visibility of this wavefront's own writes to its own later reads
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(kBlock) void k_blend_bwd(const GaussState *__restrict__ gs,
                                                      const uint32_t *__restrict__ values,
                                                      const uint2 *__restrict__ ranges, const float *__restrict__ Tfin,
                                                      const uint32_t *__restrict__ last, const float *__restrict__ dL,
                                                      int W, int H, int tiles_x, DevOptions op,
                                                      float *__restrict__ acc) {
    __shared__ float4 s_f0[kBwdBatch], s_f1[kBwdBatch];
    __shared__ float2 s_f2[kBwdBatch];
    __shared__ uint32_t s_id[kBwdBatch];
    __shared__ uint32_t s_rel[4][kBwdBatch / kWave][2];
    __shared__ float s_acc[kBwdBatch][kAcc];
    __shared__ alignas(16) float s_w[kBwdWaves][2 * kSlots][kRowPitch];
    __shared__ uint32_t s_lmax;

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile = blockIdx.x;
    const int tx = tile % tiles_x, ty = tile / tiles_x;
    const int qx = wave & 1, qy = wave >> 1;
    const int pi = tx * kTile + qx * 8 + (lane & 7);
    const int pj = ty * kTile + qy * 8 + (lane >> 3);
    const bool in_img = pi < W && pj < H;
    const float px = (float)pi + 0.5f, py = (float)pj + 0.5f;
    const size_t hw = (size_t)W * H;
    const size_t p = in_img ? (size_t)pj * W + pi : 0;

    float T = in_img ? Tfin[p] : 1.0f;
    const uint32_t L = in_img ? last[p] : 0u;
    const float g0 = in_img ? dL[p] : 0.0f, g1 = in_img ? dL[hw + p] : 0.0f, g2 = in_img ? dL[2 * hw + p] : 0.0f;
    float rest = fmaf(g0, op.bg[0], fmaf(g1, op.bg[1], g2 * op.bg[2]));  // r_n
    const float amax = op.alpha_max + 0.0f;
    const uint32_t wave_L = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(L));

    // The right operand of the products (v_mfma_f32_16x16x4_f32, 16 steps of
    // four pixels): lane l holds column l % 16 of pixel 16 (l / 16) + s in
    // step s (columns 0..5 the monomials, 6..8 dL/dRGB).
    float bm[kWave / 4];
    {
        const int col = lane & 15, kb = lane >> 4;
#pragma unroll
        for (int s = 0; s < kWave / 4; ++s) {
            const int lx = qx * 8 + (s & 7), ly = qy * 8 + 2 * kb + (s >> 3);
            const float x = (float)(s & 7) - 3.5f, y = (float)(2 * kb + (s >> 3)) - 3.5f;
            const int i = tx * kTile + lx, j = ty * kTile + ly;
            float v = col == 0 ? 1.0f : col == 1 ? x * x : col == 2 ? x * y : col == 3 ? y * y : col == 4 ? x : y;
            if (col > 5) v = 0.0f;
            if (col > 5 && col < kAcc && i < W && j < H) v = dL[(size_t)(col - 6) * hw + (size_t)j * W + i];
            bm[s] = v;
        }
    }

    if (tid == 0) s_lmax = 0;
    for (int e = tid; e < kBwdBatch * kAcc; e += kBlock) (&s_acc[0][0])[e] = 0.0f;
    __syncthreads();
    if (lane == 0) atomicMax(&s_lmax, wave_L);
    __syncthreads();
    const uint32_t lmax = s_lmax;
    const uint32_t start = ranges[tile].x;

    float(*const sw)[kRowPitch] = s_w[wave];
    const float qcx = (float)(tx * kTile + qx * 8 + 4), qcy = (float)(ty * kTile + qy * 8 + 4);  // quadrant's centre
    int n_slots = 0;      // wave-uniform: rows filled
    uint64_t slot_j = 0;  // wave-uniform: the batch entry of each slot, one byte each
    static_assert(kBwdBatch <= 256 && kSlots == 8, "one byte per slot");

    // the sums of the filled slots into s_acc
    auto reduce_slots = [&]() {
        wave_sync();
        float4v d = {0.0f, 0.0f, 0.0f, 0.0f};
        const float *row = &sw[lane & 15][16 * (lane >> 4)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 a = *reinterpret_cast<const float4 *>(row + 4 * q);
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, bm[4 * q], d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, bm[4 * q + 1], d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, bm[4 * q + 2], d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, bm[4 * q + 3], d, 0, 0, 0);
        }
        // lane l, element r: row 4 (l / 16) + r, column l % 16; rows 0..7 are
        // the slots' w (columns 0..5), rows 8..15 their a T (columns 6..8).
        // The w sums are moved to the Gaussian's centre (u, v) (relative to
        // the quadrant's) from the row's sums of 1, x and y:
        //   sum w (x - u) = sx - u s0 = X,  sum w (x - u)^2 = sxx - u (sx + X),
        //   sum w (x - u)(y - v) = sxy - u sy - v X, and so in y.
        const int col = lane & 15, blk = lane >> 4;
        const bool use = blk < 2 ? col < 6 : col >= 6 && col < kAcc;
        const uint32_t js = (blk & 1) ? (uint32_t)(slot_j >> 32) : (uint32_t)slot_j;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t j = (js >> (8 * r)) & 255u;
            float o = d[r];
            const float s0 = row_bcast<0>(o), sx = row_bcast<4>(o), sy = row_bcast<5>(o);
            const float u = s_f0[j].x - qcx, v = s_f0[j].y - qcy;
            const float X = fmaf(-u, s0, sx), Y = fmaf(-v, s0, sy);
            if (blk < 2) {
                o = col == 4 ? X : col == 5 ? Y : o;
                o = col == 1 ? fmaf(-u, sx + X, o) : col == 2 ? fmaf(-v, X, fmaf(-u, sy, o)) : o;
                o = col == 3 ? fmaf(-v, sy + Y, o) : o;
                o *= -0.5f;  // w is -2 dL/dq
            }
            if (use && 4 * (blk & 1) + r < n_slots) atomicAdd(&s_acc[j][col], o);
        }
        // every lane has read the rows before they are refilled
        wave_sync();
        n_slots = 0;
        slot_j = 0;
    };

    for (int hi = (int)lmax; hi > 0; hi -= kBwdBatch) {
        const int lo = hi > kBwdBatch ? hi - kBwdBatch : 0;
        const int nb = hi - lo;
        // Two threads per entry, each testing two of the quadrants.  The replay
        // has to blend what the forward blended: a quadrant counts only where its
        // half is met.  The half's test is taken where it can have dropped a
        // contributor, for long thin footprints aslant (a quadrant met in a half
        // that is rightly not met has no contributor, so it may count).
        {
            const int j = tid & (kBwdBatch - 1), h = tid / kBwdBatch;
            uint32_t qm = 0;
            if (j < nb) {
                const uint32_t g = values[start + (uint32_t)lo + (uint32_t)j];
                const GaussState s = gs[g];
                const int X0 = tx * kTile, Y0 = ty * kTile + h * 8;
                const float k2t = test_extent_thin(s);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (X0 + 8 * q < W && Y0 < H && region_hit(s, k2t, X0 + 8 * q, 8, Y0, W, H)) qm |= 1u << q;
                if (qm != 0 && half_test_decides(s, k2t) && !region_hit(s, test_extent(s), X0, kTile, Y0, W, H)) qm = 0;
                if (h == 0) {
                    float4 f0, f1;
                    float2 f2;
                    stage_gauss(s, f0, f1, f2);
                    s_f0[j] = f0;
                    s_f1[j] = f1;
                    s_f2[j] = f2;
                    s_id[j] = g;
                }
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint64_t bq = __ballot((qm >> q) & 1u);
                if (lane == 0) {
                    s_rel[2 * (wave >> 1) + q][wave & 1][0] = (uint32_t)bq;
                    s_rel[2 * (wave >> 1) + q][wave & 1][1] = (uint32_t)(bq >> 32);
                }
            }
        }
        __syncthreads();
        if ((uint32_t)lo < wave_L) {
            for (int wd = kBwdBatch / kWave - 1; wd >= 0; --wd) {
                uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)s_rel[wave][wd][0]) |
                             ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)s_rel[wave][wd][1]) << 32);
                while (m) {
                    const int bit = 63 - __builtin_clzll(m);
                    m &= ~(1ull << bit);
                    const int j = wd * kWave + bit;
                    const uint32_t pos = (uint32_t)(lo + j);
                    if (pos >= wave_L) continue;
                    const float4 f0 = s_f0[j], f1 = s_f1[j];
                    const float2 f2 = s_f2[j];
                    // the forward's exponent and contribution test, bit for bit
                    const float E = exponent_at(f0, row_terms(f0, f1, py), px);
                    const bool c = pos < L && E >= f1.y;
                    if (__ballot(c) == 0) continue;
                    const float e = __builtin_amdgcn_exp2f(E);
                    const float a = c ? fminf(e, amax) : 0.0f;
                    T = T * __builtin_amdgcn_rcpf(1.0f - a);  // a = 0: T unchanged
                    const float wc = a * T;
                    // (0 beside a 0 weight: an overflow stays with the pixels that blend it)
                    const float d = c ? fmaf(g0, f1.w, fmaf(g1, f2.x, fmaf(g2, f2.y, -rest))) : 0.0f;
                    rest = fmaf(a, d, rest);
                    sw[n_slots][lane] = e <= amax ? wc * d : 0.0f;
                    sw[kSlots + n_slots][lane] = wc;
                    slot_j |= (uint64_t)j << (8 * n_slots);
                    if (++n_slots == kSlots) reduce_slots();
                }
            }
            if (n_slots) reduce_slots();
        }
        __syncthreads();
        for (int e = tid; e < nb * kAccStride; e += kBlock) {
            const int j = e / kAccStride, k = e % kAccStride;
            if (k < kAcc) {
                const float v = s_acc[j][k];
                s_acc[j][k] = 0.0f;
                if (v != 0.0f) unsafeAtomicAdd(acc + (size_t)s_id[j] * kAccStride + k, v);
            }
        }
        __syncthreads();  // the entries are read before the next ones are staged
    }
}

struct DevGrad {
    float *means, *log_scales, *quats, *logits, *sh;
    int64_t stride;
};

__global__ __launch_bounds__(kBlock) void k_preprocess_bwd(DevScene sc, DevCamera cam, DevOptions op, int W, int H,
                                                           const GaussState *__restrict__ gs,
                                                           const float *__restrict__ acc, DevGrad gr) {
    const int64_t st = sc.stride, gst = gr.stride;
    // the first coefficient of each degree (and the end), as constants
    using std::integral_constant;
    constexpr integral_constant<int, 0> c0{};
    constexpr integral_constant<int, 1> c1{};
    constexpr integral_constant<int, 4> c4{};
    constexpr integral_constant<int, 9> c9{};
    constexpr integral_constant<int, 16> c16{};
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < sc.P;
         g += (int64_t)gridDim.x * blockDim.x) {
        float S[kAcc];
        bool any = false;
        {
            const float4 *const a4 = reinterpret_cast<const float4 *>(acc + (size_t)g * kAccStride);
            const float4 q0 = a4[0], q1 = a4[1], q2 = a4[2];
            const float t[kAcc] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x};
#pragma unroll
            for (int k = 0; k < kAcc; ++k) {
                S[k] = t[k];
                any |= S[k] != 0.0f;
            }
        }
        // zero for a Gaussian that is culled or that no pixel depends on; every
        // lane's gradients are stored by the same instructions, as whole lines
        float gm3[3] = {0.0f, 0.0f, 0.0f}, gls[3] = {0.0f, 0.0f, 0.0f}, gq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float glogit = 0.0f, gcol[3] = {0.0f, 0.0f, 0.0f}, Y[16] = {};
        if (any) {
            const GaussState s = gs[g];
            const float A = s.f0.z, B = s.f0.w, C = s.f1.x, o = s.f2.w;
            const float col[3] = {s.f1.w, s.f2.x, s.f2.y};
            // gradients of the blended state
            const float gA = S[1], gB = 2.0f * S[2], gC = S[3];
            const float gu = -2.0f * (A * S[4] + B * S[5]);
            const float gv = -2.0f * (B * S[4] + C * S[5]);
            const float go = -2.0f * S[0] / o;
            for (int ch = 0; ch < 3; ++ch) gcol[ch] = col[ch] > 0.0f ? S[6 + ch] : 0.0f;

            // ---- forward recomputation ----------------------------------------
            const float m[3] = {sc.means[g], sc.means[st + g], sc.means[2 * st + g]};
            const float ls[3] = {sc.log_scales[g], sc.log_scales[st + g], sc.log_scales[2 * st + g]};
            const float qr[4] = {sc.quats[g], sc.quats[st + g], sc.quats[2 * st + g], sc.quats[3 * st + g]};
            const float logit = sc.logits[g];
            const float *Rc = cam.R;
            float t[3];
            for (int r = 0; r < 3; ++r)
                t[r] = Rc[3 * r] * m[0] + Rc[3 * r + 1] * m[1] + Rc[3 * r + 2] * m[2] + cam.t[r];
            const float sc3[3] = {expf(ls[0]), expf(ls[1]), expf(ls[2])};
            const float qn = sqrtf(qr[0] * qr[0] + qr[1] * qr[1] + qr[2] * qr[2] + qr[3] * qr[3]);
            const float w = qr[0] / qn, x = qr[1] / qn, y = qr[2] / qn, z = qr[3] / qn;
            const float iz = 1.0f / t[2];
            const float xt = t[0] * iz, yt = t[1] * iz;
            const float limx = op.jac_clip * (0.5f * (float)W / cam.fx);
            const float limy = op.jac_clip * (0.5f * (float)H / cam.fy);
            const bool clipx = xt < -limx || xt > limx, clipy = yt < -limy || yt > limy;
            const float xc = fminf(fmaxf(xt, -limx), limx), yc = fminf(fmaxf(yt, -limy), limy);
            const float J00 = cam.fx * iz, J02 = -cam.fx * xc * iz, J11 = cam.fy * iz, J12 = -cam.fy * yc * iz;
            const float Rq[9] = {1.0f - 2.0f * (y * y + z * z), 2.0f * (x * y - w * z), 2.0f * (x * z + w * y),
                                 2.0f * (x * y + w * z), 1.0f - 2.0f * (x * x + z * z), 2.0f * (y * z - w * x),
                                 2.0f * (x * z - w * y), 2.0f * (y * z + w * x), 1.0f - 2.0f * (x * x + y * y)};
            float M[9];
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) M[3 * i + j] = Rq[3 * i + j] * sc3[j];
            float Sig[9];
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j)
                    Sig[3 * i + j] = M[3 * i] * M[3 * j] + M[3 * i + 1] * M[3 * j + 1] + M[3 * i + 2] * M[3 * j + 2];
            float Tm[6];
            for (int j = 0; j < 3; ++j) {
                Tm[j] = J00 * Rc[j] + J02 * Rc[6 + j];
                Tm[3 + j] = J11 * Rc[3 + j] + J12 * Rc[6 + j];
            }

            // ---- conic = inverse of X = Sigma' + dilation I: dL/dX = -Y dL/dY Y
            const float hB = 0.5f * gB;
            const float t00 = A * gA + B * hB, t01 = A * hB + B * gC, t10 = B * gA + C * hB, t11 = B * hB + C * gC;
            const float p00 = -(t00 * A + t01 * B), p01 = -(t00 * B + t01 * C);
            const float p10 = -(t10 * A + t11 * B), p11 = -(t10 * B + t11 * C);
            const float gSp[4] = {p00, p01, p10, p11};
            // ---- Sigma' = T Sigma T^T ---------------------------------------------
            // dL/dSigma = T^T gSp T;  dL/dT = (gSp + gSp^T) T Sigma
            float gSig[9];
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) {
                    float a = 0.0f;
                    for (int u = 0; u < 2; ++u)
                        for (int v = 0; v < 2; ++v) a += Tm[3 * u + i] * gSp[2 * u + v] * Tm[3 * v + j];
                    gSig[3 * i + j] = a;
                }
            float TS[6];
            for (int u = 0; u < 2; ++u)
                for (int j = 0; j < 3; ++j)
                    TS[3 * u + j] = Tm[3 * u] * Sig[j] + Tm[3 * u + 1] * Sig[3 + j] + Tm[3 * u + 2] * Sig[6 + j];
            const float P2[4] = {2.0f * p00, p01 + p10, p01 + p10, 2.0f * p11};
            float gT[6];
            for (int u = 0; u < 2; ++u)
                for (int j = 0; j < 3; ++j) gT[3 * u + j] = P2[2 * u] * TS[j] + P2[2 * u + 1] * TS[3 + j];
            // ---- T = J R_cam: only J00, J02, J11, J12 vary ------------------------
            const float gJ00 = gT[0] * Rc[0] + gT[1] * Rc[1] + gT[2] * Rc[2];
            const float gJ02 = gT[0] * Rc[6] + gT[1] * Rc[7] + gT[2] * Rc[8];
            const float gJ11 = gT[3] * Rc[3] + gT[4] * Rc[4] + gT[5] * Rc[5];
            const float gJ12 = gT[3] * Rc[6] + gT[4] * Rc[7] + gT[5] * Rc[8];
            // ---- Sigma = M M^T, M = R_q diag(s) ---------------------------------
            float gR[9], gs3[3] = {0.0f, 0.0f, 0.0f};
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) {
                    float gm = 0.0f;
                    for (int l = 0; l < 3; ++l) gm += (gSig[3 * i + l] + gSig[3 * l + i]) * M[3 * l + j];
                    gR[3 * i + j] = gm * sc3[j];
                    gs3[j] += gm * Rq[3 * i + j];
                }
            for (int j = 0; j < 3; ++j) gls[j] = gs3[j] * sc3[j];
            // ---- rotation of the unit quaternion, then the normalisation --------
            const float gw = 2.0f * (-z * gR[1] + y * gR[2] + z * gR[3] - x * gR[5] - y * gR[6] + x * gR[7]);
            const float gx = 2.0f * (y * gR[1] + z * gR[2] + y * gR[3] - 2.0f * x * gR[4] - w * gR[5] + z * gR[6] +
                                     w * gR[7] - 2.0f * x * gR[8]);
            const float gy = 2.0f * (-2.0f * y * gR[0] + x * gR[1] + w * gR[2] + x * gR[3] + z * gR[5] - w * gR[6] +
                                     z * gR[7] - 2.0f * y * gR[8]);
            const float gz = 2.0f * (-2.0f * z * gR[0] - w * gR[1] + x * gR[2] + w * gR[3] - 2.0f * z * gR[4] +
                                     y * gR[5] + x * gR[6] + y * gR[7]);
            const float dq = w * gw + x * gx + y * gy + z * gz;
            const float iqn = 1.0f / qn;
            gq[0] = (gw - w * dq) * iqn;
            gq[1] = (gx - x * dq) * iqn;
            gq[2] = (gy - y * dq) * iqn;
            gq[3] = (gz - z * dq) * iqn;
            // ---- J and (u, v) from the camera-space mean ----------------------------
            const float iz2 = iz * iz;
            float gt[3] = {0.0f, 0.0f, 0.0f};
            gt[2] += -(gJ00 * cam.fx + gJ11 * cam.fy) * iz2 + (gJ02 * cam.fx * xc + gJ12 * cam.fy * yc) * iz2;
            float gxt = clipx ? 0.0f : -gJ02 * cam.fx * iz;
            float gyt = clipy ? 0.0f : -gJ12 * cam.fy * iz;
            gxt += gu * cam.fx;
            gyt += gv * cam.fy;
            gt[0] += gxt * iz;
            gt[1] += gyt * iz;
            gt[2] -= (gxt * t[0] + gyt * t[1]) * iz2;
            for (int j = 0; j < 3; ++j) gm3[j] = Rc[j] * gt[0] + Rc[3 + j] * gt[1] + Rc[6 + j] * gt[2];
            // ---- opacity ----------------------------------------------------------
            glogit = go * o * (1.0f - o);
            // ---- SH colour at the view direction ------------------------------------
            const float dw[3] = {m[0] - cam.eye[0], m[1] - cam.eye[1], m[2] - cam.eye[2]};
            const float dn = sqrtf(dw[0] * dw[0] + dw[1] * dw[1] + dw[2] * dw[2]);
            const float idn = 1.0f / dn;
            const float d[3] = {dw[0] * idn, dw[1] * idn, dw[2] * idn};
            float wk[16];
            sh_basis(d[0], d[1], d[2], sc.D, Y);
            // (all coefficients are read together: one memory round trip)
            const float *shp = sc.sh + g;
            float shv[48];
            auto load_sh = [&](auto k0, auto k1) {
#pragma unroll
                for (int j = 3 * k0; j < 3 * k1; ++j, shp += st) shv[j] = *shp;
            };
            auto dot_sh = [&](auto k0, auto k1) {
#pragma unroll
                for (int k = k0; k < k1; ++k)
                    wk[k] = gcol[0] * shv[3 * k] + gcol[1] * shv[3 * k + 1] + gcol[2] * shv[3 * k + 2];
            };
            load_sh(c0, c1);
            if (sc.D >= 1) load_sh(c1, c4);
            if (sc.D >= 2) load_sh(c4, c9);
            if (sc.D >= 3) load_sh(c9, c16);
            dot_sh(c0, c1);
            if (sc.D >= 1) dot_sh(c1, c4);
            if (sc.D >= 2) dot_sh(c4, c9);
            if (sc.D >= 3) dot_sh(c9, c16);
            float gd[3];
            sh_basis_grad(d[0], d[1], d[2], sc.D, wk, gd);
            const float dd = d[0] * gd[0] + d[1] * gd[1] + d[2] * gd[2];
            for (int e = 0; e < 3; ++e) gm3[e] += (gd[e] - d[e] * dd) * idn;
        }
        for (int e = 0; e < 3; ++e) gr.means[e * gst + g] = gm3[e];
        for (int e = 0; e < 3; ++e) gr.log_scales[e * gst + g] = gls[e];
        for (int e = 0; e < 4; ++e) gr.quats[e * gst + g] = gq[e];
        gr.logits[g] = glogit;
        float *gsh = gr.sh + g;
        auto store_sh = [&](auto k0, auto k1) {
#pragma unroll
            for (int k = k0; k < k1; ++k)
#pragma unroll
                for (int ch = 0; ch < 3; ++ch, gsh += gst) *gsh = gcol[ch] * Y[k];
        };
        store_sh(c0, c1);
        if (sc.D >= 1) store_sh(c1, c4);
        if (sc.D >= 2) store_sh(c4, c9);
        if (sc.D >= 3) store_sh(c9, c16);
    }
}

}  // namespace

// Threads of a workgroup for accumulators of acc_stride floats per Gaussian: the
// kernels know one layout, and a launch of no threads is refused by the runtime,
// so that the caller's check of its last error sees another one.
static unsigned bwd_threads(int64_t acc_stride) { return acc_stride == kAccStride ? (unsigned)kBlock : 0u; }

void launch_blend_backward(const GaussState *gs, const uint32_t *values, const uint2 *ranges, const float *Tfin,
                           const uint32_t *last, const float *dL, int W, int H, const DevOptions &op, float *acc,
                           int64_t acc_stride, hipStream_t s) {
    const int tiles_x = (W + kTile - 1) / kTile, tiles_y = (H + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_blend_bwd, dim3((unsigned)(tiles_x * tiles_y)), dim3(bwd_threads(acc_stride)), 0, s, gs,
                       values, ranges, Tfin, last, dL, W, H, tiles_x, op, acc);
}

void launch_preprocess_backward(const DevScene &sc, const DevCamera &cam, const DevOptions &op, int W, int H,
                                const GaussState *gs, const float *acc, int64_t acc_stride, float *g_means,
                                float *g_log_scales, float *g_quats, float *g_logits, float *g_sh,
                                int64_t grad_stride, hipStream_t s) {
    if (sc.P <= 0) return;
    DevGrad gr{g_means, g_log_scales, g_quats, g_logits, g_sh, grad_stride};
    const int64_t blocks = (sc.P + kBlock - 1) / kBlock;
    const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
    hipLaunchKernelGGL(k_preprocess_bwd, dim3(grid), dim3(bwd_threads(acc_stride)), 0, s, sc, cam, op, W, H, gs, acc, gr);
}

}  // namespace fgs

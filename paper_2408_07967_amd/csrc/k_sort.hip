// Per-tile lists from the super-tile entries sorted by super-tile (the
// sort stage of Sec. 2.2: pairs ordered by tile, then depth, each tile's
// workload is its run of the list), the range of a one-run list, and a fill
// kernel used to clear counters.
//
// After the stable sort by super-tile, super-tile s holds its entries in
// depth order, each with the 64-bit mask of the Gaussian's hit tiles in s.
// The sorted pair list is the concatenation over tiles t (in id order) of
// the Gaussians hitting t in depth order, so a pair (entry i of s, tile bit
// j) goes to start(t) + #{entries of s before i with bit j set}, with start
// the exclusive scan of the tiles' pair counts.  A super-tile's entries are
// cut into chunks of kListChunk, one wavefront each, so that a dense
// super-tile spreads over many CUs:
//   k_list_chunks  up to 16 workgroups, each scanning all super-tiles and
//                  writing its share: chunk bases of the super-tiles and the
//                  super-tile of every chunk;
//   k_list_count   per chunk: the 64 tiles' hit counts (lane j: bit j), by
//                  transposing each 64 x 64 bit block of masks across lanes;
//   k_list_scan    one workgroup per super-tile: exclusive scan of its
//                  chunks' counts per tile; its tile totals, and its sum
//                  added to its row of super-tiles;
//   k_tile_starts  one workgroup per row of super-tiles (a contiguous band
//                  of tile ids): the earlier rows' sums, then an exclusive
//                  scan of the band's tile totals in tile id order ->
//                  ranges[t] = [start, start + count);
//   k_list_write   per chunk again: its masks transposed, lane j lists in LDS
//                  the entries that hit tile j behind the earlier tiles', and
//                  the list is written by all lanes, each entry's Gaussian at
//                  its tile's running position.
// Chunks are dealt to the XCDs in eight contiguous ranges, so that a
// super-tile's consecutive chunks, which write the same tiles' lists, share
// an L2.
#include <algorithm>

#include "fgs_internal.hpp"

namespace fgs {
namespace {

constexpr int kWave = 64;

__global__ void k_fill_u32(uint32_t *p, uint32_t value, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// The one range of a one-run list: every element (*n_dev of them, at most n).
__global__ void k_single_range(uint2 *__restrict__ ranges, uint32_t n, const uint32_t *__restrict__ n_dev) {
    if (threadIdx.x == 0) ranges[0] = make_uint2(0u, min(n, *n_dev));
}

// Entries [b, e) of super-tile s (start > end: none; clamped to ecap).
__device__ __forceinline__ uint2 super_entries(const uint2 *sranges, uint32_t s, uint32_t ecap) {
    const uint2 r = sranges[s];
    uint32_t b = r.x, e = r.y;
    if (b > e) b = e = 0;
    e = e < ecap ? e : ecap;
    b = b < e ? b : e;
    return make_uint2(b, e);
}

// Tile of bit j (lane) of super-tile s, or -1 past the image's edge.
__device__ __forceinline__ int64_t lane_tile(uint32_t s, uint32_t stx, int tiles_x, int tiles_y, int lane) {
    const int tx = (int)(s % stx) * kSuper + (lane & (kSuper - 1));
    const int ty = (int)(s / stx) * kSuper + (lane >> kSuperShift);
    return (tx < tiles_x && ty < tiles_y) ? (int64_t)ty * tiles_x + tx : -1;
}

// Lane l's value from lane l ^ kStep (kStep at most 16), in registers.
template <int kStep>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t x, int lane) {
    if constexpr (kStep == 16) {
        // rows of 16: the second row of each pair from the first, and back
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane & 16) ? r[0] : r[1];
    } else if constexpr (kStep == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);  // row_ror:8
    } else if constexpr (kStep == 4) {
        const int m = __builtin_amdgcn_mov_dpp((int)x, 0x141, 0xf, 0xf, true);  // row_half_mirror: l ^ 7
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1b, 0xf, 0xf, true);     // quad_perm [3, 2, 1, 0]: l ^ 3
    } else if constexpr (kStep == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4e, 0xf, 0xf, true);  // quad_perm [2, 3, 0, 1]
    } else {
        static_assert(kStep == 1, "a power of two");
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xb1, 0xf, 0xf, true);  // quad_perm [1, 0, 3, 2]
    }
}

// One stage of the transpose below: the off-diagonal kStep x kStep blocks of
// every 2 kStep x 2 kStep block change places (kLow: the low kStep bits of
// each 2 kStep bits).
template <int kStep, uint32_t kLow>
__device__ __forceinline__ void transpose_stage(uint32_t &lo, uint32_t &hi, int lane) {
    const bool up = (lane & kStep) != 0;
    const uint32_t keep = up ? ~kLow : kLow;
    const uint32_t rot = up ? kStep : 32 - kStep;  // to the right
    const uint32_t a = from_lane_xor<kStep>(lo, lane), b = from_lane_xor<kStep>(hi, lane);
    lo = (lo & keep) | (__builtin_amdgcn_alignbit(a, a, rot) & ~keep);
    hi = (hi & keep) | (__builtin_amdgcn_alignbit(b, b, rot) & ~keep);
}

// Transpose of the 64 x 64 bit matrix whose row i is lane i's word: lane j
// gets column j (bit i = bit j of row i).  Six butterfly stages swap the
// off-diagonal s x s blocks of every 2s x 2s block (s = 32 ... 1), between
// lanes by register moves: through the LDS permute and with 64-bit shifts
// k_list_count took 16.4 us at 4K and 23.9 at 8K, now 13.6 and 20.5.
__device__ __forceinline__ uint64_t transpose64(uint64_t x, int lane) {
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)(x >> 32), false, false);
    uint32_t lo = r[0], hi = r[1];
    transpose_stage<16, 0x0000ffffu>(lo, hi, lane);
    transpose_stage<8, 0x00ff00ffu>(lo, hi, lane);
    transpose_stage<4, 0x0f0f0f0fu>(lo, hi, lane);
    transpose_stage<2, 0x33333333u>(lo, hi, lane);
    transpose_stage<1, 0x55555555u>(lo, hi, lane);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// The chunks of [0, n) that this wavefront takes: n is cut into eight
// contiguous ranges, one per XCD (workgroups are placed on the eight XCDs in
// turn, and the grid is a multiple of eight workgroups), and the XCD's
// wavefronts take its range's chunks in turn.
struct ChunkWalk {
    uint32_t next, end, stride;
};
__device__ __forceinline__ ChunkWalk chunk_walk(uint32_t n, uint32_t wave_in_block, uint32_t waves_per_block) {
    const uint32_t nb = gridDim.x, x = blockIdx.x % 8u, k = blockIdx.x / 8u;
    const uint32_t nx = (nb - x + 7u) / 8u;  // workgroups on this XCD
    const uint32_t lo = (uint32_t)(((uint64_t)n * x) / 8u), hi = (uint32_t)(((uint64_t)n * (x + 1u)) / 8u);
    ChunkWalk w;
    w.next = lo + k * waves_per_block + wave_in_block;
    w.end = hi;
    w.stride = nx * waves_per_block;
    return w;
}

constexpr int kListBlock = 256;  // chunk kernels: four wavefronts, one chunk each at a time
// (The scans' workgroups are of four wavefronts too: one of sixteen starts only
// where a CU has sixteen free wave slots at once, and beside another frame's
// blend, whose small workgroups take every slot that falls free, k_list_scan
// waited up to 290 us and k_tile_starts 270: four cameras in one batch, average
// 42 and 79 us, now 28 and 27.)
constexpr int kScanBlock = 256;
constexpr int kScanWaves = kScanBlock / kWave;
constexpr uint32_t kChunkBlocks = 16;  // workgroups of k_list_chunks, at most

// cbase[s] = first chunk of super-tile s (cbase[nsuper] = the total), and
// csuper[q] = the super-tile of chunk q.  Every workgroup scans all super-tiles
// (a few thousand ranges in L2) and writes the bases and the chunks of its
// share of them: no workgroup waits for another one.
__global__ __launch_bounds__(kScanBlock) void k_list_chunks(const uint2 *__restrict__ sranges, uint32_t nsuper,
                                                            uint32_t ecap, uint32_t *cbase,
                                                            uint32_t *__restrict__ csuper,
                                                            uint32_t *__restrict__ rowsum) {
    __shared__ uint32_t s_w[kScanWaves];
    const uint32_t tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t b_lo = (uint32_t)((uint64_t)nsuper * blockIdx.x / gridDim.x);
    const uint32_t b_hi = (uint32_t)((uint64_t)nsuper * (blockIdx.x + 1) / gridDim.x);
    const uint32_t run = (nsuper + kScanBlock - 1) / kScanBlock;
    const uint32_t s0 = tid * run < nsuper ? tid * run : nsuper;
    const uint32_t s1 = s0 + run < nsuper ? s0 + run : nsuper;
    uint32_t own = 0;
#pragma unroll 8
    for (uint32_t s = s0; s < s1; ++s) {
        const uint2 r = super_entries(sranges, s, ecap);
        own += (r.y - r.x + kListChunk - 1) / kListChunk;
    }
    uint32_t x = own;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
        if (lane >= d) x += y;
    }
    if (lane == kWave - 1) s_w[wave] = x;
    __syncthreads();
    uint32_t base = x - own;
    for (int q = 0; q < kScanWaves; ++q) base += q < wave ? s_w[q] : 0u;
    // (the share's end, too: its last chunk ends there)
    if (s0 <= b_hi && s1 >= b_lo)
        for (uint32_t s = s0; s < s1; ++s) {
            const uint2 r = super_entries(sranges, s, ecap);
            if (s >= b_lo && s <= b_hi) cbase[s] = base;
            if (s >= b_lo && s < b_hi) rowsum[s] = 0;  // (the rows of super-tiles are at most nsuper)
            base += (r.y - r.x + kListChunk - 1) / kListChunk;
        }
    if (b_hi == nsuper && tid == kScanBlock - 1) cbase[nsuper] = base;
    __syncthreads();  // (and the bases are visible to the workgroup)
    // the super-tile of every chunk: a wavefront takes up to 64 of the share's
    // super-tiles and fills one's chunks after the other with all its lanes
    // (one thread per super-tile, a dense one's hundreds of chunks in turn,
    // took the kernel 19.0 us at 4K with 10M Gaussians and 21.7 at 8K; filled by
    // the sixteen wavefronts of one workgroup 8.1 and 19.1; now 5.9 and 9.5)
    uint32_t share = (b_hi - b_lo + kScanWaves - 1) / kScanWaves;
    share = share < (uint32_t)kWave ? share : (uint32_t)kWave;
    for (uint32_t b0 = b_lo + (uint32_t)wave * share; b0 < b_hi; b0 += kScanWaves * share) {
        const uint32_t s = b0 + (uint32_t)lane;
        const bool mine = (uint32_t)lane < share && s < b_hi;
        const uint32_t lo = mine ? cbase[s] : 0u, hi = mine ? cbase[s + 1] : 0u;
        for (uint32_t j = 0; j < share; ++j) {
            const uint32_t c1 = (uint32_t)__builtin_amdgcn_readlane((int)hi, (int)j);
            for (uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)j) + (uint32_t)lane; c < c1; c += kWave)
                csuper[c] = b0 + j;
        }
    }
}

__global__ __launch_bounds__(kListBlock) void k_list_count(const uint2 *__restrict__ sranges, uint32_t ecap,
                                                           const uint32_t *__restrict__ cbase, uint32_t nsuper,
                                                           const uint32_t *__restrict__ csuper,
                                                           const uint64_t *__restrict__ smask,
                                                           uint32_t *__restrict__ cnt) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t n = cbase[nsuper];
    for (ChunkWalk cw = chunk_walk(n, wv, kListBlock / kWave); cw.next < cw.end; cw.next += cw.stride) {
        const uint32_t q = cw.next;
        const uint32_t s = csuper[q];
        const uint2 r = super_entries(sranges, s, ecap);
        const uint32_t b = r.x + (q - cbase[s]) * kListChunk;
        const uint32_t e = b + kListChunk < r.y ? b + kListChunk : r.y;
        uint64_t m[kListChunk / kWave];
#pragma unroll
        for (int k = 0; k < (int)(kListChunk / kWave); ++k) {
            const uint32_t i = b + (uint32_t)(k * kWave + lane);
            m[k] = i < e ? smask[i] : 0ull;
        }
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < (int)(kListChunk / kWave); ++k) c += (uint32_t)__popcll(transpose64(m[k], lane));
        cnt[(size_t)q * kWave + lane] = c;
    }
}

// One workgroup per super-tile: its chunks' counts become exclusive
// prefixes per tile (in place), and its tile totals go to ranges[t].x.
__global__ __launch_bounds__(kScanBlock) void k_list_scan(const uint32_t *__restrict__ cbase, uint32_t stx,
                                                          int tiles_x, int tiles_y, uint32_t *__restrict__ cnt,
                                                          uint2 *__restrict__ ranges, uint32_t *__restrict__ rowsum) {
    constexpr uint32_t kStep = 8;  // chunks whose counts are read together
    __shared__ uint32_t s_sum[kScanWaves][kWave];
    const uint32_t s = blockIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t c0 = cbase[s], n = cbase[s + 1] - c0;
    const uint32_t per = (n + kScanWaves - 1) / kScanWaves;
    const uint32_t r0 = c0 + (w * per < n ? w * per : n), r1 = c0 + ((w + 1) * per < n ? (w + 1) * per : n);
    uint32_t sum = 0;
    for (uint32_t q = r0; q < r1; q += kStep) {
#pragma unroll
        for (uint32_t k = 0; k < kStep; ++k) sum += q + k < r1 ? cnt[(size_t)(q + k) * kWave + lane] : 0u;
    }
    s_sum[w][lane] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kScanWaves; ++k) {
        const uint32_t v = s_sum[k][lane];
        run += k < w ? v : 0u;
        tot += v;
    }
    for (uint32_t q = r0; q < r1; q += kStep) {
        uint32_t v[kStep];
#pragma unroll
        for (uint32_t k = 0; k < kStep; ++k) v[k] = q + k < r1 ? cnt[(size_t)(q + k) * kWave + lane] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < kStep; ++k) {
            if (q + k < r1) cnt[(size_t)(q + k) * kWave + lane] = run;
            run += v[k];
        }
    }
    if (w == 0) {
        const int64_t t = lane_tile(s, stx, tiles_x, tiles_y, lane);
        if (t >= 0) ranges[t] = make_uint2(tot, 0u);
        uint32_t st = tot;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) st += (uint32_t)__shfl_xor((int)st, d, kWave);
        if (lane == 0 && st) atomicAdd(&rowsum[s / stx], st);
    }
}

// Workgroup b: the tiles of super-tile row b (tile rows kSuper b ...
// kSuper b + kSuper - 1, a contiguous range of tile ids).  Its first start is
// the sum of the earlier rows; its tiles are scanned 1024 at a time, four
// consecutive ones per thread.
__global__ __launch_bounds__(kScanBlock) void k_tile_starts(uint2 *__restrict__ ranges, int tiles_x, uint32_t ntiles,
                                                            const uint32_t *__restrict__ rowsum, uint32_t ncap) {
    constexpr uint32_t kPer = 4;
    __shared__ uint32_t s_w[kScanWaves];
    __shared__ uint32_t s_base;
    const uint32_t tid = threadIdx.x, b = blockIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    if (wave == 0) {
        uint32_t x = 0;
        for (uint32_t q = (uint32_t)lane; q < b; q += kWave) x += rowsum[q];
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) x += (uint32_t)__shfl_xor((int)x, d, kWave);
        if (lane == 0) s_base = x;
    }
    __syncthreads();
    uint32_t start = s_base;
    const uint32_t band = (uint32_t)kSuper * (uint32_t)tiles_x;
    const uint32_t t_lo = b * band, t_hi = t_lo + band < ntiles ? t_lo + band : ntiles;
    for (uint32_t r0 = t_lo; r0 < t_hi; r0 += kScanBlock * kPer) {
        const uint32_t t = r0 + tid * kPer;
        uint32_t c[kPer], own = 0;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) c[k] = t + k < t_hi ? ranges[t + k].x : 0u;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) own += c[k];
        uint32_t x = own;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
            if (lane >= d) x += y;
        }
        if (lane == kWave - 1) s_w[wave] = x;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < kScanWaves; ++q) {
            const uint32_t v = s_w[q];
            before += q < wave ? v : 0u;
            all += v;
        }
        __syncthreads();
        uint32_t a0 = start + before + x - own;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) {
            if (t + k < t_hi) {
                const uint32_t a = a0 < ncap ? a0 : ncap;
                const uint32_t e = a0 + c[k] < ncap ? a0 + c[k] : ncap;
                ranges[t + k] = make_uint2(a, e);
            }
            a0 += c[k];
        }
        start += all;
    }
}

// A wavefront's pairs of one stretch of a chunk, tile by tile, before they are
// written: (tile << 8) | entry.  One 32-entry word has at most 32 x 64.
constexpr uint32_t kPairCap = 32 * kWave;
static_assert(kListChunk <= 256 && kWave * 256 <= 65536, "tile and entry in 16 bits");
constexpr int kListWords = 8;  // 32-entry words of a tile's column
static_assert(kListChunk == 32 * kListWords, "four 64-entry blocks");

// kBuf: values are stored through a buffer resource of ncap words, whose
// range check drops a store past the end (byte offsets: ncap < 2^29).
//
// Bound by instruction issue.  With a ballot per (tile, 64 entries) a store
// had 5 active lanes of 64 (4K, 10M Gaussians); here the masks are transposed,
// lane j walks the entries that its tile j hits and lists them in LDS behind
// the earlier tiles', and the list is then written by all lanes: one step per
// 64 pairs, with about as many separate lines as it has tiles' runs.
// 27.2M pairs of a 4K frame: 73 us before, 61 now; 76.7M of an 8K frame: 153,
// now 141 (write requests of 64 bytes: 5.1M for 307 MB of pairs); 4.6M of a
// 1080p frame: 25, now 18.  (With stores that bypass the L2's merging of the
// runs' ends 115 and 320 us; with four pairs per lane and step 60 and 152.)
// With a buffer of 4096 pairs per wavefront, i.e. four instead of seven
// workgroups per CU, the 1080p frame took 21.5.
template <bool kBuf>
__global__ __launch_bounds__(kListBlock) void k_list_write(const uint2 *__restrict__ sranges, uint32_t ecap,
                                                           const uint32_t *__restrict__ cbase, uint32_t nsuper,
                                                           const uint32_t *__restrict__ csuper, uint32_t stx,
                                                           int tiles_x, int tiles_y,
                                                           const uint32_t *__restrict__ gidx,
                                                           const uint64_t *__restrict__ smask,
                                                           const uint32_t *__restrict__ pre,
                                                           const uint2 *__restrict__ ranges,
                                                           uint32_t *__restrict__ values, uint32_t ncap) {
    __shared__ uint16_t s_pairs[kListBlock / kWave][kPairCap];
    __shared__ uint32_t s_g[kListBlock / kWave][kListChunk];
    __shared__ uint32_t s_delta[kListBlock / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint16_t *pairs = s_pairs[wv];
    uint32_t *gl = s_g[wv], *delta = s_delta[wv];
    auto lds_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const uint32_t n = cbase[nsuper];
    const __amdgpu_buffer_rsrc_t vrs =
        __builtin_amdgcn_make_buffer_rsrc(values, (short)0, kBuf ? (int)(ncap * 4u) : 0, 0x00020000);
    for (ChunkWalk cw = chunk_walk(n, wv, kListBlock / kWave); cw.next < cw.end; cw.next += cw.stride) {
        const uint32_t q = cw.next;
        const uint32_t s = csuper[q];
        const uint2 r = super_entries(sranges, s, ecap);
        const uint32_t b = r.x + (q - cbase[s]) * kListChunk;
        const uint32_t e = b + kListChunk < r.y ? b + kListChunk : r.y;
        uint64_t m[kListChunk / kWave];
        uint32_t g[kListChunk / kWave];
#pragma unroll
        for (int k = 0; k < (int)(kListChunk / kWave); ++k) {
            const uint32_t i = b + (uint32_t)(k * kWave + lane);
            m[k] = i < e ? smask[i] : 0ull;
            g[k] = i < e ? gidx[i] : 0u;
        }
        // lane j: the first output position of tile j (bit j) of this super-tile
        const int64_t t = lane_tile(s, stx, tiles_x, tiles_y, lane);
        uint32_t first = t >= 0 ? ranges[t].x + pre[(size_t)q * kWave + lane] : 0u;
        // lane j: the entries that hit tile j
        constexpr int kBlocks = kListWords / 2;
        uint32_t col[kListWords];
        uint32_t c01 = 0, c23 = 0;  // the lane's hits in the 64-entry blocks, two per word
#pragma unroll
        for (int k = 0; k < kBlocks; ++k) {
            gl[k * kWave + lane] = g[k];
            const uint64_t c = transpose64(m[k], lane);
            col[2 * k] = (uint32_t)c;
            col[2 * k + 1] = (uint32_t)(c >> 32);
            (k < 2 ? c01 : c23) += (uint32_t)__popcll(c) << (16 * (k & 1));
        }
        // the whole chunk at once where its pairs fit, else by halves, blocks
        // or words (which always fit)
        uint32_t b01 = c01, b23 = c23;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            b01 += (uint32_t)__shfl_xor((int)b01, d, kWave);
            b23 += (uint32_t)__shfl_xor((int)b23, d, kWave);
        }
        b01 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b01);
        b23 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b23);
        const uint32_t p0 = b01 & 0xffffu, p1 = b01 >> 16, p2 = b23 & 0xffffu, p3 = b23 >> 16;
        const uint32_t half = p0 + p1 > p2 + p3 ? p0 + p1 : p2 + p3;
        const uint32_t q01 = p0 > p1 ? p0 : p1, q23 = p2 > p3 ? p2 : p3;
        const int step = p0 + p1 + p2 + p3 <= kPairCap         ? 8
                         : half <= kPairCap                    ? 4
                         : (q01 > q23 ? q01 : q23) <= kPairCap ? 2
                                                               : 1;
        for (int w0 = 0; w0 < kListWords; w0 += step) {
            uint32_t cnt = 0;
#pragma unroll
            for (int w = 0; w < kListWords; ++w)
                if (w >= w0 && w < w0 + step) cnt += (uint32_t)__popc(col[w]);  // uniform
            uint32_t x = cnt;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint32_t y = (uint32_t)__shfl_up((int)x, d, kWave);
                if (lane >= d) x += y;
            }
            const uint32_t np = (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
            uint32_t p = x - cnt;
            delta[lane] = first - p;
            first += cnt;
#pragma unroll
            for (int w = 0; w < kListWords; ++w) {
                if (w < w0 || w >= w0 + step) continue;  // uniform
                uint32_t bits = col[w];
                const uint32_t tag = ((uint32_t)lane << 8) | (uint32_t)(w * 32);
                while (bits) {
                    pairs[p++] = (uint16_t)(tag + (uint32_t)__builtin_ctz(bits));
                    bits &= bits - 1u;
                }
            }
            lds_order();
            constexpr uint32_t kOut = 2;
            for (uint32_t i0 = (uint32_t)lane; i0 < np; i0 += kOut * kWave) {
                uint32_t u[kOut], gv[kOut], pos[kOut];
#pragma unroll
                for (uint32_t k = 0; k < kOut; ++k) {
                    const uint32_t i = i0 + k * kWave;
                    u[k] = pairs[i < np ? i : i0];
                }
#pragma unroll
                for (uint32_t k = 0; k < kOut; ++k) {
                    gv[k] = gl[u[k] & 255u];
                    pos[k] = delta[u[k] >> 8] + i0 + k * kWave;
                }
#pragma unroll
                for (uint32_t k = 0; k < kOut; ++k) {
                    if (i0 + k * kWave >= np) continue;
                    if constexpr (kBuf)
                        __builtin_amdgcn_raw_buffer_store_b32(gv[k], vrs, pos[k] * 4u, 0, 0);
                    else if (pos[k] < ncap)  // never leave the values
                        values[pos[k]] = gv[k];
                }
            }
            lds_order();
        }
    }
}

}  // namespace

void launch_fill_u32(uint32_t *p, uint32_t value, size_t n, hipStream_t s) {
    if (n == 0) return;
    size_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(kBlock), 0, s, p, value, n);
}

void launch_single_range(uint2 *ranges, uint32_t n, const uint32_t *n_dev, hipStream_t s) {
    hipLaunchKernelGGL(k_single_range, dim3(1), dim3(64), 0, s, ranges, n, n_dev);
}

void launch_tile_lists(int W, int H, const uint2 *sranges, const uint32_t *gidx, const uint64_t *smask,
                       uint32_t ecap, uint32_t *scratch, uint2 *ranges, uint32_t *values, uint32_t ncap,
                       hipStream_t s) {
    const int tiles_x = (W + kTile - 1) / kTile, tiles_y = (H + kTile - 1) / kTile;
    const uint32_t stx = (uint32_t)((tiles_x + kSuper - 1) >> kSuperShift);
    const uint32_t sty = (uint32_t)((tiles_y + kSuper - 1) >> kSuperShift);
    const uint32_t nsuper = stx * sty, ntiles = (uint32_t)tiles_x * (uint32_t)tiles_y;
    if (nsuper == 0) return;
    // scratch: chunk bases, chunk super-tiles, per-chunk counts (see list_scratch_words)
    const size_t g = list_chunks_max(ecap, nsuper);
    uint32_t *cbase = scratch;
    uint32_t *rowsum = cbase + nsuper + 1;
    uint32_t *csuper = cbase + (2 * nsuper + 1 + 63) / 64 * 64;
    uint32_t *cnt = csuper + (g + 63) / 64 * 64;
    // chunk grids: four chunks per workgroup, at most a few resident rounds,
    // a multiple of eight workgroups (every XCD's range has workgroups)
    const unsigned chunk_blocks = (unsigned)((std::min<size_t>((g + 3) / 4, 8192) + 7) / 8 * 8);
    hipLaunchKernelGGL(k_list_chunks, dim3(std::min<uint32_t>((nsuper + 15) / 16, kChunkBlocks)), dim3(kScanBlock), 0, s,
                       sranges, nsuper, ecap, cbase, csuper, rowsum);
    hipLaunchKernelGGL(k_list_count, dim3(chunk_blocks), dim3(kListBlock), 0, s, sranges, ecap, cbase, nsuper, csuper,
                       smask, cnt);
    hipLaunchKernelGGL(k_list_scan, dim3(nsuper), dim3(kScanBlock), 0, s, cbase, stx, tiles_x, tiles_y, cnt, ranges,
                       rowsum);
    hipLaunchKernelGGL(k_tile_starts, dim3(sty), dim3(kScanBlock), 0, s, ranges, tiles_x, ntiles, rowsum, ncap);
    if (ncap < (1u << 29))
        hipLaunchKernelGGL(k_list_write<true>, dim3(chunk_blocks), dim3(kListBlock), 0, s, sranges, ecap, cbase, nsuper,
                           csuper, stx, tiles_x, tiles_y, gidx, smask, cnt, ranges, values, ncap);
    else
        hipLaunchKernelGGL(k_list_write<false>, dim3(chunk_blocks), dim3(kListBlock), 0, s, sranges, ecap, cbase,
                           nsuper, csuper, stx, tiles_x, tiles_y, gidx, smask, cnt, ranges, values, ncap);
}

}  // namespace fgs

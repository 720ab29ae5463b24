// Full Stage I search (Sec. 2.4): matched filtering of every pixel's spectrum with a bank of
// unit-variance boxcars (the window sum over its noise standard deviation: sqrt(w) for white
// noise, sqrt(w + 2 sum_l (w - l) rho_l) when the caller gives the noise's channel correlations
// rho_l, e.g. those the periodic Hann window puts into imaged cubes), the best SNR and width per
// voxel, a Benjamini-Hochberg threshold over all searched voxels, width-aware non-maximum
// suppression along frequency and a local re-evaluation of every survivor against its flanks.
//
// Kernels:
//  * search_bank_std_kernel (the default 26 widths) and search_bank_kernel (any bank): a workgroup
//    takes 64 consecutive pixels (one per lane) and blocks of 128 channels (32 per wave), puts
//    prefix sums along frequency into LDS (relative to the block's staged channels, so window sums
//    never carry the rounding of a long running sum), and for every channel takes the maximum of
//    (P[s + w] - P[s]) / sigma_w over the widths whose window fits in the band (a test skipped for
//    channels at least 64 from both band edges, where every window fits).  They write the best SNR
//    (and, when wanted, width) cubes and each tile's largest in-horizon SNR, and add the in-horizon
//    SNRs at or above a floor F to a histogram (1/32 bins; LDS first, then one global atomic per
//    non-empty bin).  Benjamini-Hochberg never accepts a p-value above q (k q / m <= q), so no
//    voxel with S < Q^-1(q) is ever accepted; F lies at least one bin below Q^-1(q), and the
//    step-up search over the histogram is the search over all m voxels.
//  * The host walks the histogram from the lowest bin up to find the largest k with
//    p_(k) <= k q / m; only a bin where that is undecided by its edges is gathered exactly
//    (search_gather_kernel) and sorted on the host.
//  * search_accept_kernel lists the accepted voxels, search_width_kernel finds their widths when no
//    width cube was made, search_nms_kernel keeps those no neighbour suppresses, and
//    search_refine_kernel (a workgroup per survivor) re-evaluates them, its medians from an exact
//    rank count over at most 512 flank values.
#include "internal.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

namespace {

constexpr int SB_PX = 64;                                    // pixels per workgroup
constexpr int SB_CB = 128;                                   // channels per workgroup
constexpr int SB_HALO_L = NBSI_SEARCH_MAX_WIDTH / 2;         // floor(w / 2) <= 64
constexpr int SB_HALO_R = NBSI_SEARCH_MAX_WIDTH / 2 - 1;     // w - floor(w / 2) - 1 <= 63
constexpr int SB_ROWS = SB_CB + SB_HALO_L + SB_HALO_R;       // staged channels
constexpr int HIST_PER_UNIT = 32;
constexpr int HIST_SPAN = 64;                                // SNR units of 1/32 bins above F
constexpr int HIST_BINS = HIST_SPAN * HIST_PER_UNIT + 1;     // [F, F + 64) in 1/32 steps, then >= F + 64
constexpr int FLANK_MAX = 4 * NBSI_SEARCH_MAX_WIDTH;         // two flanks of at most 2 w_max each
constexpr int REEVAL_MIN_FLANK = 8;
constexpr float MAD_TO_SIGMA = 1.482602218505602f;

// The width bank: widths ascending, and per width the standard deviation sigma_w of the window
// sum of unit-variance noise with the caller's channel correlations (sqrt(w) when white) and its
// reciprocal.
struct Widths {
    int n;
    int w[NBSI_SEARCH_MAX_WIDTHS];
    float inv_sqrt[NBSI_SEARCH_MAX_WIDTHS];  // 1 / sigma_w
    float sigma[NBSI_SEARCH_MAX_WIDTHS];     // sigma_w
};

struct Cand {  // an accepted voxel
    int c, p, w;
    float s;
};

// What the passes after the bank count, read back together.
struct SearchCounts {
    int accepted;      // provisional detections
    unsigned min_key;  // order key of the smallest accepted SNR
    int survivors;     // of the suppression
};

__device__ __forceinline__ bool in_horizon(int p, int n_pix) {
    const int y = p / n_pix, x = p - y * n_pix, h = n_pix / 2;
    return (x - h) * (x - h) + (y - h) * (y - h) < h * h;
}

// Bin of an SNR s >= F = f32 / 32: bin j holds [(f32 + j) / 32, (f32 + j + 1) / 32).  s * 32 is
// exact (a power-of-two scale), so the bin edges are exact and no value lands beside its bin.
__device__ __forceinline__ int hist_bin(float s, int f32) {
    const float u = s * (float)HIST_PER_UNIT;
    return u >= (float)(f32 + HIST_BINS - 1) ? HIST_BINS - 1 : (int)floorf(u) - f32;
}

// Order-preserving map of a float to an unsigned key (negative values below positive ones).
__device__ __forceinline__ unsigned order_key(float s) {
    const unsigned b = __float_as_uint(s);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__host__ __device__ __forceinline__ float key_value(unsigned key) {  // the inverse
    const unsigned b = (key & 0x80000000u) ? (key & 0x7fffffffu) : ~key;
    float s;
    __builtin_memcpy(&s, &b, sizeof(float));
    return s;
}

// Largest in-horizon S of the tile of 64 pixels x SB_TC channels whose first channel is c (a wave's
// share of a block): the later passes visit only the tiles that reach their threshold.
constexpr int SB_TC = SB_CB / 4;
__device__ __forceinline__ void store_tile_max(float top, float *__restrict__ tmax, int c, int n_chan, int lane) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, 64));
    if (lane == 0 && c < n_chan) tmax[(size_t)(c / SB_TC) * gridDim.x + blockIdx.x] = top;
}

__global__ __launch_bounds__(256) void search_bank_kernel(const float *__restrict__ r, int n_chan, int n_pix,
                                                          Widths W, int f32, float *__restrict__ best,
                                                          uint8_t *__restrict__ wbest, unsigned *__restrict__ hist,
                                                          float *__restrict__ tmax) {
    __shared__ float P[(SB_ROWS + 1) * SB_PX];  // P[i][lane] = sum of staged rows < i (exclusive)
    __shared__ float seg_tot[4][SB_PX];
    __shared__ unsigned h_lds[HIST_BINS];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int npx = n_pix * n_pix;
    const int p0 = blockIdx.x * SB_PX, c0 = blockIdx.y * SB_CB;
    const int base = c0 - SB_HALO_L;  // channel of staged row 0
    for (int i = t; i < HIST_BINS; i += 256) h_lds[i] = 0u;
    // wave w loads its own segment of staged rows (one 256-byte row per load, its lane's pixel)
    // into registers, all loads in flight at once, scans it there and writes the prefix sums
    // once, offset by the totals of the segments below (rows outside the band or past the last
    // pixel are zero)
    constexpr int SEG = (SB_ROWS + 3) / 4;
    const int i0 = wave * SEG, i1 = min(SB_ROWS, i0 + SEG);
    const int pp = p0 + lane;
    float v[SEG];
#pragma unroll
    for (int k = 0; k < SEG; k++) {
        const int i = i0 + k, ch = base + i;
        v[k] = (i < i1 && ch >= 0 && ch < n_chan && pp < npx) ? r[(size_t)ch * npx + pp] : 0.f;
    }
    float run = 0.f;
#pragma unroll
    for (int k = 0; k < SEG; k++) {
        run += v[k];
        v[k] = run;
    }
    seg_tot[wave][lane] = run;
    if (t < SB_PX) P[t] = 0.f;
    __syncthreads();
    float off = 0.f;
    for (int k = 0; k < wave; k++) off += seg_tot[k][lane];
#pragma unroll
    for (int k = 0; k < SEG; k++)
        if (i0 + k < i1) P[(i0 + k + 1) * SB_PX + lane] = v[k] + off;
    __syncthreads();
    const int p = p0 + lane;
    const float hist_lo = (float)f32 / (float)HIST_PER_UNIT;  // exact
    const bool pix_ok = p < npx;
    const bool hor = pix_ok && in_horizon(p, n_pix);
    // eight channels at a time: sixteen independent LDS reads per width.  Every index stays
    // inside the staged block whether or not the window fits the band (h <= 64, w - h <= 64), so
    // the reads are unconditional and the band test only masks the result.
    constexpr int CQ = 8;
    float top = -INFINITY;
    for (int j = 0; j < SB_CB / 4; j += CQ) {
        const int cb = c0 + wave * (SB_CB / 4) + j;
        if (cb >= n_chan) break;
        float bs[CQ];
        int bw[CQ];
#pragma unroll
        for (int q = 0; q < CQ; q++) {
            bs[q] = -INFINITY;
            bw[q] = 0;
        }
        // every window of these channels fits the band (h <= 64, w - h <= 64): no band test
        const bool interior = cb >= SB_HALO_L && cb + CQ + SB_HALO_L <= n_chan;
        if (interior) {
            for (int k = 0; k < W.n; k++) {  // widths ascending: the narrower one wins ties
                const int w = W.w[k], h = w >> 1;
                const float inv = W.inv_sqrt[k];
                float v[CQ];
#pragma unroll
                for (int q = 0; q < CQ; q++) {
                    const int is = cb + q - base - h;
                    v[q] = (P[(is + w) * SB_PX + lane] - P[is * SB_PX + lane]) * inv;
                }
#pragma unroll
                for (int q = 0; q < CQ; q++) {
                    if (v[q] > bs[q]) {
                        bs[q] = v[q];
                        bw[q] = w;
                    }
                }
            }
        } else {
            for (int k = 0; k < W.n; k++) {
                const int w = W.w[k], h = w >> 1;
                const float inv = W.inv_sqrt[k];
                float v[CQ];
#pragma unroll
                for (int q = 0; q < CQ; q++) {
                    const int is = cb + q - base - h;
                    v[q] = (P[(is + w) * SB_PX + lane] - P[is * SB_PX + lane]) * inv;
                }
#pragma unroll
                for (int q = 0; q < CQ; q++) {
                    const int c = cb + q;
                    const bool fits = c < n_chan && c - h >= 0 && c - h + w <= n_chan;
                    if (fits && v[q] > bs[q]) {
                        bs[q] = v[q];
                        bw[q] = w;
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < CQ; q++) {
            const int c = cb + q;
            if (c >= n_chan) break;
            if (pix_ok) {
                best[(size_t)c * npx + p] = bs[q];
                wbest[(size_t)c * npx + p] = (uint8_t)bw[q];
            }
            if (hor) top = fmaxf(top, bs[q]);
            if (hor && bs[q] >= hist_lo) atomicAdd(&h_lds[hist_bin(bs[q], f32)], 1u);
        }
    }
    store_tile_max(top, tmax, c0 + wave * SB_TC, n_chan, lane);
    __syncthreads();
    for (int i = t; i < HIST_BINS; i += 256)
        if (h_lds[i]) atomicAdd(&hist[i], h_lds[i]);
}

// ---- the default bank ----
// The same sums, bit for bit, for the default widths, whose window offsets are compile-time
// constants.  A workgroup (64 pixels) marches over blocks of 128 channels; the raw scans of the
// four 64-channel segments of a block (64 below it to 63 above it) stand in an LDS ring, and the
// next block loads only its two new segments, under the current block's sums, so every input is
// read once.  A wave takes its 32 channels in two groups of 16: the 116 prefix sums that all 26
// windows of 16 channels touch (scan + offset of their segment, the general kernel's own sum) are
// read into registers once, and the windows are differences of registers.
// Bound by vector instructions first (per voxel and width a difference, a product and half of a
// three-way maximum; 94 in all, which fill 70% of the issue slots), then by the waits of two
// workgroups per CU (32% of the waves' life); the width of the maximum (a compare and a select more)
// is kept only when the caller wants the width cube.  4,096 x 256^2: 0.90 ms (1.35 with the widths),
// against 2.77 ms for the general kernel, which reads every row twice from memory and 52 prefix sums
// per voxel from LDS.
constexpr int STD_N = 26;
__host__ __device__ constexpr int std_width(int k) {
    constexpr int w[STD_N] = {1,  2,  3,  4,  5,  6,  7,  8,  9,  10, 12, 16, 20,
                              24, 28, 32, 36, 40, 44, 48, 50, 60, 70, 80, 90, 100};
    return w[k];
}
constexpr int STD_HL = std_width(STD_N - 1) / 2;  // 50
// channels per group: 16, or 8 when the widths are kept too (16 spill registers there: 2.50 ms
// against 1.91 for a whole search with cubes)
template <bool WANT_W>
struct StdGroup {
    static constexpr int CQ = WANT_W ? 8 : 16;
    static constexpr int NP = CQ + std_width(STD_N - 1);  // prefix sums its windows touch
};
constexpr int SEG_ROWS = 64;
constexpr unsigned STD_WGS = 4096;  // workgroups a search is cut into (2 per CU run at once)
constexpr size_t WIDTH_VOX = 4096;
constexpr int REFINE_WGS = 4096;    // workgroups of the re-evaluation (they stride over the survivors)
constexpr int FIRST_SURV = 2048;    // survivors copied back with the counts

// Every pixel of a pixel block lies outside the visible hemisphere.
__device__ __forceinline__ bool block_outside(int p0, int n_pix, int lane) {
    const int p = p0 + lane;
    return __ballot(in_horizon(p, n_pix)) == 0ull;
}

template <bool WANT_W>
__global__ __launch_bounds__(256, 2) void search_bank_std_kernel(const float *__restrict__ r, int n_chan, int n_pix,
                                                                 Widths W, int f32, int blocks_per_wg, bool skip_outside,
                                                                 float *__restrict__ best, uint8_t *__restrict__ wbest,
                                                                 unsigned *__restrict__ hist, float *__restrict__ tmax) {
    constexpr int STD_CQ = StdGroup<WANT_W>::CQ, STD_NP = StdGroup<WANT_W>::NP;
    __shared__ float ring[4 * SEG_ROWS * SB_PX];  // slot g % 4 holds the scan of segment g
    __shared__ unsigned h_lds[HIST_BINS];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int npx = n_pix * n_pix;
    const int p0 = blockIdx.x * SB_PX, p = p0 + lane;
    const int b0 = blockIdx.y * blocks_per_wg;
    const int b1 = min((n_chan + SB_CB - 1) / SB_CB, b0 + blocks_per_wg);
    if (skip_outside && block_outside(p0, n_pix, lane)) {  // (uniform over the workgroup)
        for (int b = b0; b < b1; b++) store_tile_max(-INFINITY, tmax, b * SB_CB + wave * SB_TC, n_chan, lane);
        return;
    }
    for (int i = t; i < HIST_BINS; i += 256) h_lds[i] = 0u;
    // segment g holds channels 64 g - 64 .. 64 g - 1; block b uses segments 2 b .. 2 b + 3.  Rows
    // outside the band read the nearest one inside and count as zero (a branch per row, or a
    // pointer per row, would cost more than the sums); every pixel block is whole (n_pix is a
    // multiple of 8).
    float v[SEG_ROWS];
    auto load_seg = [&](int g) __attribute__((always_inline)) {
        const int ch0 = (g - 1) * SEG_ROWS;
#pragma unroll
        for (int k = 0; k < SEG_ROWS; k++) {
            const int ch = min(max(ch0 + k, 0), n_chan - 1);
            v[k] = r[(size_t)ch * npx + p];
        }
    };
    auto store_seg = [&](int g) __attribute__((always_inline)) {
        float *dst = ring + (g & 3) * SEG_ROWS * SB_PX + lane;
        const int ch0 = (g - 1) * SEG_ROWS;
        float run = 0.f;
#pragma unroll
        for (int k = 0; k < SEG_ROWS; k++) {
            run += (unsigned)(ch0 + k) < (unsigned)n_chan ? v[k] : 0.f;
            dst[k * SB_PX] = run;
        }
    };
    load_seg(2 * b0 + wave);
    store_seg(2 * b0 + wave);
    __syncthreads();
    const float hist_lo = (float)f32 / (float)HIST_PER_UNIT;  // exact
    const bool hor = in_horizon(p, n_pix);
    for (int b = b0; b < b1; b++) {
        const int c0 = b * SB_CB;
        // the two new segments of the next block load while this one is searched
        const bool loads = b + 1 < b1 && (wave >> 1) == (b & 1);
        const int g_new = 2 * b + 4 + (wave & 1);
        if (loads) load_seg(g_new);
        // offsets of the block's segments: totals of those before them, in order
        float off[4];
        off[0] = 0.f;
#pragma unroll
        for (int s = 0; s < 3; s++)
            off[s + 1] = off[s] + ring[(((2 * b + s) & 3) * SEG_ROWS + SEG_ROWS - 1) * SB_PX + lane];
        float top = -INFINITY;
#pragma unroll 1
        for (int grp = 0; grp < SB_TC / STD_CQ; grp++) {
            const int o = wave * SB_TC + grp * STD_CQ;  // first channel of the group in the block
            const int cb = c0 + o;
            if (cb >= n_chan) break;
            // P[x] = sum of the block's staged rows below row o + 14 + x (row = channel - c0 + 64)
            float P[STD_NP];
#pragma unroll
            for (int j = 0; j < (STD_NP + 13 + STD_CQ - 1) / STD_CQ; j++) {
                const int row = o + STD_CQ * j, s = row >> 6;  // (these STD_CQ rows lie in one segment)
                const float *src = ring + ((((2 * b + s) & 3) << 6) + (row & 63)) * SB_PX + lane;
                const float of = s == 0 ? off[0] : s == 1 ? off[1] : s == 2 ? off[2] : off[3];
#pragma unroll
                for (int k = 0; k < STD_CQ; k++) {
                    const int x = STD_CQ * j + k - 13;
                    if (x >= 0 && x < STD_NP) P[x] = src[k * SB_PX] + of;
                }
            }
            float bs[STD_CQ];
            int bw[STD_CQ];
#pragma unroll
            for (int q = 0; q < STD_CQ; q++) {
                bs[q] = -INFINITY;
                bw[q] = 0;
            }
            auto value = [&](int k, int q) __attribute__((always_inline)) {
                const int x = STD_HL + q - std_width(k) / 2;
                return (P[x + std_width(k)] - P[x]) * W.inv_sqrt[k];
            };
            const bool interior = cb >= SB_HALO_L && cb + STD_CQ + SB_HALO_L <= n_chan;
            if (interior && !WANT_W) {
#pragma unroll
                for (int k = 0; k < STD_N; k += 2)
#pragma unroll
                    for (int q = 0; q < STD_CQ; q++) bs[q] = fmaxf(fmaxf(bs[q], value(k, q)), value(k + 1, q));
            } else if (interior) {
#pragma unroll
                for (int k = 0; k < STD_N; k++)
#pragma unroll
                    for (int q = 0; q < STD_CQ; q++) {
                        const float x = value(k, q);
                        if (x > bs[q]) {  // widths ascending: the narrower one wins ties
                            bs[q] = x;
                            bw[q] = std_width(k);
                        }
                    }
            } else {
#pragma unroll
                for (int k = 0; k < STD_N; k++) {
                    const int w = std_width(k), h = w >> 1;
#pragma unroll
                    for (int q = 0; q < STD_CQ; q++) {
                        const int c = cb + q;
                        const float x = value(k, q);
                        if (c < n_chan && c - h >= 0 && c - h + w <= n_chan && x > bs[q]) {
                            bs[q] = x;
                            bw[q] = w;
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < STD_CQ; q++) {
                const int c = cb + q;
                if (c < n_chan) {
                    best[(size_t)c * npx + p] = bs[q];
                    if (WANT_W) wbest[(size_t)c * npx + p] = (uint8_t)bw[q];
                    if (hor) top = fmaxf(top, bs[q]);
                    if (hor && bs[q] >= hist_lo) atomicAdd(&h_lds[hist_bin(bs[q], f32)], 1u);
                }
            }
        }
        store_tile_max(top, tmax, c0 + wave * SB_TC, n_chan, lane);
        __syncthreads();  // every wave is done with the segments that the new ones replace
        if (loads) store_seg(g_new);
        __syncthreads();
    }
    for (int i = t; i < HIST_BINS; i += 256)
        if (h_lds[i]) atomicAdd(&hist[i], h_lds[i]);
}

// The width of each listed voxel (S without its width cube): the default bank's sums of that voxel
// again, rounded as the bank rounds them.  One wave per voxel.
__global__ __launch_bounds__(64) void search_width_kernel(const float *__restrict__ r, int n_chan, int n_pix, Widths W,
                                                          Cand *__restrict__ cands, int cap,
                                                          const SearchCounts *__restrict__ cnt) {
    __shared__ float P[4 * SEG_ROWS + 1];
    const int lane = threadIdx.x, n = min(cnt->accepted, cap);
    const size_t npx = (size_t)n_pix * n_pix;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const Cand cd = cands[i];
        const int c0 = cd.c / SB_CB * SB_CB, base = c0 - SB_HALO_L;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const int ch = base + s * SEG_ROWS + lane;
            P[1 + s * SEG_ROWS + lane] = (ch >= 0 && ch < n_chan) ? r[(size_t)ch * npx + cd.p] : 0.f;
        }
        __syncthreads();
        if (lane < 4) {  // a segment each
            float run = 0.f;
            for (int k = 0; k < SEG_ROWS; k++) {
                run += P[1 + lane * SEG_ROWS + k];
                P[1 + lane * SEG_ROWS + k] = run;
            }
        }
        if (lane == 0) P[0] = 0.f;
        __syncthreads();
        const float t0 = P[SEG_ROWS], t1 = P[2 * SEG_ROWS], t2 = P[3 * SEG_ROWS];
        const float off[4] = {0.f, 0.f + t0, (0.f + t0) + t1, ((0.f + t0) + t1) + t2};
        auto prefix = [&](int x) { return x ? P[x] + off[(x - 1) >> 6] : 0.f; };
        float v = -INFINITY;
        int w = 0;
        if (lane < STD_N) {
            const int wk = W.w[lane], h = wk >> 1, is = cd.c - base - h;
            if (cd.c - h >= 0 && cd.c - h + wk <= n_chan) {
                v = (prefix(is + wk) - prefix(is)) * W.inv_sqrt[lane];
                w = wk;
            }
        }
        // widths ascend with the lane: the first lane that holds the (non-NaN) maximum
        float m = v;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        const unsigned long long hit = __ballot(w > 0 && v == m);
        const int first = hit ? (int)__ffsll((long long)hit) - 1 : 0;
        if (lane == first) cands[i].w = hit ? w : 0;
    }
}

// Appends every in-horizon voxel with lo <= S < hi: append(i, channel, pixel, S) with i counted up
// from *counter, one atomic per tile that holds any.  Returns the lane's smallest S taken (NaN: none;
// +inf is a value like any other).  A wave takes tpw <= 64 tiles, reads their maxima and visits the
// tiles that reach lo (a pass over the S cube took 0.30 ms at 4,096 x 256^2; a search's threshold
// lies in a few thousand of its 131,072 tiles).
template <typename F>
__device__ __forceinline__ float append_voxels(const float *__restrict__ best, const float *__restrict__ tmax, int tpw,
                                               int n_chan, int n_pix, float lo, float hi, int *__restrict__ counter,
                                               F append) {
    const int lane = threadIdx.x & 63, npx = n_pix * n_pix;
    const int n_pb = (npx + SB_PX - 1) / SB_PX, n_tiles = n_pb * ((n_chan + SB_TC - 1) / SB_TC);
    const int t0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * tpw;
    const bool have = lane < tpw && t0 + lane < n_tiles;
    unsigned long long todo = __ballot(have && tmax[have ? t0 + lane : 0] >= lo);
    float least = NAN;
    while (todo) {
        const int tile = t0 + (int)__ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const int c0 = tile / n_pb * SB_TC, p = tile % n_pb * SB_PX + lane;
        const bool hor = p < npx && in_horizon(p, n_pix);
        float s[SB_TC];
#pragma unroll
        for (int k = 0; k < SB_TC; k++)
            s[k] = best[(size_t)min(c0 + k, n_chan - 1) * npx + min(p, npx - 1)];
        unsigned mine = 0u;  // the lane's channels that are taken
#pragma unroll
        for (int k = 0; k < SB_TC; k++)
            mine |= (hor && c0 + k < n_chan && s[k] >= lo && !(s[k] >= hi)) ? 1u << k : 0u;
        const int cnt = __popc(mine);
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        const int total = __shfl(incl, 63, 64);
        if (total == 0) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(counter, total);
        at = __shfl(at, 0, 64) + incl - cnt;
#pragma unroll
        for (int k = 0; k < SB_TC; k++) {
            if ((mine >> k) & 1u) {
                append(at++, c0 + k, p, s[k]);
                least = fminf(least, s[k]);
            }
        }
    }
    return least;
}

// SNRs of in-horizon voxels in [lo, hi) (at most cap are written; counter counts all).
__global__ __launch_bounds__(256) void search_gather_kernel(const float *__restrict__ best,
                                                            const float *__restrict__ tmax, int tpw, int n_chan, int n_pix,
                                                            float lo, float hi, float *__restrict__ vals, int cap,
                                                            int *__restrict__ counter) {
    append_voxels(best, tmax, tpw, n_chan, n_pix, lo, hi, counter, [&](int i, int, int, float s) {
        if (i < cap) vals[i] = s;
    });
}

// In-horizon voxels with SNR >= thr (the provisional detections) and the order key of the
// smallest such SNR.  Without a width cube (wbest null) search_width_kernel fills the widths in.
__global__ __launch_bounds__(256) void search_accept_kernel(const float *__restrict__ best,
                                                            const uint8_t *__restrict__ wbest,
                                                            const float *__restrict__ tmax, int tpw, int n_chan, int n_pix,
                                                            float thr, Cand *__restrict__ out, int cap,
                                                            SearchCounts *__restrict__ cnt) {
    const size_t npx = (size_t)n_pix * n_pix;
    // (an infinite S is taken too: nothing lies above the upper bound, NaN)
    float least = append_voxels(best, tmax, tpw, n_chan, n_pix, thr, NAN, &cnt->accepted, [&](int i, int c, int p, float s) {
        if (i < cap) out[i] = Cand{c, p, wbest ? (int)wbest[(size_t)c * npx + p] : 0, s};
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) least = fminf(least, __shfl_xor(least, o, 64));
    if ((threadIdx.x & 63) == 0 && least == least) atomicMin(&cnt->min_key, order_key(least));
}

// Suppression: a provisional detection survives when no other provisional detection (SNR >= thr) at
// its pixel within max(floor(w/2), 1) channels is higher (below: or equal, the lower channel winning
// ties); survivors are appended to surv.  Up to NMS_WAVES detections take a wave each, whose lanes
// read the neighbours at once (one after the other, a thread per detection waited 46 us for them).
// More of them stand so close that the nearest neighbours beat most: a wave then takes up to 64, a
// lane tests its own against the NMS_NEAR nearest on each side, and only what is left is tested by
// the whole wave.  640 x 64^2 with nearly all voxels accepted: 308 us (2 to 16 nearest
// alike), 2,004 with a wave each, 313 with a thread each.
constexpr int NMS_WAVES = 8192, NMS_NEAR = 4;
__global__ __launch_bounds__(64) void search_nms_kernel(const float *__restrict__ best, int n_chan, int n_pix,
                                                        const Cand *__restrict__ cands, int cap, float thr,
                                                        Cand *__restrict__ surv, SearchCounts *__restrict__ cnt) {
    const size_t npx = (size_t)n_pix * n_pix;
    const int lane = threadIdx.x, n = min(cnt->accepted, cap);
    const int per = min(64, (n + (int)gridDim.x - 1) / (int)gridDim.x);  // detections per wave
    auto beaten_at = [&](int c, int p, float s, int d) {
        bool b = false;
        if (c - d >= 0) {
            const float o = best[(size_t)(c - d) * npx + p];
            b = o >= thr && o >= s;
        }
        if (c + d < n_chan) {
            const float o = best[(size_t)(c + d) * npx + p];
            b |= o >= thr && o > s;
        }
        return b;
    };
    for (int64_t base = (int64_t)blockIdx.x * per; base < n; base += (int64_t)gridDim.x * per) {
        const bool have = lane < per && base + lane < n;
        const Cand cd = cands[have ? base + lane : base];
        const int h = max(cd.w >> 1, 1);  // at most NBSI_SEARCH_MAX_WIDTH / 2 = 64 channels each way
        bool lost = !have;
        if (per > 1)
            for (int d = 1; d <= NMS_NEAR; d++)
                if (!lost && d <= h) lost = beaten_at(cd.c, cd.p, cd.s, d);
        unsigned long long todo = __ballot(!lost), won = 0ull;
        while (todo) {
            const int k = (int)__ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int c = __builtin_amdgcn_readlane(cd.c, k), p = __builtin_amdgcn_readlane(cd.p, k);
            const float s = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cd.s), k));
            const int d = lane + 1;
            const bool b = d <= __builtin_amdgcn_readlane(h, k) && beaten_at(c, p, s, d);
            if (__ballot(b) == 0ull) won |= 1ull << k;
        }
        if (!won) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&cnt->survivors, __popcll(won));
        at = __shfl(at, 0, 64);
        if ((won >> lane) & 1ull) surv[at + __popcll(won & ((1ull << lane) - 1ull))] = cd;
    }
}
static_assert(NBSI_SEARCH_MAX_WIDTH / 2 <= 64, "a lane per neighbour");

// Median of vals[0..n) in LDS (mean of the two central order statistics), by counting each
// value's exact rank (ties broken by index); vals holds a multiple of four values, +inf past n.
__device__ float median_lds(const float *vals, int n, float *slot) {
    const int t = threadIdx.x, ka = (n - 1) / 2, kb = n / 2;
    for (int i = t; i < n; i += 256) {
        const float v = vals[i];
        int rank = 0;
        for (int j = 0; j < n; j += 4) {
            const float4 u = *reinterpret_cast<const float4 *>(vals + j);
            rank += (u.x < v || (u.x == v && j < i)) + (u.y < v || (u.y == v && j + 1 < i)) +
                    (u.z < v || (u.z == v && j + 2 < i)) + (u.w < v || (u.w == v && j + 3 < i));
        }
        if (rank == ka) slot[0] = v;
        if (rank == kb) slot[1] = v;
    }
    __syncthreads();
    const float out = 0.5f * (slot[0] + slot[1]);
    __syncthreads();
    return out;
}

// One workgroup per survivor of the suppression: keep[i] = its SNR re-evaluated against its
// flanks reproduces at or above S* (sstar, or the smallest accepted SNR when sstar is NaN).
__global__ __launch_bounds__(256) void search_refine_kernel(const float *__restrict__ r, int n_chan, int n_pix,
                                                            const Cand *__restrict__ cands, float sstar,
                                                            Widths W, int *__restrict__ keep,
                                                            const SearchCounts *__restrict__ cnt) {
    __shared__ __attribute__((aligned(16))) float flank[FLANK_MAX + 4];
    __shared__ __attribute__((aligned(16))) float dev[FLANK_MAX + 4];
    __shared__ float red[256];
    __shared__ float slot[2];
    const int t = threadIdx.x, n_surv = cnt->survivors;
    const int npx = n_pix * n_pix;
    if (sstar != sstar) sstar = key_value(cnt->min_key);
    for (int e = blockIdx.x; e < n_surv; e += gridDim.x) {
        const Cand cd = cands[e];
        // re-evaluation against the flanks outside a guard of w channels on each side
        const int w = cd.w, s0 = cd.c - (w >> 1), g = w, L = max(16, 2 * w);
        const int la = max(0, s0 - g - L), lb = max(0, s0 - g);              // left flank [la, lb)
        const int ra = min(n_chan, s0 + w + g), rb = min(n_chan, s0 + w + g + L);  // right [ra, rb)
        const int nl = max(0, lb - la), nr = max(0, rb - ra), n = nl + nr;
        if (n < REEVAL_MIN_FLANK) {  // (uniform)
            if (t == 0) keep[e] = 0;
            continue;
        }
        __syncthreads();  // (the previous survivor's last reads of the LDS buffers)
        for (int i = t; i < n + 4; i += 256) {
            const int ch = i < nl ? la + i : ra + (i - nl);
            flank[i] = i < n ? r[(size_t)ch * npx + cd.p] : INFINITY;
        }
        __syncthreads();
        const float b = median_lds(flank, n, slot);
        for (int i = t; i < n + 4; i += 256) dev[i] = i < n ? fabsf(flank[i] - b) : INFINITY;
        __syncthreads();
        const float mad = median_lds(dev, n, slot);
        float part = 0.f;
        for (int j = t; j < w; j += 256) part += r[(size_t)(s0 + j) * npx + cd.p] - b;
        red[t] = part;
        __syncthreads();
        for (int sdn = 128; sdn > 0; sdn >>= 1) {
            if (t < sdn) red[t] += red[t + sdn];
            __syncthreads();
        }
        if (t == 0) {
            const float sigma = MAD_TO_SIGMA * mad;
            float sw = sqrtf((float)w);  // (every candidate's width is one of the bank's)
            for (int k = 0; k < W.n; k++)
                if (W.w[k] == w) sw = W.sigma[k];
            const float snr2 = sigma > 0.f ? red[0] / (sw * sigma) : -INFINITY;
            keep[e] = snr2 >= sstar ? 1 : 0;
        }
    }
}

double q_tail(double s) { return 0.5 * erfc(s / sqrt(2.0)); }

}  // namespace

extern "C" int nbsi_search_corr(nbsi_ctx *ctx, const float *snr, int n_chan, int n_pix, const int32_t *widths_host,
                                int n_widths, const double *rho_host, int n_rho, double fdr_q, float *best_snr,
                                uint8_t *best_width, nbsi_cand *out, int max_out, int *n_out, float *thresh_host,
                                int64_t *n_provisional_host) {
    if (!ctx) return NBSI_EINVAL;
    int rc = nbsi_check_detect(n_chan, n_pix, NBSI_DETECT_PER_PIXEL, max_out);
    if (rc) return nbsi_fail(ctx, rc, "nbsi_search: bad shape");
    if (!snr || !n_out || (max_out > 0 && !out)) return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: null pointer");
    if (!aligned16(snr) || (out && !aligned16(out)) || (best_snr && !aligned16(best_snr)) ||
        (best_width && !aligned16(best_width)))
        return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: misaligned pointer");
    if (!(fdr_q > 0.0 && fdr_q < 1.0)) return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: fdr_q must be in (0, 1)");
    if (n_rho < 0 || n_rho > NBSI_SEARCH_MAX_LAG || (n_rho > 0 && !rho_host))
        return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: n_rho out of range or rho missing");
    for (int l = 0; l < n_rho; l++)
        if (!(rho_host[l] > -1.0 && rho_host[l] < 1.0))
            return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: channel correlations must be in (-1, 1)");
    std::vector<int> ws;
    if (widths_host) {
        if (n_widths < 1 || n_widths > NBSI_SEARCH_MAX_WIDTHS)
            return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: n_widths out of range");
        ws.assign(widths_host, widths_host + n_widths);
    } else {
        for (int k = 0; k < STD_N; k++) ws.push_back(std_width(k));
    }
    std::sort(ws.begin(), ws.end());
    ws.erase(std::unique(ws.begin(), ws.end()), ws.end());
    if (ws.front() < 1 || ws.back() > NBSI_SEARCH_MAX_WIDTH)
        return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: widths must be in [1, NBSI_SEARCH_MAX_WIDTH]");
    Widths W{};
    W.n = (int)ws.size();
    for (int k = 0; k < W.n; k++) {
        // variance of the sum of w consecutive unit-variance samples: w + 2 sum_l (w - l) rho_l
        const int w = ws[k];
        double var = (double)w;
        for (int l = 1; l <= std::min(w - 1, n_rho); l++) var += 2.0 * (double)(w - l) * rho_host[l - 1];
        if (!(var > 0.0))
            return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_search: channel correlations give a window sum of no variance");
        W.w[k] = w;
        W.inv_sqrt[k] = (float)(1.0 / sqrt(var));
        W.sigma[k] = (float)sqrt(var);
    }
    // histogram floor F = f32 / 32: a whole bin below Q^-1(q) (q_tail(f32 / 32 + 1 / 32) > q), far
    // beyond erfc's rounding, so every voxel BH can accept is counted
    int kq = -32 * HIST_PER_UNIT;
    while (kq < HIST_SPAN * HIST_PER_UNIT && q_tail((double)(kq + 1) / HIST_PER_UNIT) > fdr_q) kq++;
    const int f32 = kq - 1;
    DeviceGuard g(ctx->device);
    const size_t npx = (size_t)n_pix * n_pix, nvox = (size_t)n_chan * npx;
    // the default bank takes the kernel built for it, and its width cube is made only when wanted
    bool std_bank = W.n == STD_N;
    for (int k = 0; k < W.n && std_bank; k++) std_bank = W.w[k] == std_width(k);
    void *S = best_snr, *Wc = best_width, *hist = nullptr;
    if (!S && (rc = nbsi_scratch(ctx, SLOT_SEARCH_S, sizeof(float) * nvox, &S))) return rc;
    if (!Wc && !std_bank && (rc = nbsi_scratch(ctx, SLOT_SEARCH_W, nvox, &Wc))) return rc;
    const unsigned n_pb = (unsigned)((npx + SB_PX - 1) / SB_PX), n_cb = (unsigned)((n_chan + SB_CB - 1) / SB_CB);
    const size_t n_tiles = (size_t)n_pb * ((n_chan + SB_TC - 1) / SB_TC);
    if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_HIST, sizeof(unsigned) * HIST_BINS + sizeof(float) * n_tiles, &hist))) return rc;
    float *tmax = (float *)((unsigned *)hist + HIST_BINS);
    NBSI_TRY_HIP(ctx, hipMemsetAsync(hist, 0, sizeof(unsigned) * HIST_BINS, ctx->stream));
    auto bank = [&](void *wc) {
        if (!std_bank) {
            hipLaunchKernelGGL(search_bank_kernel, dim3(n_pb, n_cb), dim3(256), 0, ctx->stream, snr, n_chan, n_pix, W, f32,
                               (float *)S, (uint8_t *)wc, (unsigned *)hist, tmax);
            return hipGetLastError();
        }
        // marches long enough to keep the re-read segments few, short enough to fill the chip evenly
        const unsigned cuts = std::min(n_cb, (STD_WGS + n_pb - 1) / n_pb);
        const int per_wg = (int)((n_cb + cuts - 1) / cuts);
        const dim3 grid(n_pb, (n_cb + per_wg - 1) / per_wg);
        const bool skip = !best_snr && !best_width;  // nothing outside the horizon is read later
        if (wc)
            hipLaunchKernelGGL(search_bank_std_kernel<true>, grid, dim3(256), 0, ctx->stream, snr, n_chan, n_pix, W, f32,
                               per_wg, skip, (float *)S, (uint8_t *)wc, (unsigned *)hist, tmax);
        else
            hipLaunchKernelGGL(search_bank_std_kernel<false>, grid, dim3(256), 0, ctx->stream, snr, n_chan, n_pix, W, f32,
                               per_wg, skip, (float *)S, nullptr, (unsigned *)hist, tmax);
        return hipGetLastError();
    };
    NBSI_TRY_HIP(ctx, bank(Wc));
    std::vector<unsigned> h(HIST_BINS);
    NBSI_TRY_HIP(ctx, hipMemcpyAsync(h.data(), hist, sizeof(unsigned) * HIST_BINS, hipMemcpyDeviceToHost, ctx->stream));
    // number of searched voxels: in-horizon pixels x channels (counted while the bank runs)
    int64_t n_hor = 0;
    const int hp = n_pix / 2;
    for (int y = 0; y < n_pix; y++)
        for (int x = 0; x < n_pix; x++) n_hor += ((x - hp) * (x - hp) + (y - hp) * (y - hp) < hp * hp) ? 1 : 0;
    NBSI_TRY_HIP(ctx, hipStreamSynchronize(ctx->stream));

    const double m = (double)n_hor * (double)n_chan;
    std::vector<int64_t> above(HIST_BINS + 1, 0);  // above[j] = #{S >= lower edge of bin j}
    for (int j = HIST_BINS - 1; j >= 0; j--) above[j] = above[j + 1] + h[j];
    auto lo_of = [f32](int j) { return (double)(f32 + j) / HIST_PER_UNIT; };

    // Benjamini-Hochberg: the largest k with p_(k) <= k q / m.  Bins are visited from the lowest
    // SNR (largest k) up; a bin is skipped when even its highest SNR cannot satisfy the rule,
    // accepted whole when its lowest edge already does, and otherwise resolved exactly.
    // tiles per wave of the passes over tiles: waves enough to fill the chip first
    const int tpw = (int)std::max<size_t>(1, std::min<size_t>(64, n_tiles / 16384));
    const unsigned tile_wgs = (unsigned)((n_tiles + 4 * tpw - 1) / (4 * tpw));
    int64_t kstar = 0;
    float thr_acc = INFINITY;  // accept S >= thr_acc
    float sstar = INFINITY;    // the k*-th largest S
    bool exact = false;
    for (int j = 0; j < HIST_BINS && kstar == 0; j++) {
        if (h[j] == 0) continue;
        const int64_t nj = above[j], nj1 = above[j + 1];
        const double lo = lo_of(j), hi = (j == HIST_BINS - 1) ? INFINITY : lo_of(j + 1);
        if (!(q_tail(hi) < (double)nj * fdr_q / m)) continue;
        if (q_tail(lo) <= (double)nj * fdr_q / m) {
            kstar = nj;
            thr_acc = (float)lo;
            break;
        }
        void *vals = nullptr;
        if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_VALS, sizeof(float) * (size_t)h[j], &vals))) return rc;
        NBSI_TRY_HIP(ctx, hipMemsetAsync(ctx->d_counter, 0, sizeof(int), ctx->stream));
        hipLaunchKernelGGL(search_gather_kernel, dim3(tile_wgs), dim3(256), 0, ctx->stream, (const float *)S, tmax, tpw, n_chan, n_pix,
                           (float)lo, j == HIST_BINS - 1 ? INFINITY : (float)hi, (float *)vals, (int)h[j], ctx->d_counter);
        NBSI_TRY_HIP(ctx, hipGetLastError());
        std::vector<float> v(h[j]);
        NBSI_TRY_HIP(ctx, hipMemcpyAsync(v.data(), vals, sizeof(float) * v.size(), hipMemcpyDeviceToHost, ctx->stream));
        NBSI_TRY_HIP(ctx, hipStreamSynchronize(ctx->stream));
        std::sort(v.begin(), v.end(), std::greater<float>());  // k = nj1 + 1 .. nj
        for (int64_t i = (int64_t)v.size() - 1; i >= 0; i--) {
            const int64_t k = nj1 + i + 1;
            if (q_tail((double)v[i]) <= (double)k * fdr_q / m) {
                kstar = k;
                sstar = v[i];
                thr_acc = v[i];
                exact = true;
                break;
            }
        }
    }
    *n_out = 0;
    if (thresh_host) *thresh_host = INFINITY;
    if (n_provisional_host) *n_provisional_host = kstar;
    if (kstar == 0) return NBSI_OK;

    // provisional detections
    const int j_acc = (int)floor((double)thr_acc * HIST_PER_UNIT) - f32;  // the bin holding thr_acc
    const int cap = (int)above[std::min(HIST_BINS - 1, std::max(0, j_acc))];
    void *cands = nullptr, *keep = nullptr;
    if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_CAND, sizeof(Cand) * (size_t)std::max(cap, 1), &cands))) return rc;
    if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_KEEP, sizeof(int) * (size_t)std::max(cap, 1), &keep))) return rc;
    void *surv = nullptr;
    if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_SURV, sizeof(Cand) * (size_t)std::max(cap, 1), &surv))) return rc;
    // no width cube yet: the few provisional detections get their widths one by one (each reads 256
    // channels of its pixel, a line each); more than one in WIDTH_VOX voxels, and the bank makes the cube
    if (!Wc && (size_t)cap > 1024 + nvox / WIDTH_VOX) {
        if ((rc = nbsi_scratch(ctx, SLOT_SEARCH_W, nvox, &Wc))) return rc;
        NBSI_TRY_HIP(ctx, bank(Wc));
    }
    // acceptance, widths, suppression and re-evaluation follow one another on the device's own
    // counts, and the counts come back with the first survivors: one wait
    const SearchCounts init = {0, 0xffffffffu, 0};
    SearchCounts *cnt = (SearchCounts *)ctx->d_counter;
    const unsigned cand_wgs = (unsigned)std::min(std::max(cap, 1), 1 << 16);
    NBSI_TRY_HIP(ctx, hipMemcpyAsync(cnt, &init, sizeof(init), hipMemcpyHostToDevice, ctx->stream));
    hipLaunchKernelGGL(search_accept_kernel, dim3(tile_wgs), dim3(256), 0, ctx->stream, (const float *)S, (const uint8_t *)Wc,
                       tmax, tpw, n_chan, n_pix, thr_acc, (Cand *)cands, cap, cnt);
    NBSI_TRY_HIP(ctx, hipGetLastError());
    if (!Wc) {
        hipLaunchKernelGGL(search_width_kernel, dim3(cand_wgs), dim3(64), 0, ctx->stream, snr, n_chan, n_pix, W,
                           (Cand *)cands, cap, cnt);
        NBSI_TRY_HIP(ctx, hipGetLastError());
    }
    hipLaunchKernelGGL(search_nms_kernel, dim3((unsigned)std::min(std::max(cap, 1), NMS_WAVES)), dim3(64), 0, ctx->stream,
                       (const float *)S, n_chan, n_pix, (const Cand *)cands, cap, thr_acc, (Cand *)surv, cnt);
    NBSI_TRY_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(search_refine_kernel, dim3((unsigned)std::min(std::max(cap, 1), REFINE_WGS)), dim3(256), 0, ctx->stream,
                       snr, n_chan, n_pix, (const Cand *)surv, exact ? sstar : NAN, W, (int *)keep, cnt);
    NBSI_TRY_HIP(ctx, hipGetLastError());
    const int first = std::min(cap, FIRST_SURV);
    std::vector<Cand> hc(first);
    std::vector<int> hk(first);
    SearchCounts got = init;
    NBSI_TRY_HIP(ctx, hipMemcpyAsync(&got, cnt, sizeof(got), hipMemcpyDeviceToHost, ctx->stream));
    NBSI_TRY_HIP(ctx, hipMemcpyAsync(hc.data(), surv, sizeof(Cand) * first, hipMemcpyDeviceToHost, ctx->stream));
    NBSI_TRY_HIP(ctx, hipMemcpyAsync(hk.data(), keep, sizeof(int) * first, hipMemcpyDeviceToHost, ctx->stream));
    NBSI_TRY_HIP(ctx, hipStreamSynchronize(ctx->stream));
    if (got.accepted > cap) return nbsi_fail(ctx, NBSI_EHIP, "nbsi_search: provisional detections exceed the histogram count");
    if (!exact) sstar = key_value(got.min_key);
    if (thresh_host) *thresh_host = sstar;
    const int n_surv = got.survivors;
    hc.resize(n_surv);
    hk.resize(n_surv);
    if (n_surv > first) {
        NBSI_TRY_HIP(ctx, hipMemcpyAsync(hc.data() + first, (const Cand *)surv + first, sizeof(Cand) * (n_surv - first),
                                         hipMemcpyDeviceToHost, ctx->stream));
        NBSI_TRY_HIP(ctx, hipMemcpyAsync(hk.data() + first, (const int *)keep + first, sizeof(int) * (n_surv - first),
                                         hipMemcpyDeviceToHost, ctx->stream));
        NBSI_TRY_HIP(ctx, hipStreamSynchronize(ctx->stream));
    }
    std::vector<nbsi_cand> rec;
    for (int i = 0; i < n_surv; i++)
        if (hk[i]) rec.push_back(nbsi_cand{hc[i].p % n_pix, hc[i].p / n_pix, hc[i].c, hc[i].w, hc[i].s});
    std::sort(rec.begin(), rec.end(), [](const nbsi_cand &a, const nbsi_cand &b) {
        return a.y != b.y ? a.y < b.y : a.x != b.x ? a.x < b.x : a.c < b.c;
    });
    *n_out = (int)rec.size();
    const int n_write = std::min((int)rec.size(), max_out);
    if (n_write > 0) {
        NBSI_TRY_HIP(ctx, hipMemcpyAsync(out, rec.data(), sizeof(nbsi_cand) * n_write, hipMemcpyHostToDevice, ctx->stream));
        NBSI_TRY_HIP(ctx, hipStreamSynchronize(ctx->stream));
    }
    return (int)rec.size() > max_out ? NBSI_ETRUNC : NBSI_OK;
}

extern "C" int nbsi_search(nbsi_ctx *ctx, const float *snr, int n_chan, int n_pix, const int32_t *widths_host,
                           int n_widths, double fdr_q, float *best_snr, uint8_t *best_width, nbsi_cand *out,
                           int max_out, int *n_out, float *thresh_host, int64_t *n_provisional_host) {
    return nbsi_search_corr(ctx, snr, n_chan, n_pix, widths_host, n_widths, nullptr, 0, fdr_q, best_snr, best_width,
                            out, max_out, n_out, thresh_host, n_provisional_host);
}

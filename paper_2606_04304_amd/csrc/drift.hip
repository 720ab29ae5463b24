// Drift-rate search (the paper's Doppler-drift discussion, Sec. 2): residual cubes of S
// sub-integrations of one dump are summed along drifting tracks, c + shift(d, s) in
// sub-integration s with shift(d, s) = round(d s / (S - 1)) (halves away from zero), for every
// total drift d = -D..D channels, as (1 / sqrt(S)) sum_s r_s[c + shift(d, s)]; per voxel the
// largest sum and its drift are kept (trials in the order 0, -1, +1, -2, ... with a strict
// comparison), where the whole track lies in the band.
//
// dedoppler_kernel: a thread owns one pixel (a wave 64 consecutive ones, so every load is one
// 256-byte row) and marches along a segment of channels, CQ at a time, with the window of every
// sub-integration that the drifting tracks of those channels meet held in registers: sub-integration
// s needs channels c - S_s .. c + CQ - 1 + S_s, S_s = shift(D_MAX, s).  A step shifts the windows
// down by CQ registers and appends the channels loaded while the previous step computed, so each
// input value is read once per segment (plus its ends) and the 2D + 1 trials run from registers:
// no LDS, no barriers.  Channels outside the band stand in the windows as -inf, so that tracks which
// leave the band need no test: with a test per trial, the segments at the band's ends set the time
// of every small search (2 x 400 x 48^2, full range: 25.0 us a call; 21.5 with windows in LDS, 13.9
// without the tests).
// Bound by vector instructions (per voxel 33 x (compare, two selects; a multiply where 1 / sqrt(n_sub)
// is not exact) and ~70 additions, partial sums shared by several trials being formed once).
// 4 x 4,096 x 256^2, 33 trials: 1.26 ms (4.5 TB/s of the cubes in and the results out); 2.55 ms when
// the windows stood in LDS (67 reads per voxel, and 1.5x the input through the halos).
#include "internal.h"

#include <algorithm>

namespace {

constexpr int DD_NT = 256;                          // pixels per workgroup
constexpr int D_MAX = NBSI_DEDOPPLER_MAX_DRIFT;
constexpr int DD_SEG_MIN = 16;                      // channels per segment: its ends re-read 2 D_MAX
constexpr int DD_WAVES = 8192;                      // segments are cut until this many waves run

__host__ __device__ constexpr int drift_shift(int d, int s, int n_sub) {
    if (n_sub <= 1 || d == 0 || s == 0) return 0;
    const int ad = d < 0 ? -d : d;
    const int mag = (2 * ad * s + (n_sub - 1)) / (2 * (n_sub - 1));
    return d > 0 ? mag : -mag;
}

// Four channels a step: the windows of eight sub-integrations fit 256 registers, and four
// sub-integrations run three waves per SIMD (eight channels, 177 registers and two waves: 1.47 ms
// against 1.31 at 4 x 4,096 x 256^2, and spills from six sub-integrations on; two channels: 1.37).
template <int NS>
struct Windows {
    static constexpr int CQ = 4;  // channels per step
    // 1 / sqrt(NS) is a power of two: scaling keeps the order of the sums and which of them are
    // equal (above 2^-125), so they are compared unscaled and the best one is scaled
    static constexpr bool EXACT = NS == 1 || NS == 4;
    static constexpr int half(int s) { return drift_shift(D_MAX, s, NS); }
    static constexpr int size(int s) { return CQ + 2 * half(s); }
    static constexpr int off(int s) {  // first register of sub-integration s
        int o = 0;
        for (int k = 0; k < s; k++) o += size(k);
        return o;
    }
    static constexpr int TOTAL = off(NS);
};

template <int NS>
__global__ __launch_bounds__(DD_NT) void dedoppler_kernel(const float *__restrict__ r, int n_chan, int n_pix,
                                                          int max_drift, int seg, float *__restrict__ best,
                                                          int8_t *__restrict__ drift) {
    using W = Windows<NS>;
    constexpr int CQ = W::CQ;
    const size_t npx = (size_t)n_pix * n_pix;
    const size_t p = (size_t)blockIdx.x * DD_NT + threadIdx.x;
    if (p >= npx) return;
    const int c_begin = blockIdx.y * seg, c_end = min(n_chan, c_begin + seg);
    const float *rp = r + p;
    // channels outside the band are -inf: a track that leaves the band (it does so for good, and its
    // last value stands outside) sums to -inf, or to NaN, and neither is greater than any maximum
    auto load = [&](int s, int ch) __attribute__((always_inline)) {  // (ch is uniform)
        return (ch >= 0 && ch < n_chan) ? rp[((size_t)s * n_chan + ch) * npx] : -INFINITY;
    };
    float w[W::TOTAL], nx[NS][CQ];
#pragma unroll
    for (int s = 0; s < NS; s++)
#pragma unroll
        for (int i = 0; i < W::size(s); i++) w[W::off(s) + i] = load(s, c_begin - W::half(s) + i);
    const float inv = NS == 1 ? 1.f : NS == 4 ? 0.5f : rsqrtf((float)NS);
    const int n_trial = 2 * max_drift + 1;
    for (int c = c_begin; c < c_end; c += CQ) {
        if (c + CQ < c_end) {  // the next step's channels load under this one's trials
#pragma unroll
            for (int s = 0; s < NS; s++)
#pragma unroll
                for (int q = 0; q < CQ; q++) nx[s][q] = load(s, c + CQ + W::half(s) + q);
        }
        float bv[CQ];
        int bd[CQ];
        // trial k of channel c + q: drifts 0, -1, +1, -2, +2, ...
        auto trial = [&](int k, int q) __attribute__((always_inline)) {
            const int d = (k == 0) ? 0 : ((k & 1) ? -((k + 1) >> 1) : (k >> 1));
            float acc = 0.f;
#pragma unroll
            for (int s = 0; s < NS; s++) acc += w[W::off(s) + W::half(s) + q + drift_shift(d, s, NS)];
            const float v = W::EXACT ? acc : acc * inv;
            if (v > bv[q]) {
                bv[q] = v;
                bd[q] = d;
            }
        };
#pragma unroll
        for (int q = 0; q < CQ; q++) {
            bv[q] = -INFINITY;
            bd[q] = 0;
        }
        if (max_drift == D_MAX) {
#pragma unroll
            for (int q = 0; q < CQ; q++)
#pragma unroll
                for (int k = 0; k < 2 * D_MAX + 1; k++) trial(k, q);
        } else {
#pragma unroll
            for (int k = 0; k < 2 * D_MAX + 1; k++) {
                if (k < n_trial) {  // (uniform)
#pragma unroll
                    for (int q = 0; q < CQ; q++) trial(k, q);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < CQ; q++) {
            if (c + q < c_end) {
                best[(size_t)(c + q) * npx + p] = W::EXACT ? bv[q] * inv : bv[q];
                drift[(size_t)(c + q) * npx + p] = (int8_t)bd[q];
            }
        }
#pragma unroll
        for (int s = 0; s < NS; s++) {
#pragma unroll
            for (int i = 0; i < 2 * W::half(s); i++) w[W::off(s) + i] = w[W::off(s) + i + CQ];
#pragma unroll
            for (int q = 0; q < CQ; q++) w[W::off(s) + 2 * W::half(s) + q] = nx[s][q];
        }
    }
}

}  // namespace

extern "C" int nbsi_dedoppler(nbsi_ctx *ctx, const float *snr_sub, int n_sub, int n_chan, int n_pix, int max_drift,
                              float *best, int8_t *drift) {
    if (!ctx) return NBSI_EINVAL;
    if (n_sub < 1 || n_sub > NBSI_DEDOPPLER_MAX_SUB || max_drift < 0 || max_drift > NBSI_DEDOPPLER_MAX_DRIFT)
        return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_dedoppler: n_sub or max_drift out of range");
    int rc = nbsi_check_detect(n_chan, n_pix, NBSI_DETECT_PER_PIXEL, 0);
    if (rc) return nbsi_fail(ctx, rc, "nbsi_dedoppler: bad shape");
    if (!snr_sub || !best || !drift) return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_dedoppler: null pointer");
    if (!aligned16(snr_sub) || !aligned16(best) || !aligned16(drift))
        return nbsi_fail(ctx, NBSI_EINVAL, "nbsi_dedoppler: misaligned pointer");
    DeviceGuard g(ctx->device);
    const size_t npx = (size_t)n_pix * n_pix;
    // segments as long as the chip stays full: their ends re-read 2 D_MAX channels
    const size_t px_blocks = (npx + DD_NT - 1) / DD_NT;
    const size_t want = std::max<size_t>(1, DD_WAVES / (DD_NT / 64) / px_blocks);
    const int seg = (int)std::max<size_t>(DD_SEG_MIN, ((((size_t)n_chan + want - 1) / want) + 7) & ~(size_t)7);
    const dim3 grid((unsigned)px_blocks, (unsigned)((n_chan + seg - 1) / seg));
#define NBSI_DD(NS)                                                                                                \
    case NS:                                                                                                       \
        hipLaunchKernelGGL(dedoppler_kernel<NS>, grid, dim3(DD_NT), 0, ctx->stream, snr_sub, n_chan, n_pix,        \
                           max_drift, seg, best, drift);                                                           \
        break;
    switch (n_sub) {
        NBSI_DD(1) NBSI_DD(2) NBSI_DD(3) NBSI_DD(4) NBSI_DD(5) NBSI_DD(6) NBSI_DD(7) NBSI_DD(8)
    }
#undef NBSI_DD
    const hipError_t e = hipGetLastError();
    NBSI_TRY_HIP(ctx, e);
    return NBSI_OK;
}

// Narrowband detection pass over a spectral cube (the paper's Sec. 2.4, Stage I with the
// width-1 matched filter), gfx950.
//
// Per-pixel kernel: a workgroup stages the spectra of PPW neighbouring pixels in LDS (one
// read of the cube), and one wave per pixel computes the exact median and MAD by a wave-local
// selection (sampled brackets checked by exact counts, no atomics and no barriers; see
// wave_select), scores every channel and keeps threshold crossings that survive +-1 channel
// non-maximum suppression (ties keep the lower channel).  Candidates are appended with a
// global atomic counter and sorted afterwards by (y, x, c) with a bitonic network.
//
// Per-image mode first computes each channel image's median and MAD over the visible
// hemisphere (a histogram selection over the image in global memory, one block per channel),
// then runs the per-pixel kernel on the standardised values with only the spectral median
// removed.
#include "internal.h"

namespace {

constexpr float MAD_K = 1.482602218505602f;


__device__ __forceinline__ bool in_horizon(int x, int y, int n) {
    const int h = n / 2, dx = x - h, dy = y - h;
    return dx * dx + dy * dy < h * h;
}

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

__device__ __forceinline__ unsigned wave_min_u(unsigned v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = min(v, (unsigned)__shfl_xor((int)v, d, 64));
    return v;
}

__device__ __forceinline__ float wave_min_f(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = fminf(v, __shfl_xor(v, d, 64));
    return v;
}
__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}

// Bin of x in [lo, hi] split into 256 equal parts: non-decreasing in x, safe for a zero-width range
// (everything in bin 0) and, through the power of two h, for ranges so narrow that 256 over them
// overflows (h = 2^100; lo is below 2^-76 then) or wider than the largest float (h = 1/2).
struct BinMap {
    float lo, h, scale;
    __device__ __forceinline__ BinMap(float lo_, float hi) : lo(lo_) {
        const float range = hi - lo;
        h = range < 0x1p-100f ? 0x1p100f : range < INFINITY ? 1.f : 0.5f;
        scale = 256.f / (hi * h - lo * h);
    }
    __device__ __forceinline__ int operator()(float x) const {
        const float t = fmaf(x, h, -(lo * h)) * scale;
        return t >= 256.f ? 255 : (t > 0.f ? (int)t : 0);
    }
};

// Block-wide sum / min / max over SEL_NT threads through `red` (SEL_NT / 64 slots of LDS); every
// thread gets the result.  Callers keep the calls uniform across the block.
constexpr int SEL_NT = 1024;
constexpr int SEL_NW = SEL_NT / 64;
constexpr int SEL_POOL = 1024;

__device__ __forceinline__ int block_sum(int v, int *red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int q = 0; q < SEL_NW; q++) s += red[q];
    return s;
}
__device__ __forceinline__ float block_min_f(float v, float *red) {
    v = wave_min_f(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float s = INFINITY;
#pragma unroll
    for (int q = 0; q < SEL_NW; q++) s = fminf(s, red[q]);
    return s;
}
// Mean over the waves of a wave-uniform value, in wave order (waves with ok false take no part;
// none when no wave does).
__device__ __forceinline__ float block_mean_f(float v, bool ok, float none, float *red, int *ired) {
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        red[w] = ok ? v : 0.f;
        ired[w] = ok;
    }
    __syncthreads();
    float s = 0.f;
    int n = 0;
#pragma unroll
    for (int q = 0; q < SEL_NW; q++) {
        s += red[q];
        n += ired[q];
    }
    return n ? s / (float)n : none;
}
__device__ __forceinline__ float block_max_f(float v, float *red) {
    v = wave_max_f(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    float s = -INFINITY;
#pragma unroll
    for (int q = 0; q < SEL_NW; q++) s = fmaxf(s, red[q]);
    return s;
}

// LDS of one block selection
struct SelLds {
    unsigned hist[4][256];  // four copies (by wave % 4) against atomic contention
    float pool[SEL_POOL];
    int ired[SEL_NW];
    float fred[SEL_NW];
    int sel[4];             // selected bin, values below it, values in it, pool fill
    float res, res_next;    // the selected value and the next one up
};

// Ascending bitonic sort of one value per lane across the wave (64 values).
__device__ __forceinline__ float wave_sort64(float v, int lane) {
#pragma unroll
    for (int size = 2; size <= 64; size <<= 1)
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const float o = __shfl_xor(v, stride, 64);
            const bool keep_min = ((lane & stride) == 0) == ((lane & size) == 0);
            v = keep_min ? fminf(v, o) : fmaxf(v, o);
        }
    return v;
}

// The next float above / below a finite x (the bracket bounds around a dropped pivot value).
__device__ __forceinline__ float float_up(float x) {
    if (x == 0.f) return __int_as_float(1);  // smallest positive denormal
    const int b = __float_as_int(x);
    return __int_as_float(x > 0.f ? b + 1 : b - 1);
}
__device__ __forceinline__ float float_down(float x) { return -float_up(-x); }

// The rank-th smallest (0-based) of the values a block of SEL_NT threads enumerates, and the next
// one up when it was seen (have_hi): each(f) calls f on every value the calling thread owns, and on
// NaN, which counts for nothing.  [a, b] is a proposal for the rank's place.  One pass counts the
// values below a exactly and bins those inside [a, b], spread over 256 bins; the next gathers the
// bin that holds the rank (ranked exactly by comparing all its values) or, when more than SEL_POOL
// values share it, narrows [a, b] to its smallest and largest value.  A proposal that missed the
// rank is replaced by the whole side the rank lies on, so the loop ends.
template <typename Each>
__device__ __forceinline__ float block_select(Each each, float a, float b, int rank, SelLds &L, float &vhi,
                                              bool &have_hi) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    float vlo = a;
    vhi = 0.f;
    have_hi = false;
    for (int iter = 0; iter < 64; iter++) {
        const BinMap bin(a, b);
        for (int e = t; e < 4 * 256; e += SEL_NT) (&L.hist[0][0])[e] = 0;
        __syncthreads();
        int below = 0;
        each([&](float x) __attribute__((always_inline)) {
            below += x < a;
            if (x >= a && x <= b) atomicAdd(&L.hist[w & 3][bin(x)], 1u);
        });
        below = block_sum(below, L.ired);  // (its barriers also order the histogram)
        const int k = rank - below;
        // threads 0..255 own one bin each (waves 0..3)
        int cnt = 0, incl = 0;
        if (t < 256) {
            cnt = (int)(L.hist[0][t] + L.hist[1][t] + L.hist[2][t] + L.hist[3][t]);
            incl = wave_inclusive_scan(cnt, lane);
        }
        __syncthreads();
        if (t < 256 && lane == 63) L.ired[w] = incl;
        if (t == 0) {
            L.sel[0] = -1;  // no bin holds the rank
            L.sel[3] = 0;
        }
        __syncthreads();
        if (t < 256) {
            for (int q = 0; q < w; q++) incl += L.ired[q];
            if (incl - cnt <= k && k < incl) {
                L.sel[0] = t;
                L.sel[1] = incl - cnt;
                L.sel[2] = cnt;
            }
        }
        __syncthreads();
        const int bsel = L.sel[0], kb = k - L.sel[1], in_bin = L.sel[2];
        const bool found = bsel >= 0, pool = found && in_bin <= SEL_POOL;
        if (found && a == b) {  // in_bin values equal a
            vlo = vhi = a;
            have_hi = kb + 1 < in_bin;
            break;
        }
        // the values of the bin, into the pool or as their smallest and largest; without a bin, the
        // smallest and largest of all values
        float nlo = INFINITY, nhi = -INFINITY;
        each([&](float x) __attribute__((always_inline)) {
            if (!found || (x >= a && x <= b && bin(x) == bsel)) {
                if (pool) {
                    L.pool[atomicAdd(&L.sel[3], 1)] = x;
                } else {
                    nlo = fminf(nlo, x);
                    nhi = fmaxf(nhi, x);
                }
            }
        });
        if (pool) {
            __syncthreads();
            for (int e = t; e < in_bin; e += SEL_NT) {
                const float v = L.pool[e];
                int less = 0, eq = 0;
                for (int j = 0; j < in_bin; j++) {
                    const float y = L.pool[j];
                    less += y < v;
                    eq += y == v;
                }
                if (less <= kb && kb < less + eq) L.res = v;  // every writer writes the same value
                if (less <= kb + 1 && kb + 1 < less + eq) L.res_next = v;
            }
            __syncthreads();
            vlo = L.res;
            vhi = L.res_next;
            have_hi = kb + 1 < in_bin;
            break;
        }
        nlo = block_min_f(nlo, L.fred);
        nhi = block_max_f(nhi, L.fred);
        if (found) {
            a = nlo;
            b = nhi;
        } else if (k < 0) {  // below a
            b = float_down(a);
            a = nlo;
        } else {
            a = float_up(b);
            b = nhi;
        }
        vlo = a;
    }
    __syncthreads();  // (the results have been read)
    return vlo;
}

// Median of the n values of a block (mean of the central pair for even n; exact order statistics).
// smp is one of the thread's values (NaN: none).  Every wave sorts its 64 samples and proposes the
// ones a few places either side of the rank's expected place; their means over the waves bracket
// the rank among about a tenth of the values (no samples at all: every finite value).  compact(a, b, below) lists the values inside [a, b]
// in LDS, per wave and without atomics, and counts those below a: one pass over all values, after
// which the selection runs over the listed ones (list(f)).  It returns how many it listed, or -1
// when it could not; then, or when the bracket missed the rank, the selection runs over all values.
template <typename Each, typename Compact, typename List>
__device__ __forceinline__ float block_median(Each each, Compact compact, List list, float smp, int n, SelLds &L) {
    constexpr int D = 4;
    const int lane = threadIdx.x & 63;
    const int rank = (n - 1) / 2;
    smp = smp == smp ? smp : INFINITY;
    const float srt = wave_sort64(smp, lane);
    const int s_n = __popcll(__ballot(smp < INFINITY));
    const int p = (int)(((long long)rank * s_n) / n);
    const float pa = __shfl(srt, max(p - D, 0), 64), pb = __shfl(srt, min(p + D, max(s_n - 1, 0)), 64);
    const float a = block_mean_f(pa, s_n > 0, -__FLT_MAX__, L.fred, L.ired);
    const float b = block_mean_f(pb, s_n > 0, __FLT_MAX__, L.fred, L.ired);
    int below = 0;
    const int n_in = compact(a, b, below);
    float vhi;
    bool have_hi;
    const float vlo = (rank >= below && rank < below + n_in) ? block_select(list, a, b, rank - below, L, vhi, have_hi)
                                                             : block_select(each, a, b, rank, L, vhi, have_hi);
    if (n & 1) return vlo;
    if (have_hi) return 0.5f * (vlo + vhi);
    // rank n / 2: vlo itself when more than n / 2 values are <= vlo, else the next larger value
    int le = 0;
    float nxt = INFINITY;
    each([&](float x) __attribute__((always_inline)) {
        le += x <= vlo;
        nxt = fminf(nxt, x > vlo ? x : INFINITY);
    });
    le = block_sum(le, L.ired);
    nxt = block_min_f(nxt, L.fred);
    vhi = (le >= n / 2 + 1) ? vlo : nxt;
    return 0.5f * (vlo + vhi);
}

// A wave-uniform value moved to a scalar register (frees vector registers in the selection loops).
__device__ __forceinline__ float uniform_f(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ int uniform_i(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Pseudo-random 32-bit hash of (i, round), for reservoir sampling.
__device__ __forceinline__ unsigned mix_hash(unsigned i, unsigned round) {
    unsigned h = i * 0x9E3779B1u + round * 0x85EBCA77u;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    return h;
}

// The rank-th smallest (0-based) of val(i), i < n (finite values), for one wave, without
// atomics or barriers.  The wave keeps a bracket [lo, hi] of values known to hold the answer,
// with c_lt values below it and c_le values at or below its top (c_lt <= rank < c_le).  Each
// round sorts a sample of in-bracket values (one per lane, drawn from the entries l, l + 64, ...),
// takes the sample values D places either side of the rank's expected place as a candidate
// [a, b] (a single pivot value when the bracket did not shrink last round), and counts the data
// below a and at or below b: the rank then lies below a, in [a, b] or above b, and the bracket
// becomes that part.  The counting pass also keeps the first value of the lane's entries in
// [a, b], the next sample when the rank is there (the usual case); otherwise, and from round
// RESAMPLE_FROM on, a separate pass draws a uniform in-bracket sample by reservoir sampling,
// which keeps sorted or trending data from skewing the sample.  A pivot round always removes
// the pivot, so the loop ends; noise-like spectra need 3-4 rounds.  At most 64 values are left in
// the bracket then; they are gathered into `pool` (64 floats) and ranked exactly.
template <typename ValFn>
__device__ float wave_select(ValFn val, int n, int rank, float *pool, int lane) {
    constexpr int D = 8, RESAMPLE_FROM = 4;
    float lo = -INFINITY, hi = INFINITY;
    int c_lt = 0, c_le = n;
    float smp = lane < n ? val(lane) : INFINITY;  // this lane's sample of the bracket (+inf: none)
    bool pivot = false, resample = false;
    for (int round = 0; round < 2 * n + 2; round++) {
        const int m = c_le - c_lt;
        if (m <= 64 || lo == hi) break;
        if (resample || round >= RESAMPLE_FROM) {
            // uniform in-bracket value of this lane's entries (reservoir sampling)
            smp = INFINITY;
            int k = 0;
            for (int i = lane; i < n; i += 64) {
                const float x = val(i);
                if (x >= lo && x <= hi) {
                    k++;
                    if ((mix_hash((unsigned)i, (unsigned)round) >> 20) * (unsigned)k < 4096u) smp = x;
                }
            }
        }
        const float srt = wave_sort64(smp, lane);
        const int s_n = wave_sum(smp < INFINITY ? 1 : 0);  // >= 1: m > 64 values over 64 lanes
        const int p = min(s_n - 1, (int)(((long long)(rank - c_lt) * s_n) / m));
        float a, b;
        if (pivot) {
            a = b = __shfl(srt, p, 64);
        } else {
            a = p - D >= 0 ? __shfl(srt, p - D, 64) : lo;
            b = p + D < s_n ? __shfl(srt, p + D, 64) : hi;
            if (a == lo && b == hi) a = b = __shfl(srt, p, 64);
        }
        int n_lt = 0, n_le = 0;
        float s_in = INFINITY;
        for (int i = lane; i < n; i += 64) {
            const float x = val(i);
            n_lt += x < a;
            n_le += x <= b;
            s_in = (s_in == INFINITY && x >= a && x <= b) ? x : s_in;
        }
        n_lt = wave_sum(n_lt);
        n_le = wave_sum(n_le);
        resample = true;
        if (rank < n_lt) {  // below a
            hi = float_down(a);
            c_le = n_lt;
        } else if (rank >= n_le) {  // above b
            lo = float_up(b);
            c_lt = n_le;
        } else {  // in [a, b]
            if (a == b) return a;
            lo = a;
            hi = b;
            c_lt = n_lt;
            c_le = n_le;
            smp = s_in;
            resample = false;
        }
        pivot = c_le - c_lt == m;  // nothing left the bracket: split at a pivot next round
    }
    if (lo == hi) return lo;
    // at most 64 values in [lo, hi]: gather them and rank exactly
    int base = 0;
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        float x = 0.f;
        bool in = false;
        if (i < n) {
            x = val(i);
            in = x >= lo && x <= hi;
        }
        const unsigned long long bm = __ballot(in);
        if (in) pool[base + __popcll(bm & ((1ull << lane) - 1ull))] = x;
        base += __popcll(bm);
    }
    const int m = base;
    const int k = rank - c_lt;
    float mine = 0.f;
    bool hit = false;
    if (lane < m) {
        mine = pool[lane];
        int less = 0, eq = 0;
        for (int j = 0; j < m; j++) {
            const float y = pool[j];
            less += y < mine;
            eq += y == mine;
        }
        hit = less <= k && k < less + eq;
    }
    const unsigned long long hb = __ballot(hit);
    return __shfl(mine, hb ? (int)(__ffsll((long long)hb) - 1) : 0, 64);
}

// Median of val(i), i < n (finite values; mean of the central pair for even n), wave-local.
template <typename ValFn>
__device__ float wave_median_fast(ValFn val, int n, float *pool, int lane) {
    const float vlo = wave_select(val, n, (n - 1) / 2, pool, lane);
    if (n & 1) return vlo;
    int le = 0;
    float nxt = INFINITY;
    for (int i = lane; i < n; i += 64) {
        const float x = val(i);
        le += x <= vlo;
        if (x > vlo) nxt = fminf(nxt, x);
    }
    le = wave_sum(le);
    nxt = wave_min_f(nxt);
    const float vhi = (le >= n / 2 + 1) ? vlo : nxt;
    return 0.5f * (vlo + vhi);
}

// ---- spectra held in registers (n_chan <= 64 NR) ----
// Lane l of a wave holds channels l + 64 j, j < NR, of its pixel in v[j] (NaN past n_chan, which
// every comparison below treats as false).  The same algorithm as wave_select, with every pass
// over registers instead of LDS; a pass costs two compares and a select per held value on the
// vector unit, while the counts (popcounts of the compare masks) run on the scalar unit.
// The rank-th smallest held value, and the next one up when the last bracket shows it (NaN
// otherwise), for held values that are finite or NaN (NaN is never counted).
template <int NR>
__device__ float2 reg_select(const float (&v)[NR], int n, int rank, float *pool, int lane) {
    constexpr int D = 8, RESAMPLE_FROM = 4;
    float lo = -INFINITY, hi = INFINITY;
    int c_lt = 0, c_le = n;
    // first sample: lane l holds channel l + 64 (l mod NR), spread over the band (NaN past n);
    // the lanes that take register j form a constant mask
    float smp = INFINITY;
#pragma unroll
    for (int j = 0; j < NR; j++) {
        unsigned long long lanes_j = 0ull;
#pragma unroll
        for (int l = j % 64; l < 64; l += NR) lanes_j |= 1ull << l;
        smp = __builtin_amdgcn_inverse_ballot_w64(lanes_j) ? v[j] : smp;
    }
    smp = smp == smp ? smp : INFINITY;
    bool pivot = false, resample = false;
    for (int round = 0; round < 2 * n + 2; round++) {
        const int m = c_le - c_lt;
        if (m <= 64 || lo == hi) break;
        if (resample || round >= RESAMPLE_FROM) {
            smp = INFINITY;
            int k = 0;
#pragma unroll
            for (int j = 0; j < NR; j++) {
                const float x = v[j];
                if (x >= lo && x <= hi) {
                    k++;
                    if ((mix_hash((unsigned)(lane + 64 * j), (unsigned)round) >> 20) * (unsigned)k < 4096u) smp = x;
                }
            }
        }
        const float srt = wave_sort64(smp, lane);
        const int s_n = __popcll(__ballot(smp < INFINITY));
        const int p = min(s_n - 1, (int)(((long long)(rank - c_lt) * s_n) / m));
        float a, b;
        if (pivot) {
            a = b = __shfl(srt, p, 64);
        } else {
            a = p - D >= 0 ? __shfl(srt, p - D, 64) : lo;
            b = p + D < s_n ? __shfl(srt, p + D, 64) : hi;
            if (a == lo && b == hi) a = b = __shfl(srt, p, 64);
        }
        a = uniform_f(a);
        b = uniform_f(b);
        // count below a and at or below b (popcounts of the compare masks, on the scalar unit);
        // keep each lane's last held value in [a, b] (selected by the mask le & ~lt)
        int n_lt = 0, n_le = 0;
        float s_in = INFINITY;
#pragma unroll
        for (int j = 0; j < NR; j++) {
            const float x = v[j];
            const unsigned long long m_lt = __ballot(x < a), m_le = __ballot(x <= b);
            n_lt += __popcll(m_lt);
            n_le += __popcll(m_le);
            s_in = __builtin_amdgcn_inverse_ballot_w64(m_le & ~m_lt) ? x : s_in;
            // (an empty asm that takes s_in makes each select happen here: left alone, the
            // compiler defers the select chain and keeps every value's masks alive)
            asm volatile("" : "+v"(s_in));
        }
        // (the next sample is chosen before branching: were s_in needed on one path only, the
        // compiler would sink its selects there and keep every pass mask alive until then)
        const bool inside = rank >= n_lt && rank < n_le;
        smp = inside ? s_in : smp;
        resample = !inside;
        if (rank < n_lt) {
            hi = float_down(a);
            c_le = n_lt;
        } else if (rank >= n_le) {
            lo = float_up(b);
            c_lt = n_le;
        } else {
            if (a == b) return make_float2(a, rank + 1 < n_le ? a : NAN);
            lo = a;
            hi = b;
            c_lt = n_lt;
            c_le = n_le;
        }
        pivot = c_le - c_lt == m;
    }
    if (lo == hi) return make_float2(lo, rank + 1 < c_le ? lo : NAN);
    // at most 64 values remain in [lo, hi]: gathered one per lane through `pool`, sorted across
    // the wave, and read at the rank (and the next place, when it is in the bracket)
    int base = 0;
#pragma unroll
    for (int j = 0; j < NR; j++) {
        const float x = v[j];
        const bool in = x >= lo && x <= hi;
        const unsigned long long bm = __ballot(in);
        if (bm == 0ull) continue;  // (most registers hold none of them)
        if (in) pool[base + __popcll(bm & ((1ull << lane) - 1ull))] = x;
        base += __popcll(bm);
    }
    const int m = base;
    const float srt = wave_sort64(lane < m ? pool[lane] : INFINITY, lane);
    const int k = rank - c_lt;
    const float vk = __shfl(srt, k, 64), vk1 = __shfl(srt, min(k + 1, 63), 64);
    return make_float2(vk, k + 1 < m ? vk1 : NAN);
}

template <int NR>
__device__ float reg_median(const float (&v)[NR], int n, float *pool, int lane) {
    const float2 r = reg_select<NR>(v, n, (n - 1) / 2, pool, lane);
    if (n & 1) return r.x;
    float vhi = r.y;
    if (vhi != vhi) {  // the upper middle value was not in the last bracket: one more pass
        int le = 0;
        float nxt = INFINITY;
#pragma unroll
        for (int j = 0; j < NR; j++) {
            const float x = v[j];
            le += __popcll(__ballot(x <= r.x));
            nxt = fminf(nxt, x > r.x ? x : INFINITY);
        }
        nxt = wave_min_f(nxt);
        vhi = (le >= n / 2 + 1) ? r.x : nxt;
    }
    return 0.5f * (r.x + vhi);
}

// Per-pixel detection for spectra of up to 64 NR channels: a workgroup of REG_PX waves takes
// REG_PX adjacent pixels of one row; each staging round loads 1,024 channels x REG_PX pixels
// (4 REG_PX contiguous bytes per channel row) through an LDS tile, and every wave keeps its
// pixel's spectrum in registers, so the selections and the scoring run without LDS or barriers.
// Four-wave workgroups (four per CU at 128 registers, so staging reads run under other
// workgroups' selections) free their slot as soon as their slowest pixel is done: the rounds a
// selection needs vary from pixel to pixel, and eight-wave workgroups, which wait for the
// slowest of eight, were 5% slower (sixteen-wave ones 17%).
constexpr int REG_PX = 4;
constexpr int REG_LINE = 128 / (4 * REG_PX);  // workgroups that share a 128-byte line of a row
template <int NR>
__global__ __launch_bounds__(64 * REG_PX, 4) void detect_pixel_reg_kernel(const float *__restrict__ img, int n_chan, int n_pix,
                                                                int mode, const float2 *__restrict__ stats,
                                                                float thresh, float *__restrict__ pix_stats,
                                                                nbsi_cand *__restrict__ cand, int cap,
                                                                int *__restrict__ counter, unsigned *__restrict__ flags) {
    constexpr int CH = 1024;              // channels per staging round (16 registers)
    constexpr int TPC = REG_PX / 4;       // threads per channel row segment (16 bytes each)
    constexpr int CPS = 64 * REG_PX / TPC;  // channels per load step (256)
    static_assert(NR % (CH / 64) == 0 && CH % CPS == 0, "staging rounds");
    __shared__ float tile[CH][REG_PX + 1];
    __shared__ float pool_all[REG_PX][64];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int groups_per_row = n_pix / REG_PX;
    // XCD-aware order: workgroups are dealt to the 8 XCDs round robin, so the REG_LINE groups
    // that split each 128-byte line of a channel row go to blocks b, b + 8, ... of one XCD,
    // which run together and share the line in that XCD's L2
    constexpr int RUN = 8 * REG_LINE;
    const int nbr = (int)gridDim.x / RUN * RUN, b = blockIdx.x;
    const int grp = b < nbr ? (b / RUN) * RUN + (b & 7) * REG_LINE + ((b >> 3) % REG_LINE) : b;
    const int gy = grp / groups_per_row, gx0 = (grp % groups_per_row) * REG_PX;
    const size_t npix2 = (size_t)n_pix * n_pix;
    // staging: thread t loads pixels sp .. sp + 3 (16 bytes; n_pix is a multiple of 8) of
    // channels sc + CPS q
    const int sp = 4 * (t % TPC), sc = t / TPC;
    const float *src = img + (size_t)gy * n_pix + gx0 + sp;
    // the loads of round k + 1 are issued before round k's tile is read back, so they are in
    // flight across its barrier
    auto load = [&](int k, float4 (&r)[CH / CPS]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < CH / CPS; q++) {
            const int c = k * CH + sc + CPS * q;
            r[q] = c < n_chan ? *reinterpret_cast<const float4 *>(src + (size_t)c * npix2)
                                          : make_float4(NAN, NAN, NAN, NAN);
        }
    };
    float v[NR];
    float4 r[CH / CPS];
    // pixels of the workgroup whose spectrum holds a non-finite value (bit = pixel), gathered
    // while staging
    __shared__ unsigned s_bad;
    if (t == 0) s_bad = 0u;
    load(0, r);
#pragma unroll
    for (int k = 0; k < NR / (CH / 64); k++) {
        __syncthreads();  // the previous round's tile has been read (and s_bad is cleared)
        unsigned bad_px = 0u;
#pragma unroll
        for (int q = 0; q < CH / CPS; q++) {
            const int c = k * CH + sc + CPS * q;
            float e[4] = {r[q].x, r[q].y, r[q].z, r[q].w};
            if (mode == NBSI_DETECT_PER_IMAGE && c < n_chan) {
                const float2 st = stats[c];
#pragma unroll
                for (int i = 0; i < 4; i++)  // (x * 0: non-finite stays non-finite)
                    e[i] = st.y > 0.f ? (e[i] - st.x) / st.y : e[i] * 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; i++) {
                tile[sc + CPS * q][sp + i] = e[i];
                if (c < n_chan && !__builtin_isfinite(e[i])) bad_px |= 1u << (sp + i);
            }
        }
        if (bad_px) atomicOr(&s_bad, bad_px);
        if (k + 1 < NR / (CH / 64)) load(k + 1, r);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CH / 64; q++) v[(CH / 64) * k + q] = tile[lane + 64 * q][wave];
    }
    const int x = gx0 + wave, y = gy;
    // (n_pix is a multiple of REG_PX: every wave has a pixel)
    // a spectrum holding a non-finite value is not searched (wave-uniform: one pixel per wave)
    const bool finite = ((s_bad >> wave) & 1u) == 0u;
    const bool in_hor = in_horizon(x, y, n_pix);
    if (in_hor && !finite && lane == 0 && flags) atomicOr(flags, NBSI_FLAG_CUBE_NONFINITE);
    const bool active = in_hor && finite;
    float *pool = pool_all[wave];
    float scale = 1.f, med = 0.f;
    bool ok = active;
    if (active) {
        med = reg_median<NR>(v, n_chan, pool, lane);
        // the deviations x - med replace the values (rounded as the score rounds them); for the
        // MAD their magnitudes, with the signs kept in a bit mask, so that both selections rank
        // values held in registers (a rank over |x - med| computed on the fly has the compiler
        // hoist all NR of them out of the selection rounds and spill)
        unsigned long long neg = 0ull;
#pragma unroll
        for (int j = 0; j < NR; j++) {
            const float d = v[j] - med;
            neg |= (unsigned long long)(d < 0.f) << j;
            v[j] = fabsf(d);  // (NaN past n_chan stays NaN)
        }
        if (mode == NBSI_DETECT_PER_PIXEL) {
            const float mad = reg_median<NR>(v, n_chan, pool, lane);
            scale = MAD_K * mad;
            ok = mad > 0.f;
        }
#pragma unroll
        for (int j = 0; j < NR; j++) v[j] = ((neg >> j) & 1ull) ? -v[j] : v[j];
    }
    // SNR = (x - med) / scale as a product with the float32 reciprocal; neighbours along
    // frequency come from the adjacent lane (channel c +- 1), across register rows at lanes 0/63
    const float inv = ok ? 1.f / scale : 0.f;
#pragma unroll
    for (int j = 0; j < NR; j++) {
        const int c = lane + 64 * j;
        const float xv = v[j];  // x - med
        const float z = ok ? xv * inv : 0.f;
        const bool hit = ok && c < n_chan && z >= thresh;
        // the neighbours are fetched (with every lane taking part) only when a lane crosses
        if (__ballot(hit) == 0ull) continue;
        const float up = __shfl_up(xv, 1, 64), dn = __shfl_down(xv, 1, 64);
        const float prev_row = j > 0 ? __shfl(v[j > 0 ? j - 1 : 0], 63, 64) : 0.f;
        const float next_row = j + 1 < NR ? __shfl(v[j + 1 < NR ? j + 1 : j], 0, 64) : 0.f;
        if (!hit) continue;
        const float xl = lane > 0 ? up : prev_row, xr = lane < 63 ? dn : next_row;
        if (c > 0 && !(z > xl * inv)) continue;
        if (c + 1 < n_chan && !(z >= xr * inv)) continue;
        const int idx = atomicAdd(counter, 1);
        if (idx < cap) {
            nbsi_cand r;
            r.x = x;
            r.y = y;
            r.c = c;
            r.width = 1;
            r.snr = z;
            cand[idx] = r;
        }
    }
    // the pixel's median and scale, for snr_cube_kernel (inv = 0: not searched)
    if (pix_stats && lane == 0) {
        pix_stats[(size_t)gy * n_pix + x] = ok ? med : 0.f;
        pix_stats[npix2 + (size_t)gy * n_pix + x] = inv;
    }
}

// The SNR cube from the medians and scales of detect_pixel_reg_kernel (two planes of n_pix^2; without
// room for them they stand in the cube's own first two planes): channels c0 .. n_chan - 1, a thread takes 4
// adjacent pixels of SNR_CPB channels (all loads in flight) with 16-byte accesses.  Bound by HBM (8
// bytes per voxel).  The pixel kernel cannot write the cube well itself: it holds 4 pixels x all
// channels, and 16-byte pieces of 128-byte lines leave its eight line-sharing workgroups at different
// times (4,096 x 256^2, whole call: 3.25 ms with 4-byte stores from the lanes, 1.57 ms with 16-byte
// ones through the tile, 1.22 ms with the two kernels, of which this one takes 0.35; 0.36 with eight
// channels a thread).
constexpr int SNR_CPB = 4;
__global__ __launch_bounds__(256) void snr_cube_kernel(const float *__restrict__ img, int n_chan, int n_pix, int mode,
                                                       const float2 *__restrict__ stats, const float *pix_stats, int c0,
                                                       float *snr) {
    const size_t npix2 = (size_t)n_pix * n_pix;
    const size_t p = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (p >= npix2) return;
    const int cb = c0 + blockIdx.y * SNR_CPB;
    const float4 med = *reinterpret_cast<const float4 *>(pix_stats + p);
    const float4 inv = *reinterpret_cast<const float4 *>(pix_stats + npix2 + p);
    float4 x[SNR_CPB];
#pragma unroll
    for (int q = 0; q < SNR_CPB; q++)
        if (cb + q < n_chan) x[q] = *reinterpret_cast<const float4 *>(img + (size_t)(cb + q) * npix2 + p);
#pragma unroll
    for (int q = 0; q < SNR_CPB; q++) {
        const int c = cb + q;
        if (c >= n_chan) break;
        float e[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
        const float m[4] = {med.x, med.y, med.z, med.w}, s[4] = {inv.x, inv.y, inv.z, inv.w};
        if (mode == NBSI_DETECT_PER_IMAGE) {  // the same standardised value the pixel kernel staged
            const float2 st = stats[c];
#pragma unroll
            for (int i = 0; i < 4; i++) e[i] = st.y > 0.f ? (e[i] - st.x) / st.y : e[i] * 0.f;
        }
        // (a pixel that is not searched may hold non-finite values; + 0: no negative zeros)
#pragma unroll
        for (int i = 0; i < 4; i++) e[i] = s[i] != 0.f ? fmaf(e[i] - m[i], s[i], 0.f) : 0.f;
        *reinterpret_cast<float4 *>(snr + (size_t)c * npix2 + p) = make_float4(e[0], e[1], e[2], e[3]);
    }
}

// stats: per-channel (median, k * MAD) for PER_IMAGE mode, else unused.
template <int PPW>
__global__ __launch_bounds__(64 * PPW) void detect_pixel_kernel(
    const float *__restrict__ img, int n_chan, int n_pix, int mode, const float2 *__restrict__ stats,
    float thresh, float *__restrict__ snr_out, nbsi_cand *__restrict__ cand, int cap, int *__restrict__ counter,
    int n_groups, unsigned *__restrict__ flags) {
    extern __shared__ float spec[];  // [PPW][n_chan]
    __shared__ float pool_all[PPW][64];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    // XCD-aware order: consecutive pixel groups of one XCD share cache lines of the cube rows
    const int id = blockIdx.x;
    const int xcd = id & 7, slot = id >> 3;
    const int grp = (slot >> 3) * 64 + xcd * 8 + (slot & 7);
    const size_t npix2 = (size_t)n_pix * n_pix;
    const int groups_per_row = n_pix / PPW;
    const bool grp_ok = grp < n_groups;
    const int gy = grp_ok ? grp / groups_per_row : 0;
    const int gx0 = grp_ok ? (grp % groups_per_row) * PPW : 0;
    // stage PPW consecutive pixels of row gy, all channels
    for (int e = t; e < PPW * n_chan; e += 64 * PPW) {
        const int c = e / PPW, pl = e % PPW;
        float v = 0.f;
        if (grp_ok) {
            v = img[(size_t)c * npix2 + (size_t)gy * n_pix + gx0 + pl];
            if (mode == NBSI_DETECT_PER_IMAGE) {
                const float2 st = stats[c];
                v = st.y > 0.f ? (v - st.x) / st.y : v * 0.f;  // (v * 0: non-finite stays non-finite)
            }
        }
        spec[pl * n_chan + c] = v;
    }
    __syncthreads();
    const int x = gx0 + wave, y = gy;
    float *s = spec + wave * n_chan;
    // a spectrum holding a non-finite value is not searched (wave-uniform: one pixel per wave)
    bool bad = false;
    for (int c = lane; c < n_chan; c += 64) bad |= !__builtin_isfinite(s[c]);
    const bool finite = __ballot(bad) == 0ull;
    const bool in_hor = grp_ok && in_horizon(x, y, n_pix);
    if (in_hor && !finite && lane == 0 && flags) atomicOr(flags, NBSI_FLAG_CUBE_NONFINITE);
    const bool active = in_hor && finite;
    float *pool = pool_all[wave];
    auto val_x = [&](int i) { return s[i]; };
    const float med = finite ? wave_median_fast(val_x, n_chan, pool, lane) : 0.f;
    float scale = 1.f;  // SNR = (x - med) / scale
    bool ok = active;
    if (mode == NBSI_DETECT_PER_PIXEL && finite) {
        auto val_d = [&](int i) { return fabsf(s[i] - med); };
        const float mad = wave_median_fast(val_d, n_chan, pool, lane);
        scale = MAD_K * mad;
        ok = ok && mad > 0.f;
    }
    // SNR = (x - med) / scale, applied as a product with the float32 reciprocal (within an ulp of
    // the quotient; the same form scores neighbours for the suppression test)
    const float inv = ok ? 1.f / scale : 0.f;
    for (int c = lane; c < n_chan; c += 64) {
        const float z = ok ? (s[c] - med) * inv : 0.f;
        if (snr_out && grp_ok) snr_out[(size_t)c * npix2 + (size_t)y * n_pix + x] = z;
        if (!ok || z < thresh) continue;
        if (c > 0 && !(z > (s[c - 1] - med) * inv)) continue;
        if (c + 1 < n_chan && !(z >= (s[c + 1] - med) * inv)) continue;
        const int idx = atomicAdd(counter, 1);
        if (idx < cap) {
            nbsi_cand r;
            r.x = x;
            r.y = y;
            r.c = c;
            r.width = 1;
            r.snr = z;
            cand[idx] = r;
        }
    }
}

// Per-channel median and k*MAD over the visible hemisphere (PER_IMAGE mode), one block of SEL_NT
// threads per channel image.  Thread t owns column x = t % n_pix and the rows
// y = y_lo(x) + t / n_pix, + G, ... (G = SEL_NT / n_pix row groups; for n_pix > SEL_NT a thread
// owns several columns) inside the hemisphere, whose extent in each column is an integer square
// root: coalesced row reads, no masking.  Up to 256 x 256 pixels a thread owns at most 64 values,
// which are read once and kept in registers, so every pass of the selections runs from there;
// larger images are re-read each pass with eight loads in flight (the passes of many channels at
// once do not fit the caches).  4,096 x 256^2: 1.16 ms, of which the loads, which nothing overlaps
// (a workgroup's registers fill its CU), take about a third; 2.13 ms when half of the values stood
// in LDS and each selection binned every value over the full range (the LDS adds of a bell-shaped
// distribution collide in its middle bins), then found the bin's ends, then gathered it.
__device__ __forceinline__ int isqrt_floor(int q) {  // largest r >= 0 with r * r <= q (q >= 0)
    int r = (int)sqrtf((float)q);
    while (r * r > q) r--;
    while ((r + 1) * (r + 1) <= q) r++;
    return r;
}

// NV: values per thread in registers (0: read in each pass)
constexpr int STATS_LIST = 1024;  // values a wave can list (a quarter of its 64 x 64)
template <int NV>
__global__ __launch_bounds__(SEL_NT) void image_stats_kernel(const float *__restrict__ img, int n_pix,
                                                             float2 *__restrict__ stats) {
    __shared__ SelLds L;
    __shared__ float s_list[NV < 64 ? 1 : SEL_NW * STATS_LIST];
    const int c = blockIdx.x, t = threadIdx.x;
    const float *im = img + (size_t)c * n_pix * n_pix;
    const int h = n_pix / 2;
    const int G = n_pix <= SEL_NT ? SEL_NT / n_pix : 1;  // row groups
    const int g = n_pix <= SEL_NT ? t / n_pix : 0;
    const bool on = g < G;
    const int x0 = n_pix <= SEL_NT ? t % n_pix : t;
    // rows y0 + g, + G, ... <= y1 of column x in the hemisphere:
    // (x - h)^2 + (y - h)^2 < h^2  <=>  |y - h| <= isqrt(h^2 - (x - h)^2 - 1)
    auto rows = [&](int x, int &y0, int &y1) __attribute__((always_inline)) {
        const int q = h * h - (x - h) * (x - h);
        if (q <= 0) {
            y0 = 1;
            y1 = 0;
            return;
        }
        const int r = isqrt_floor(q - 1);
        y0 = h - r + g;
        y1 = h + r;
    };
    // the thread's values, NaN where there is none (non-finite pixels take no part in the statistics)
    float v[NV ? NV : 1];
    float smp = NAN;  // one of them, from the middle of its column if it can be
    if constexpr (NV > 0) {
        int y0 = 1, y1 = 0;
        if (on) rows(x0, y0, y1);
        const int nv = y1 >= y0 ? (y1 - y0) / G + 1 : 0;  // at most ceil(n_pix / G) <= NV
#pragma unroll
        for (int j = 0; j < NV; j++)  // (rows past the last read it again: no branch, all loads in flight)
            v[j] = im[(nv ? y0 + min(j, nv - 1) * G : h) * n_pix + min(x0, n_pix - 1)];
        float any = NAN;
#pragma unroll
        for (int j = 0; j < NV; j++) {
            v[j] = j < nv && __builtin_isfinite(v[j]) ? v[j] : NAN;
            any = v[j] == v[j] ? v[j] : any;
            // (lane l samples around its own place, so that a wave's samples spread over the image; on
            // 8 x 8 images such places have no value, and without the others a call on 2,000 of them
            // took 0.39 ms instead of 0.18)
            smp = (j & 7) == (t & 7) && v[j] == v[j] && (j <= nv / 2 + 4 || smp != smp) ? v[j] : smp;
        }
        smp = smp == smp ? smp : any;
    } else if (on && x0 < n_pix) {
        int y0, y1;
        rows(x0, y0, y1);
        if (y1 >= y0) smp = im[(size_t)((y0 + y1) / 2) * n_pix + x0];
        smp = __builtin_isfinite(smp) ? smp : NAN;
    }
    auto visit = [&](auto f) __attribute__((always_inline)) {
        if constexpr (NV > 0) {
#pragma unroll
            for (int j = 0; j < NV; j++) f(v[j]);
        } else {
            if (!on) return;
            for (int x = x0; x < n_pix; x += SEL_NT) {
                int y0, y1;
                rows(x, y0, y1);
                int y = y0;
                for (; y + 7 * G <= y1; y += 8 * G) {
                    float u[8];
#pragma unroll
                    for (int k = 0; k < 8; k++) u[k] = im[(size_t)(y + k * G) * n_pix + x];
#pragma unroll
                    for (int k = 0; k < 8; k++)
                        if (__builtin_isfinite(u[k])) f(u[k]);
                }
                for (; y <= y1; y += G) {
                    const float u1 = im[(size_t)y * n_pix + x];
                    if (__builtin_isfinite(u1)) f(u1);
                }
            }
        }
    };
    int n_in = 0;
    visit([&](float x) __attribute__((always_inline)) { n_in += x == x; });
    n_in = block_sum(n_in, L.ired);
    if (n_in == 0) {  // no finite pixel in this channel image (uniform)
        if (t == 0) stats[c] = make_float2(0.f, 0.f);
        return;
    }
    // the median, then the median of the deviations from it (which replace the values in registers)
    float med = 0.f, mad = 0.f;
#pragma unroll 1
    for (int pass = 0; pass < 2; pass++) {
        int listed = 0;  // by this wave
        const float m = block_median(
            [&](auto f) __attribute__((always_inline)) {
                if constexpr (NV > 0) visit(f);
                else visit([&](float x) __attribute__((always_inline)) { f(pass ? fabsf(x - med) : x); });
            },
            [&](float a, float b, int &below) __attribute__((always_inline)) {
                if constexpr (NV < 64) return -1;  // (few values: the passes over them cost less than the list)
                float *mine = s_list + (NV < 64 ? 0 : t >> 6) * STATS_LIST;
                int lt = 0, n_list = 0;
#pragma unroll
                for (int j = 0; j < NV; j++) {
                    const unsigned long long m_lt = __ballot(v[j] < a), m_in = __ballot(v[j] <= b) & ~m_lt;
                    lt += __popcll(m_lt);
                    const int at = n_list + __builtin_amdgcn_mbcnt_hi((unsigned)(m_in >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((unsigned)m_in, 0u));
                    if (((m_in >> (t & 63)) & 1ull) && at < STATS_LIST) mine[at] = v[j];
                    n_list += __popcll(m_in);
                }
                listed = n_list;
                // (counts per wave, added up by block_sum: one lane of each wave holds them)
                below = block_sum((t & 63) == 0 ? lt : 0, L.ired);
                const int full = block_sum((t & 63) == 0 && n_list > STATS_LIST, L.ired);
                const int total = block_sum((t & 63) == 0 ? n_list : 0, L.ired);
                return full ? -1 : total;
            },
            [&](auto f) __attribute__((always_inline)) {
                for (int i = t & 63; i < listed; i += 64) f(s_list[NV < 64 ? 0 : (t >> 6) * STATS_LIST + i]);
            },
            smp, n_in, L);
        if (pass == 0) {
            med = m;
            smp = fabsf(smp - med);
            if constexpr (NV > 0) {
#pragma unroll
                for (int j = 0; j < NV; j++) v[j] = fabsf(v[j] - med);
            }
        } else {
            mad = m;
        }
    }
    if (t == 0) stats[c] = make_float2(med, MAD_K * mad);
}

__device__ __forceinline__ unsigned long long cand_key(const nbsi_cand &r, int n_chan, int n_pix) {
    return ((unsigned long long)((unsigned)r.y * (unsigned)n_pix + (unsigned)r.x)) * (unsigned)n_chan +
           (unsigned)r.c;
}

__global__ void sort_keys_kernel(const nbsi_cand *__restrict__ cand, int n, int n_pow2, int n_chan, int n_pix,
                                 unsigned long long *__restrict__ keys) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pow2) return;
    // key in the high bits, original index in the low 24 bits
    keys[i] = (i < n) ? ((cand_key(cand[i], n_chan, n_pix) << 24) | (unsigned long long)i) : ~0ull;
}

__global__ void bitonic_step_kernel(unsigned long long *__restrict__ keys, int n_pow2, int j, int k) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pow2) return;
    const int p = i ^ j;
    if (p > i) {
        const unsigned long long a = keys[i], b = keys[p];
        const bool up = (i & k) == 0;
        if ((a > b) == up) {
            keys[i] = b;
            keys[p] = a;
        }
    }
}

// The same bitonic network for at most SORT1_MAX candidates in one workgroup: keys in LDS, a
// barrier between steps (each pair (i, i ^ j) is handled by the thread of its lower index), and
// the gather of the sorted records.  One launch instead of one per step.
constexpr int SORT1_MAX = 4096;
__global__ __launch_bounds__(1024) void sort_small_kernel(const nbsi_cand *__restrict__ cand, int n, int n_pow2,
                                                          int n_chan, int n_pix, int n_out,
                                                          nbsi_cand *__restrict__ out) {
    __shared__ unsigned long long s[SORT1_MAX];
    const int t = threadIdx.x;
    for (int i = t; i < n_pow2; i += 1024)
        s[i] = (i < n) ? ((cand_key(cand[i], n_chan, n_pix) << 24) | (unsigned long long)i) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= n_pow2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = t; i < n_pow2; i += 1024) {
                const int p = i ^ j;
                if (p > i) {
                    const unsigned long long a = s[i], b = s[p];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        s[i] = b;
                        s[p] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int i = t; i < n_out; i += 1024) out[i] = cand[(int)(s[i] & 0xffffffull)];
}

// The small sort with the count read on the device: n = *counter candidates (when n <= cap and
// n <= SORT1_MAX; otherwise the host sorts once it has read n), the first min(n, n_out) of them
// written to out in (y, x, c) order.
__global__ __launch_bounds__(1024) void sort_small_dev_kernel(const nbsi_cand *__restrict__ cand,
                                                              const int *__restrict__ counter, int cap, int n_chan,
                                                              int n_pix, int n_out, nbsi_cand *__restrict__ out) {
    __shared__ unsigned long long s[SORT1_MAX];
    const int n = *counter;
    if (n <= 0 || n > cap || n > SORT1_MAX) return;
    int n_pow2 = 1;
    while (n_pow2 < n) n_pow2 <<= 1;
    const int t = threadIdx.x;
    for (int i = t; i < n_pow2; i += 1024)
        s[i] = (i < n) ? ((cand_key(cand[i], n_chan, n_pix) << 24) | (unsigned long long)i) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= n_pow2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = t; i < n_pow2; i += 1024) {
                const int p = i ^ j;
                if (p > i) {
                    const unsigned long long a = s[i], b = s[p];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) {
                        s[i] = b;
                        s[p] = a;
                    }
                }
            }
            __syncthreads();
        }
    const int m = min(n, n_out);
    for (int i = t; i < m; i += 1024) out[i] = cand[(int)(s[i] & 0xffffffull)];
}

__global__ void gather_sorted_kernel(const unsigned long long *__restrict__ keys, const nbsi_cand *__restrict__ cand,
                                     int n_out, nbsi_cand *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_out) return;
    out[i] = cand[(int)(keys[i] & 0xffffffull)];
}

}  // namespace

int detect_ppw(int n_chan) {
    int ppw = 65536 / (n_chan * 4);
    if (ppw >= 4) return 4;
    if (ppw >= 2) return 2;
    return 1;
}

hipError_t launch_detect_stats(const float *img, int n_chan, int n_pix, int mode, float *stats,
                               hipStream_t st) {
    if (mode != NBSI_DETECT_PER_IMAGE) return hipSuccess;
    // values per thread: ceil(n_pix / G) rows of a column, G = SEL_NT / n_pix row groups
#define NBSI_STATS(NV) \
    hipLaunchKernelGGL(image_stats_kernel<NV>, dim3(n_chan), dim3(SEL_NT), 0, st, img, n_pix, reinterpret_cast<float2 *>(stats))
    if (n_pix <= 128) NBSI_STATS(16);
    else if (n_pix <= 256) NBSI_STATS(64);
    else NBSI_STATS(0);
#undef NBSI_STATS
    return hipGetLastError();
}

hipError_t launch_detect_scan(const float *img, int n_chan, int n_pix, int mode, const float *stats,
                              float thresh, float *snr, float *pix_stats, nbsi_cand *cand, int cap, int *counter,
                              hipStream_t st, unsigned *flags) {
    const float2 *s2 = reinterpret_cast<const float2 *>(stats);
    // (an SNR cube that overlaps the images takes the kernel that has read a pixel's spectrum
    // whole before it writes that pixel's SNRs)
    const size_t npix2 = (size_t)n_pix * n_pix, cube_bytes = sizeof(float) * npix2 * n_chan;
    const uintptr_t a0 = (uintptr_t)img, b0 = (uintptr_t)snr;
    const bool overlap = snr && a0 < b0 + cube_bytes && b0 < a0 + cube_bytes;
    if (n_chan <= 64 * 64 && !overlap) {
        // the spectrum's registers are sized to it: every selection pass visits all NR of them
        const int n_blocks = n_pix * (n_pix / REG_PX);
        float *ps = !snr ? nullptr : pix_stats ? pix_stats : snr;
#define NBSI_REG(NR)                                                                                                 \
    hipLaunchKernelGGL(detect_pixel_reg_kernel<NR>, dim3(n_blocks), dim3(64 * REG_PX), 0, st, img, n_chan, n_pix,    \
                       mode, s2, thresh, ps, cand, cap, counter, flags)
        if (n_chan <= 64 * 16) NBSI_REG(16);
        else if (n_chan <= 64 * 32) NBSI_REG(32);
        else NBSI_REG(64);
#undef NBSI_REG
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || !snr) return e;
        // all channels at once, or channels 2 and up and then the two planes that held the statistics
        const unsigned nx = (unsigned)((npix2 / 4 + 255) / 256);
        const int c0 = ps == snr ? 2 : 0;
        hipLaunchKernelGGL(snr_cube_kernel, dim3(nx, (unsigned)((n_chan - c0 + SNR_CPB - 1) / SNR_CPB)), dim3(256), 0,
                           st, img, n_chan, n_pix, mode, s2, ps, c0, snr);
        if (c0) hipLaunchKernelGGL(snr_cube_kernel, dim3(nx, 1), dim3(256), 0, st, img, 2, n_pix, mode, s2, ps, 0, snr);
        return hipGetLastError();
    }
    const int ppw = detect_ppw(n_chan);
    const int n_groups = n_pix * n_pix / ppw;
    // grid covers every group id produced by the XCD-aware mapping (blocks of 64 groups)
    const int n_blocks = ((n_groups + 63) / 64) * 64;
    const size_t lds = (size_t)ppw * n_chan * sizeof(float);
    // the staged spectra may exceed the default 64 KiB of dynamic LDS (gfx950 has 160 KiB)
    hipError_t ea = hipSuccess;
    if (ppw == 4) ea = hipFuncSetAttribute((const void *)detect_pixel_kernel<4>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    else if (ppw == 2) ea = hipFuncSetAttribute((const void *)detect_pixel_kernel<2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    else ea = hipFuncSetAttribute((const void *)detect_pixel_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (ea != hipSuccess) return ea;
    switch (ppw) {
        case 4:
            hipLaunchKernelGGL(detect_pixel_kernel<4>, dim3(n_blocks), dim3(256), lds, st, img, n_chan, n_pix, mode,
                               s2, thresh, snr, cand, cap, counter, n_groups, flags);
            break;
        case 2:
            hipLaunchKernelGGL(detect_pixel_kernel<2>, dim3(n_blocks), dim3(128), lds, st, img, n_chan, n_pix, mode,
                               s2, thresh, snr, cand, cap, counter, n_groups, flags);
            break;
        default:
            hipLaunchKernelGGL(detect_pixel_kernel<1>, dim3(n_blocks), dim3(64), lds, st, img, n_chan, n_pix, mode,
                               s2, thresh, snr, cand, cap, counter, n_groups, flags);
    }
    return hipGetLastError();
}

hipError_t launch_detect_sort_small_dev(const nbsi_cand *cand, const int *counter, int cap, int n_chan, int n_pix,
                                       nbsi_cand *out, int n_out, hipStream_t st) {
    if (n_out <= 0) return hipSuccess;
    hipLaunchKernelGGL(sort_small_dev_kernel, dim3(1), dim3(1024), 0, st, cand, counter, cap, n_chan, n_pix, n_out,
                       out);
    return hipGetLastError();
}

int detect_sort_small_max() { return SORT1_MAX; }

hipError_t launch_detect_sort(nbsi_cand *cand, int n, unsigned long long *keys, int n_chan, int n_pix,
                              nbsi_cand *out, int n_out, hipStream_t st) {
    if (n <= 0 || n_out <= 0) return hipSuccess;
    int n_pow2 = 1;
    while (n_pow2 < n) n_pow2 <<= 1;
    if (n_pow2 <= SORT1_MAX) {
        hipLaunchKernelGGL(sort_small_kernel, dim3(1), dim3(1024), 0, st, cand, n, n_pow2, n_chan, n_pix,
                           n_out <= n ? n_out : n, out);
        return hipGetLastError();
    }
    const int blocks = (n_pow2 + 255) / 256;
    hipLaunchKernelGGL(sort_keys_kernel, dim3(blocks), dim3(256), 0, st, cand, n, n_pow2, n_chan, n_pix, keys);
    for (int k = 2; k <= n_pow2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1)
            hipLaunchKernelGGL(bitonic_step_kernel, dim3(blocks), dim3(256), 0, st, keys, n_pow2, j, k);
    hipLaunchKernelGGL(gather_sorted_kernel, dim3((n_out + 255) / 256), dim3(256), 0, st, keys, cand, n_out, out);
    return hipGetLastError();
}

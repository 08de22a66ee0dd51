// Stand-alone compress / decompress with the quantizers that the paper ablates for the second moment (Sec. 4.1,
// Tab. 1): block-wise normalization with block size 128 or 2048 or rank-1 normalization, the 4-bit
// dynamic-exponent map (unsigned for non-negative input, signed for signed input), the same map without its zero
// ("DE-0", 15 points) or the Linear map, rounding to the nearest entry or stochastic rounding (App. D.3).  None of
// them is on an optimizer step's path except B128 / signed DE, B128 / Linear and rank-1 / Linear, which the step
// kernels implement themselves; these kernels are for studying the quantizers on real tensors.
//
// Laid out like the stand-alone conversions: 4 elements per lane, 4096 per workgroup; with stochastic rounding or rank-1 scales 2048 in
// smaller tensors (kAblShortElems).  The compress kernels are
// bound by the vector units, not by memory, so what counts is instructions per element.  As in the step kernels a value is normalized
// with an approximate reciprocal and its code found through a table of 257 (signed maps: 513) buckets in LDS, and a wave in which
// that leaves a doubt does its four elements again with IEEE divisions and a search.  Of the rest most is SplitMix64: six 32-bit
// multiplications, which run at a quarter of the rate.
// Measured on 4096 x 4096, DE-0, stochastic rounding: compress under the three normalizations 43, 43 and 45 us with a division and a
// search of four dependent LDS reads per element, 32, 32 and 38 this way (57, 58 and 69 vector instructions an element, 9 of them to set
// the tables up; 83 to 85 % of the issue cycles); decompress 12.6.  SplitMix64
// with its cross products as dot products of 16-bit halves, at the full rate, takes as long (all six calls 152.4 us, 153.3).
#pragma once

#include "convert.hpp"

namespace lpmm {

// What a compress kernel searches by.  Kernels are handed what they use and no more, and set up with one barrier: a call on a small
// tensor takes little else (64 x 64, block 128, to nearest 4.15 us with all tables of both roundings in the arguments, a barrier in
// front of the buckets and another behind, 3.29 so).
struct AblMap {
    float v[kCodes];          // increasing, +inf beyond the last.  Stochastic rounding: the entries; to nearest: the largest floats not
                              // above the midpoints of neighbouring entries
    int bucket[kCodes];       // of v, kBuckets beyond the last one
    int n;                    // entries
    uint32_t zero4;           // the codes of four zeros: a zero's is the same under every scale and either rounding
    float least;              // of the normalized values: 0, signed maps -1
};
// stochastic rounding, by the number of entries below a value: 2^24 over the distance from the entry below it to the next, so that the
// next entry itself gives no less than 2^24
struct AblGaps {
    float inv[kCodes];
};
template <bool SR> struct AblSearch : AblMap {};
template <> struct AblSearch<true> : AblMap, AblGaps {};
struct AblEntries {           // what the decompress kernel looks up
    float T[kCodes];          // 0 beyond the last
};

struct AblArgs {
    const float* x_in;        // compress: input
    float* x_out;             // decompress: output
    const uint32_t* q_in;
    uint32_t* q_out;
    float* sa;                // block scales, or row maxima
    float* sb;                // column maxima (rank-1)
    int64_t rows, cols, P;
    int stochastic;
    uint64_t seed;
};

struct AblLds {
    SearchEntry bucket[kBucketsPadded];      // how many of v lie in the buckets below, and the next one
    float2 gap[kCodes];       // {entry below, AblGaps::inv}; the first entry where there is none below
    float v[kCodes];
};
// A bucket without one of v compares with the next one above, which is larger than everything in the bucket.
template <bool SR>
__device__ __forceinline__ void abl_load_map(AblLds& s, const AblSearch<SR>& m) {
    const int t = threadIdx.x;
    if (t < kCodes) {
        s.v[t] = m.v[t];
        if constexpr (SR) s.gap[t] = make_float2(m.v[t > 0 ? t - 1 : 0], m.inv[t]);
    }
    for (int b = (m.least < 0.0f ? 0 : kBucketHalf) + t; b < kBuckets; b += kThreads) {
        uint32_t below = 0;
        float next = m.v[0];
#pragma unroll
        for (int k = 0; k < kCodes; ++k) {
            const bool under = m.bucket[k] < b;
            below += under ? 1u : 0u;
            next = under ? (k + 1 < kCodes ? m.v[k + 1] : __builtin_inff()) : next;
        }
        s.bucket[b] = SearchEntry{next, below};
    }
    __syncthreads();
}

// number of a[0..14] (increasing) that lie below n; 0 for NaN
__device__ __forceinline__ int abl_count_below(const float* a, float n) {
    int c = n > a[7] ? 8 : 0;
    c += n > a[c + 3] ? 4 : 0;
    c += n > a[c + 1] ? 2 : 0;
    c += n > a[c] ? 1 : 0;
    return c;
}

// Uniform number of element `idx`: the top 24 bits of output number idx + 1 of the SplitMix64 generator started at
// `seed`, in units of 2^-24.  (The generator's last step, z ^= z >> 31, does not reach them.)
constexpr uint64_t kSplitMixStep = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t abl_generator(uint64_t seed, uint64_t idx) { return seed + (idx + 1) * kSplitMixStep; }
__device__ __forceinline__ uint64_t abl_xorshift(uint64_t z, int k) {          // z ^ (z >> k), k < 32, in 32-bit operations
    const uint32_t lo = uint32_t(z), hi = uint32_t(z >> 32);
    return uint64_t(hi ^ (hi >> k)) << 32 | (lo ^ __builtin_amdgcn_alignbit(hi, lo, k));
}
__device__ __forceinline__ float abl_uniform24(uint64_t z) {
    z = abl_xorshift(z, 30) * 0xBF58476D1CE4E5B9ull;
    z = abl_xorshift(z, 27) * 0x94D049BB133111EBull;
    return float(uint32_t(z >> 32) >> 8);
}

// App. D.3: the candidates are the entry at or below n and the entry at or above it; one candidate if n is an entry or
// outside the table's range; else the upper one with probability p = (n - T[q1]) / (T[q2] - T[q1]), in fp32 with IEEE
// division.  The quotient is first taken with the approximate reciprocal, which is within 2^-21 of p; only where that
// does not settle u < p is the division done.
__device__ __forceinline__ uint32_t abl_stochastic(const AblLds& m, int n_entries, float n, float u) {
    int lt = abl_count_below(m.v, n);                       // entries below n
    if (lt == 15 && n > m.v[15]) lt = 16;
    const float hi = m.v[lt < 15 ? lt : 15];
    const int le = lt + (lt < n_entries && hi == n ? 1 : 0);     // entries at or below n
    const int q1 = le - 1, q2 = lt;
    if (q1 < 0) return uint32_t(q2 < n_entries ? q2 : 0);
    if (q2 >= n_entries || q1 == q2) return uint32_t(q1);
    const float d = n - m.v[q1], w = hi - m.v[q1];
    float p = d * __builtin_amdgcn_rcpf(w);
    if (fabsf(u - p) < 0x1p-18f) p = d / w;
    return uint32_t(u < p ? q2 : q1);
}

// Codes of 4 elements with scales s[e]; idx = row-major index of the first.
//
// The approximate n' = x * rcp(s) is within 2^-22 of the exact n, relatively; to nearest, the guard is that of the step's first
// moment (kMinDistM).  For stochastic rounding the reciprocal is raised by 2^-22, so that n' of a block's largest element comes out
// as 1, and n' is within 2^-21.  With the distance of neighbouring entries at least n / 17.9 everywhere, the probability p' is then
// within 2^-16.8 of the exact one, and the code can differ only if the random number is that close to it.  If n' and n lie on
// different sides of an entry, one of the two probabilities is that close to 1 and the other to 0: either way the entry between them
// is taken unless the random number itself is that close to 0 or 1.  So what counts as a doubt hangs on the random number alone, about
// one element in 10^4 whatever the values; one that is 0, next to 0 or its own scale (n is an entry, or all but one) is no likelier.
// (Where closeness of p' to 0 or 1 was a doubt, one zero under a map that has one sent its wave both ways: DE, 4096 x 4096,
// stochastic rounding, block 128, 1 % zeros 47.7 us, 30 without; with division and search for everything 39.)  A wave of nothing but
// zeros, rows that had no gradient yet, needs none of it (nine rows of ten, rank-1: 50 us, 37 so; 45 with division and search).  NaN comes out as
// the first entry both ways; extreme scales count as doubts.
constexpr float kMarginSr = 256.0f;          // 2^-16 in units of 2^-24
template <bool SR>
__device__ __forceinline__ uint32_t abl_codes4(const AblLds& m, const AblMap& map, uint64_t seed, int64_t idx, const float x[4],
                                               const float s[4], const float inv[4], bool tame) {
    uint32_t bits = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) bits |= __float_as_uint(x[e]) << 1;
    if (__ballot(bits != 0) == 0) return map.zero4;
    uint32_t w = 0;
    bool doubt = !tame;
    const uint64_t z0 = abl_generator(seed, uint64_t(idx));
    float u[4];
    if constexpr (SR) {
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = abl_uniform24(z0 + uint64_t(e) * kSplitMixStep);
    }
    uint32_t dist = 0xFFFFFFFFu;
    float close = 0x1p24f, off_centre = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float n = __builtin_amdgcn_fmed3f(x[e] * inv[e], map.least, 1.0f);
        const SearchEntry b = search_entry(m.bucket, n);
        const uint32_t below = b.base + (n > b.thr ? 1u : 0u);
        if constexpr (SR) {
            const float2 g = m.gap[below];          // n <= 1, the last entry, so below < kCodes
            const float p = (n - g.x) * g.y;
            close = fminf(close, fabsf(u[e] - p));
            off_centre = fmaxf(off_centre, fabsf(u[e] - 0x1p23f));
            w |= (__builtin_elementwise_sub_sat(below, 1u) + (u[e] < p ? 1u : 0u)) << (4 * e);
        } else {
            uint32_t d;
            asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(__float_as_uint(n)), "v"(__float_as_uint(b.thr)));
            dist = min(dist, d);
            w |= below << (4 * e);
        }
    }
    if constexpr (SR) doubt = bool(int(doubt) | int(close < kMarginSr) | int(off_centre > 0x1p23f - kMarginSr));
    if constexpr (!SR) doubt = bool(int(doubt) | int(dist < kMinDistM));
    if (__builtin_expect(__ballot(doubt) != 0, 0)) {
        w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float n = (s[e] == 0.0f) ? 0.0f : x[e] / s[e];
            uint32_t q;
            if constexpr (SR) q = abl_stochastic(m, map.n, n, u[e] * 0x1p-24f);
            else q = uint32_t(abl_count_below(m.v, n));        // nearest entry, ties to the lower index
            w |= q << (4 * e);
        }
    }
    return w;
}
// 1 / s for that; 0 for 0
template <bool SR>
__device__ __forceinline__ float abl_inverse(float s) { return approx_inv(s) * (SR ? 1.0f + 0x1p-22f : 1.0f); }

// Block-wise normalization: a workgroup takes UNITS runs of 1024 elements, four (two blocks of 2048 or 32 of 128) or, with
// stochastic rounding in tensors of at most 2^21 elements, two: there the chain of a lane's 16 roundings is what the call
// takes (a call with the copies of its arguments, before AblSearch: 64 x 64 8.8 us with four, 7.8 with two; 4096 x 100: 9.1, 7.9).
constexpr int64_t kAblShortElems = int64_t(1) << 21;
template <int BLOCK, bool SR, int UNITS>
__global__ __launch_bounds__(kThreads) void abl_quant_block_kernel(const AblArgs a, const AblSearch<SR> m) {
    static_assert(BLOCK == 128 || BLOCK == 2048, "block sizes of Tab. 1");
    static_assert(UNITS % 2 == 0 && kCvtUnitElems == 1024, "two units of a workgroup make one block of 2048");
    constexpr int kBlocks = UNITS / 2;                    // of 2048
    __shared__ AblLds s_map;
    __shared__ float s_part[kBlocks][kThreads / 64];
    const int64_t first = int64_t(blockIdx.x) * (UNITS * kCvtUnitElems) + threadIdx.x * 4;
    float x[UNITS][4], sc[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) cvt_load4(a.x_in, first + u * kCvtUnitElems, a.P, x[u]);
    abl_load_map<SR>(s_map, m);
#pragma unroll
    for (int u = 0; u < UNITS; ++u)
        sc[u] = group32_allmax(cvt_absmax4(x[u]));
    if constexpr (BLOCK == 2048) {
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            float v = fmaxf(sc[2 * b], sc[2 * b + 1]);
            v = fmaxf(v, __shfl_xor(v, 32));
            if ((threadIdx.x & 63) == 0) s_part[b][threadIdx.x >> 6] = v;
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            sc[2 * b] = sc[2 * b + 1] = fmaxf(fmaxf(s_part[b][0], s_part[b][1]), fmaxf(s_part[b][2], s_part[b][3]));
        if (threadIdx.x < kBlocks) {
            const int64_t blk = int64_t(blockIdx.x) * kBlocks + threadIdx.x;
            if (blk * 2048 < a.P) a.sa[blk] = threadIdx.x ? sc[2 * (kBlocks - 1)] : sc[0];
        }
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const int64_t base = first + u * kCvtUnitElems;
        if (base >= a.P) continue;
        const float s[4] = {sc[u], sc[u], sc[u], sc[u]}, i = abl_inverse<SR>(sc[u]), inv[4] = {i, i, i, i};
        cvt_store_codes(a.q_out, base, a.P, abl_codes4<SR>(s_map, m, a.seed, base, x[u], s, inv, scale_is_tame(sc[u])));
        if constexpr (BLOCK == 128)
            if ((threadIdx.x & 31) == 0) a.sa[base >> 7] = sc[u];
    }
}

// Rank-1 normalization, second stage: codes against min(r_i, c_j) (the maxima are complete in sa / sb).  Two runs in short tensors, whatever
// the rounding (all six calls on 1000 x 1001 40.0 us with four, 37.9 so; 300 x 16000 to nearest 46.4 and 47.5, 7484 x 4483 265.4 and 267.2).
template <bool SR, int UNITS>
__global__ __launch_bounds__(kThreads) void abl_quant_rank1_kernel(const AblArgs a, const AblSearch<SR> m) {
    __shared__ AblLds s_map;
    const int64_t wg_first = int64_t(blockIdx.x) * (UNITS * kCvtUnitElems);
    const CvtOrigin o = cvt_origin(wg_first, a.cols);
    float x[UNITS][4], s[UNITS][4];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const uint32_t off = u * kCvtUnitElems + threadIdx.x * 4;
        cvt_load4(a.x_in, wg_first + off, a.P, x[u]);
        rank1_scales4(o, off, a.rows, a.sa, a.sb, s[u]);
    }
    abl_load_map<SR>(s_map, m);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const int64_t base = wg_first + u * kCvtUnitElems + threadIdx.x * 4;
        if (base >= a.P) continue;
        float inv[4];
        bool tame = true;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            inv[e] = abl_inverse<SR>(s[u][e]);
            tame = bool(int(tame) & int(scale_is_tame(s[u][e])));
        }
        cvt_store_codes(a.q_out, base, a.P, abl_codes4<SR>(s_map, m, a.seed, base, x[u], s[u], inv, tame));
    }
}

// norm: 0 = block 128, 1 = block 2048, 2 = rank-1
__global__ __launch_bounds__(kThreads) void abl_dequant_kernel(const AblArgs a, const AblEntries m, int norm) {
    __shared__ float s_T[kCodes];
    const int64_t wg_first = int64_t(blockIdx.x) * kCvtElems;
    uint32_t w[kCvtUnits];
    float s[kCvtUnits][4];
    if (norm == 2) {
        const CvtOrigin o = cvt_origin(wg_first, a.cols);
#pragma unroll
        for (int u = 0; u < kCvtUnits; ++u) rank1_scales4(o, u * kCvtUnitElems + threadIdx.x * 4, a.rows, a.sa, a.sb, s[u]);
    } else {
        const int shift = norm == 0 ? 7 : 11;
#pragma unroll
        for (int u = 0; u < kCvtUnits; ++u) {
            const int64_t base = wg_first + u * kCvtUnitElems + threadIdx.x * 4;
            s[u][0] = s[u][1] = s[u][2] = s[u][3] = base < a.P ? a.sa[base >> shift] : 0.0f;
        }
    }
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) w[u] = cvt_load_codes(a.q_in, wg_first + u * kCvtUnitElems + threadIdx.x * 4, a.P);
    if (threadIdx.x < kCodes) s_T[threadIdx.x] = m.T[threadIdx.x];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = s_T[(w[u] >> (4 * e)) & 15u] * s[u][e];
        cvt_store4(a.x_out, wg_first + u * kCvtUnitElems + threadIdx.x * 4, a.P, v);
    }
}

}  // namespace lpmm

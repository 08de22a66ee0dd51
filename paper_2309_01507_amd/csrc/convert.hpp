// Stand-alone compress / decompress of one moment (the quantizer M o N of Sec. 2.2 and its inverse): checkpoints,
// conversion from and to fp32 states, and the building blocks of the ablation quantizers.
//
// What bounds these kernels is memory: 4 bytes of fp32 and half a byte of codes per element, each touched once.  So a
// lane owns FOUR consecutive elements of the row-major flattening (one 128-bit access, 16 bits of codes), a wave's
// access is contiguous, a workgroup takes four runs of 1024 elements (with rank-1 scales two, see kRankShortElems) whose loads are all issued
// before the first use, and the 64-bit division that finds a position's row is done once per workgroup, for its first element.
// Measured on an 11008 x 4096 moment, before (one lane per 8 elements, scalar accesses, a 64-bit division each) and now:
// compress the first moment 106 -> 39 us, its codes alone for the second 170 -> 35 us, decompress the first 111 -> 31 us,
// the second 139 -> 30.5 us.  The fp32 arrays and the
// scales need only be 4-byte aligned: the wide accesses are typed so.
// What is read for the last time and the decompressed values pass by the memory-side cache (non-temporal), which then still
// holds what a later kernel reads again: the second moment for its codes, the codes and scales for the way back.  Both moments
// of an 11008 x 4096 matrix there and back 232 -> 183 us (one-touch bytes at 4.5 TB/s), of 16384 x 8192 636 -> 520; with the maxima's tiles
// and the shorter workgroups below 170 (4.8 TB/s) and 505.
// The decompressed values do so at every size: kept, they are written back during the kernels that follow.  Plain / non-temporal
// stores: there and back 2048 x 2048 40 / 38 us, 4096 x 4096 92 / 79, 8192 x 4096 164 / 137, 11008 x 4096 231 / 183; decompression and a
// kernel that scales the values into another array 16.6 / 16.8, 38.8 / 39.9, 69.9 / 65.2, 90.8 / 96.0.  Who only reads them, right
// away, pays up to the cache's 256 MB: with a sum behind it 23.2 / 23.2, 39.2 / 44.1, 55.8 / 66.9 and 66.9 / 82.7, from there on less
// (16384 x 4096 131 / 120).
#pragma once

#include "kernels.hpp"

namespace lpmm {

struct QuantArgs {
    const uint32_t* q_in;   // dequant: codes
    uint32_t* q_out;        // quant: codes
    const float* x_in;      // quant: fp32 moment
    float* x_out;           // dequant: fp32 moment
    float* sa;              // block scales or row maxima
    float* sb;              // column maxima (second moment)
    int64_t rows, cols, P;
};

typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));     // 128-bit access at 4-byte alignment

constexpr int kCvtUnits = 4;
constexpr int kCvtUnitElems = kThreads * 4;
constexpr int kCvtElems = kCvtUnits * kCvtUnitElems;      // elements per workgroup (two blocks of 2048)
// Kernels with rank-1 scales take two runs in tensors of up to kRankShortElems elements, four in larger ones: a run's chain of rows, columns and
// scales is long (four runs and two: 11008 x 4096 codes 37.3 and 35.9 us, decompress 32.9 and 30.5; 3000 x 1001 7.6 and 6.0, both; 16000 x
// 16001 210 and 209, 160 and 164).
constexpr int64_t kRankShortElems = int64_t(1) << 27;

// ---- accesses of a lane's 4 elements; `base` is a multiple of 4, elements at or beyond P do not exist ----

// STREAM: the array is not read again soon (non-temporal: it takes no room in the memory-side cache from what is).
template <bool STREAM = false>
__device__ __forceinline__ void cvt_load4(const float* x, int64_t base, int64_t P, float out[4]) {
    if (base + 4 <= P) {
        const v4f_a4* p = reinterpret_cast<const v4f_a4*>(x + base);
        const v4f_a4 v = STREAM ? __builtin_nontemporal_load(p) : *p;
        out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = base + e < P ? x[base + e] : 0.0f;
    }
}
__device__ __forceinline__ void cvt_store4(float* x, int64_t base, int64_t P, const float v[4]) {
    if (base + 4 <= P) {
        const v4f_a4 w = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(w, reinterpret_cast<v4f_a4*>(x + base));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (base + e < P) x[base + e] = v[e];
    }
}
// 16 bits of codes; in the tail the bytes that hold an existing element (the unused nibble of an odd tail is 0)
__device__ __forceinline__ uint32_t cvt_load_codes(const uint32_t* q, int64_t base, int64_t P) {
    const uint8_t* b = reinterpret_cast<const uint8_t*>(q) + (base >> 1);
    if (base + 4 <= P) return *reinterpret_cast<const uint16_t*>(b);
    uint32_t w = 0;
    if (base < P) w = b[0];
    if (base + 2 < P) w |= uint32_t(b[1]) << 8;
    return w;
}
__device__ __forceinline__ void cvt_store_codes(uint32_t* q, int64_t base, int64_t P, uint32_t w) {
    uint8_t* b = reinterpret_cast<uint8_t*>(q) + (base >> 1);
    if (base + 4 <= P) {
        *reinterpret_cast<uint16_t*>(b) = uint16_t(w);
    } else {
        const int nv = base < P ? int(P - base) : 0;             // 0..3
        w &= (1u << (4 * nv)) - 1u;
        if (nv > 0) b[0] = uint8_t(w);
        if (nv > 2) b[1] = uint8_t(w >> 8);
    }
}

// Largest magnitude of a lane's 4 elements, from 0 on: a NaN raises nothing, also where all four are NaN, so that it costs
// its block its own code and not the scale.
__device__ __forceinline__ float cvt_absmax4(const float x[4]) {
    return fmaxf(fmaxf(fmaxf(fmaxf(0.0f, fabsf(x[0])), fabsf(x[1])), fabsf(x[2])), fabsf(x[3]));
}

// Row and column of a workgroup's first element; rows and columns of its other elements follow by 32-bit arithmetic
// (cols <= 2^31, and a workgroup spans kCvtElems elements).
struct CvtOrigin {
    int64_t i;
    uint32_t j, cols;
};
__device__ __forceinline__ CvtOrigin cvt_origin(int64_t first, int64_t cols) {
    CvtOrigin o;
    o.i = first / cols;
    o.j = uint32_t(first - o.i * cols);
    o.cols = uint32_t(cols);
    return o;
}
// The rank-1 scales min(r_i, c_j) of the 4 elements that lie `off` behind the workgroup's first one.  Elements beyond
// the tensor get scale 0.
__device__ __forceinline__ void rank1_scales4(const CvtOrigin& o, uint32_t off, int64_t rows, const float* r, const float* c,
                                              float s[4]) {
    uint32_t j = o.j + off;                                       // < 2^31 + kCvtElems
    int64_t i = o.i;
    if (j >= o.cols) {
        const uint32_t q = j / o.cols;
        i += q;
        j -= q * o.cols;
    }
    if (i < rows && j + 4u <= o.cols) {
        const float rv = r[i];
        const v4f_a4 cv = *reinterpret_cast<const v4f_a4*>(c + j);
        s[0] = fminf(rv, cv.x); s[1] = fminf(rv, cv.y); s[2] = fminf(rv, cv.z); s[3] = fminf(rv, cv.w);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = i < rows ? fminf(r[i], c[j]) : 0.0f;
            if (++j == o.cols) { j = 0; ++i; }
        }
    }
}

// ---- first moment ----------------------------------------------------------------------------------------------------

__global__ __launch_bounds__(kThreads) void dequant_m_kernel(const QuantArgs q) {
    __shared__ float2 s_deq[256];
    const float2* gd = reinterpret_cast<const float2*>(d_byte_decode);
    s_deq[threadIdx.x] = gd[threadIdx.x];
    const int64_t first = int64_t(blockIdx.x) * kCvtElems + threadIdx.x * 4;
    uint32_t w[kCvtUnits];
    float s[kCvtUnits];
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        const int64_t base = first + u * kCvtUnitElems;
        w[u] = cvt_load_codes(q.q_in, base, q.P);
        s[u] = base < q.P ? q.sa[base >> 7] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        const float2 a = s_deq[w[u] & 255u], b = s_deq[w[u] >> 8];
        const float v[4] = {a.x * s[u], a.y * s[u], b.x * s[u], b.y * s[u]};
        cvt_store4(q.x_out, first + u * kCvtUnitElems, q.P, v);
    }
}

__global__ __launch_bounds__(kThreads) void quant_m_kernel(const QuantArgs q) {
    __shared__ SearchEntry s_search[kBucketsPadded];
    const int64_t first = int64_t(blockIdx.x) * kCvtElems + threadIdx.x * 4;
    float x[kCvtUnits][4];
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) cvt_load4<true>(q.x_in, first + u * kCvtUnitElems, q.P, x[u]);
    const uint2* gs = reinterpret_cast<const uint2*>(d_search);
    uint2* ss = reinterpret_cast<uint2*>(s_search);
    for (int i = threadIdx.x; i < kBucketsPadded; i += kThreads) ss[i] = gs[i];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        const int64_t base = first + u * kCvtUnitElems;
        const float sc = group32_allmax(cvt_absmax4(x[u]));
        cvt_store_codes(q.q_out, base, q.P, compress_m4(s_search, x[u], sc));
        if ((threadIdx.x & 31) == 0 && base < q.P) q.sa[base >> 7] = sc;
    }
}

// ---- second moment ---------------------------------------------------------------------------------------------------

// codes of 4 elements under the Linear map: reciprocal and guard, IEEE division for a wave that needs it.  The inputs
// of lanes beyond the tensor are 0 with scale 0.
__device__ __forceinline__ uint32_t linear_codes4(const float x[4], const float s[4]) {
    uint32_t lo = 0, hi = 0;
    float closest = 0.5f, fa, fb;
    bool tame = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) tame = bool(int(tame) & int(scale_is_tame(s[e])));
    lo = quant_v_code_fast<0>(x[0], approx_inv16(s[0]), lo, fa);
    hi = quant_v_code_fast<0>(x[1], approx_inv16(s[1]), hi, fb);
    closest = fminf(fminf(closest, fabsf(fa)), fabsf(fb));
    lo = quant_v_code_fast<1>(x[2], approx_inv16(s[2]), lo, fa);
    hi = quant_v_code_fast<1>(x[3], approx_inv16(s[3]), hi, fb);
    closest = fminf(fminf(closest, fabsf(fa)), fabsf(fb));
    uint32_t w = lo | (hi << 4);
    if (__builtin_expect(__ballot(closest < kMarginV || !tame) != 0, 0)) {
        w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w |= quant_v_code(x[e], s[e]) << (4 * e);
    }
    return w;
}

template <int UNITS>
__global__ __launch_bounds__(kThreads) void dequant_v_kernel(const QuantArgs q) {
    const int64_t wg_first = int64_t(blockIdx.x) * (UNITS * kCvtUnitElems);
    const CvtOrigin o = cvt_origin(wg_first, q.cols);
    uint32_t w[UNITS];
    float s[UNITS][4];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const uint32_t off = u * kCvtUnitElems + threadIdx.x * 4;
        w[u] = cvt_load_codes(q.q_in, wg_first + off, q.P);
        rank1_scales4(o, off, q.rows, q.sa, q.sb, s[u]);
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = dequant_v((w[u] >> (4 * e)) & 15u, s[u][e]);
        cvt_store4(q.x_out, wg_first + u * kCvtUnitElems + threadIdx.x * 4, q.P, v);
    }
}

// second moment with block scales (1-dimensional / flattened tensors)
__global__ __launch_bounds__(kThreads) void dequant_vb_kernel(const QuantArgs q) {
    const int64_t first = int64_t(blockIdx.x) * kCvtElems + threadIdx.x * 4;
    uint32_t w[kCvtUnits];
    float s[kCvtUnits];
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        const int64_t base = first + u * kCvtUnitElems;
        w[u] = cvt_load_codes(q.q_in, base, q.P);
        s[u] = base < q.P ? q.sa[base >> 7] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = dequant_v((w[u] >> (4 * e)) & 15u, s[u]);
        cvt_store4(q.x_out, first + u * kCvtUnitElems, q.P, v);
    }
}

// block-wise second moment (values >= 0): block maximum, Linear map
__global__ __launch_bounds__(kThreads) void quant_vb_kernel(const QuantArgs q) {
    const int64_t first = int64_t(blockIdx.x) * kCvtElems + threadIdx.x * 4;
    float x[kCvtUnits][4];
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) cvt_load4<true>(q.x_in, first + u * kCvtUnitElems, q.P, x[u]);
#pragma unroll
    for (int u = 0; u < kCvtUnits; ++u) {
        const int64_t base = first + u * kCvtUnitElems;
        const float sc = group32_allmax(cvt_absmax4(x[u]));
        const float s[4] = {sc, sc, sc, sc};
        cvt_store_codes(q.q_out, base, q.P, linear_codes4(x[u], s));
        if ((threadIdx.x & 31) == 0 && base < q.P) q.sa[base >> 7] = sc;
    }
}

// Row and column maxima of a rows x cols matrix into sa / sb (zero on entry), for rank-1 normalization.
//
// A workgroup takes rows_per_wg rows x a strip of 8 * TX columns: TX lanes take 8 columns each of one row, 256 / TX rows side by
// side.  Column maxima stay in registers down the tile, a row's maximum is reduced over its lanes, and one global atomic per row and
// per column of the tile follows at the end.  A maximum may be taken twice, so nothing needs a branch at the edges: the last lane that
// has columns takes the last 8 of the row, lanes and rows beyond repeat what others take.  As few lanes to a row as its columns need:
// with 16 for every narrow matrix a wave took its 4 rows no sooner than 128 columns (with codes, us, before and so: 2000000 x 16 94 and
// 86, 1000000 x 32 72 and 64).  SINGLE: matrices of up to 64 columns whose rows begin anywhere; lane x takes columns x, x + TX and so on, an
// element at a time (2000001 x 15 149 in 16-byte loads by 16 lanes, 142 by 4, 99 so; 1000001 x 33 113, 110 and 89).
// Bound by those atomics and by latency where the matrix is small, else by memory.  Strips of 1024 columns by 4 to 32 rows, as the
// filling of the chip asked for them, sent two to three times as many atomics, which were what the pass took: 3000 x 1001 18.6 us, 6.3
// so, 1000 x 1001 8.0 and 4.2, 4096 x 4096 15.3 and 13.8, 11008 x 4096 43 and 35.5 (5.1 TB/s).
// Wide matrices: `run` strips to a workgroup, see launch_maxima.
constexpr int kMaxTileRows = 512;
constexpr int kMaxCols = 8;               // of a lane

struct MaxTiling {
    int rows_per_wg;      // <= kMaxTileRows
    int strips;           // ceil(cols / (8 * TX))
    int run;              // strips that a workgroup takes one after the other
    int groups;           // ceil(strips / run)
    int whole;            // all rows in one tile: column maxima are complete, and stored
};

// maximum over the TX lanes of a row of the bits of values >= +0, the same in all of them
template <int TX>
__device__ __forceinline__ uint32_t lanes_allmax(uint32_t v) {
    static_assert(TX == 4 || TX == 8 || TX == 16 || TX == 32, "lanes of a row: a quad to a half-wave");
    if constexpr (TX == 32) return __float_as_uint(group32_allmax(__uint_as_float(v)));
    v = dpp_umax<0xB1>(v);
    v = dpp_umax<0x4E>(v);
    if constexpr (TX >= 8) v = dpp_umax<0x141>(v);
    if constexpr (TX >= 16) v = dpp_umax<0x140>(v);
    return v;
}

template <int TX, bool SINGLE>
__global__ __launch_bounds__(kThreads) void quant_v_max_kernel(const QuantArgs q, const MaxTiling t) {
    constexpr int kTy = kThreads / TX, kDepth = 4;
    __shared__ uint32_t s_row[kMaxTileRows];
    __shared__ uint32_t s_col[kTy][TX * kMaxCols];
    const int first = int(blockIdx.x % t.groups) * t.run, end = min(first + t.run, t.strips);
    const int64_t row0 = int64_t(blockIdx.x / t.groups) * t.rows_per_wg;
    const int64_t left = q.rows - row0;
    const int n = left < t.rows_per_wg ? int(left) : t.rows_per_wg;
    const int x = threadIdx.x % TX, y = threadIdx.x / TX;
    const int64_t last = SINGLE ? 0 : q.cols - kMaxCols;
    // a value's bits, 0 unless it is above 0 (a NaN raises no maximum)
    auto bits = [](float v) { return v > 0.0f ? __float_as_uint(v) : 0u; };
    for (int strip = first; strip < end; ++strip) {
        const int64_t strip0 = int64_t(strip) * (TX * kMaxCols), own = strip0 + kMaxCols * x;
        const float* p = q.x_in + row0 * q.cols + (SINGLE ? 0 : own < last ? own : last);
        int off[kMaxCols];
#pragma unroll
        for (int e = 0; e < kMaxCols; ++e) off[e] = x + e * TX < int(q.cols) ? x + e * TX : int(q.cols) - 1;
        uint32_t cm[kMaxCols];
#pragma unroll
        for (int e = 0; e < kMaxCols; ++e) cm[e] = 0u;
        for (int base = 0; base < n; base += kTy * kDepth) {          // the same rounds in all lanes
            float v[kDepth][kMaxCols];
#pragma unroll
            for (int u = 0; u < kDepth; ++u) {
                const int il = base + u * kTy + y;
                const float* pr = p + int64_t(il < n ? il : n - 1) * q.cols;
                if constexpr (SINGLE) {
#pragma unroll
                    for (int e = 0; e < kMaxCols; ++e) v[u][e] = pr[off[e]];
                } else {
                    const v4f_a4 a = reinterpret_cast<const v4f_a4*>(pr)[0], b = *reinterpret_cast<const v4f_a4*>(pr + 4);
                    v[u][0] = a.x; v[u][1] = a.y; v[u][2] = a.z; v[u][3] = a.w;
                    v[u][4] = b.x; v[u][5] = b.y; v[u][6] = b.z; v[u][7] = b.w;
                }
            }
#pragma unroll
            for (int u = 0; u < kDepth; ++u) {
                const int il = base + u * kTy + y;
                uint32_t rm = 0u;
#pragma unroll
                for (int e = 0; e < kMaxCols; ++e) {
                    const uint32_t z = bits(v[u][e]);
                    cm[e] = max(cm[e], z);
                    rm = max(rm, z);
                }
                const uint32_t all = lanes_allmax<TX>(rm);
                if (x == 0 && il < n) s_row[il] = strip == first ? all : max(s_row[il], all);
            }
        }
#pragma unroll
        for (int e = 0; e < kMaxCols; ++e) s_col[y][SINGLE ? x + e * TX : x * kMaxCols + e] = cm[e];
        __syncthreads();
        if (int(threadIdx.x) < TX * kMaxCols) {
            const int64_t lane_own = strip0 + (SINGLE ? threadIdx.x : threadIdx.x & ~(kMaxCols - 1)), lane0 = SINGLE || lane_own < last ? lane_own : last;
            const int64_t col = SINGLE ? lane_own : lane0 + threadIdx.x % kMaxCols;
            uint32_t m = 0u;
#pragma unroll
            for (int k = 0; k < kTy; ++k) m = max(m, s_col[k][threadIdx.x]);
            if (m && lane_own < q.cols) {
                if (t.whole) q.sb[col] = __uint_as_float(m);
                else atomicMax(reinterpret_cast<unsigned int*>(q.sb) + col, m);
            }
        }
        if (strip + 1 < end) __syncthreads();
    }
    for (int k = threadIdx.x; k < n; k += kThreads)
        if (s_row[k]) atomicMax(reinterpret_cast<unsigned int*>(q.sa) + row0 + k, s_row[k]);
}

// second moment, after the maxima: codes against min(r_i, c_j)
template <int UNITS>
__global__ __launch_bounds__(kThreads) void quant_v_code_kernel(const QuantArgs q) {
    const int64_t wg_first = int64_t(blockIdx.x) * (UNITS * kCvtUnitElems);
    const CvtOrigin o = cvt_origin(wg_first, q.cols);
    float x[UNITS][4], s[UNITS][4];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const uint32_t off = u * kCvtUnitElems + threadIdx.x * 4;
        cvt_load4<true>(q.x_in, wg_first + off, q.P, x[u]);
        rank1_scales4(o, off, q.rows, q.sa, q.sb, s[u]);
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u)
        cvt_store_codes(q.q_out, wg_first + u * kCvtUnitElems + threadIdx.x * 4, q.P, linear_codes4(x[u], s[u]));
}

// zero two float arrays in one launch (row and column maxima before they are raised)
__global__ __launch_bounds__(kThreads) void clear_two_kernel(float* a, int64_t na, float* b, int64_t nb) {
    const int64_t stride = int64_t(gridDim.x) * kThreads;
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < na + nb; i += stride) {
        if (i < na) a[i] = 0.0f;
        else b[i - na] = 0.0f;
    }
}

}  // namespace lpmm

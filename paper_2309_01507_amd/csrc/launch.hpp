// The __global__ kernels of the optimizer steps: thin wrappers around the tile functions of kernels.hpp and ragged.hpp for
// one tensor, the phase kernels of the multi-tensor plans, and the small kernels between and around them.
#pragma once

#include <type_traits>

#include "kernels.hpp"
#include "ragged.hpp"

namespace lpmm {

// =====================================================================================================
// Kernels for one tensor: two launches per step.
// =====================================================================================================

template <bool BF16>
__global__ __launch_bounds__(kThreads) void maxima_fast(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) maxima_tile<BF16>(a, h, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void update_fast(const Tensor4 a, const Hyper h) {
    __shared__ LdsRank1 s;
    __shared__ int s_last[2];
    const int wg = logical_wg(a.skew2);
    if (wg >= a.n_wg2) return;
    TicketSync sync{a.counter, unsigned(wg), 0u};
    update_tile<BF16, false>(a, h, wg, s, sync);
    finish_rank1(a, unsigned(wg), unsigned(a.n_wg2), sync.ticket, s_last);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void b128_kernel(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) b128_work<BF16>(a, h, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_stats_fast(const Tensor4 a) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) factor_stats_tile<BF16>(a, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_update_fast(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    __shared__ int s_last;
    const int wg = logical_wg(a.skew2);
    if (wg >= a.n_wg2) return;
    TicketSync sync{a.counter, unsigned(wg), 0u};
    factor_update_tile<BF16>(a, h, wg, s, sync);
    if (ticket_is_last(a.counter, unsigned(wg), unsigned(a.n_wg2), sync.ticket, s_last)) factor_publish(a, h);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_stats_general(const Tensor4 a) {
    __shared__ Lds s;
    factor_stats_general_tile<BF16>(a, blockIdx.x, gridDim.x, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_update_general(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    __shared__ int s_last;
    load_tables(s);
    factor_update_general_tile<BF16>(a, h, blockIdx.x, s);
    if (last_to_arrive(a.counter, blockIdx.x, gridDim.x, s_last)) factor_publish(a, h);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_stats_ragged_kernel(const Tensor4 a) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) factor_stats_ragged<BF16>(a, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void factor_update_ragged_kernel(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    __shared__ int s_last;
    const int wg = logical_wg(a.skew2);
    if (wg < a.n_wg2) factor_update_ragged<BF16>(a, h, wg, s);
    if (last_to_arrive(a.counter, blockIdx.x, gridDim.x, s_last)) factor_publish(a, h);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void sgdm4_kernel(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) b128_work<BF16, true>(a, h, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void sgdm32_kernel(float* p, const void* g, float* m, int64_t n, const Hyper h) {
    sgdm32_tile<BF16>(p, g, m, n, h, blockIdx.x);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void pass1_general(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    pass1_general_tile<BF16>(a, h, blockIdx.x, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void pass2_general(const Tensor4 a, const Hyper h) {
    __shared__ int s_last[2];
    pass2_general_chunk<BF16>(a, h, int64_t(blockIdx.x) * kGenChunkElems);
    __syncthreads();
    finish_rank1(a, blockIdx.x, gridDim.x, take_ticket(a.counter, blockIdx.x), s_last);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void maxima_ragged_kernel(const Tensor4 a, const Hyper h) {
    __shared__ Lds s;
    const int wg = logical_wg(a.skew);
    if (wg < a.n_wg) maxima_ragged<BF16>(a, h, wg, s);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void update_ragged_kernel(const Tensor4 a, const Hyper h) {
    __shared__ LdsRank1 s;
    __shared__ int s_last[2];
    const int wg = logical_wg(a.skew2);
    if (wg >= a.n_wg2) return;
    TicketSync sync{a.counter, unsigned(wg), 0u};
    update_ragged<BF16, false>(a, h, wg, s, sync);
    finish_rank1(a, unsigned(wg), unsigned(a.n_wg2), sync.ticket, s_last);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void adamw32_kernel(float* p, const void* g, float* m, float* v,
                                                           int64_t n, const Hyper h) {
    adamw32_tile<BF16>(p, g, m, v, n, h, blockIdx.x);
}

// =====================================================================================================
// Phase kernel of the multi-tensor step.  A phase has the "A" work of one set of tensors (first passes
// of tensors with two, the whole step of the others) and the "B" work of the previous set (second
// passes).  By default each is a launch of its own; in one launch they are interleaved in proportion.
// =====================================================================================================

// Hyper-parameters of a plan's launches: by value, or -- for a step that is captured into a graph and replayed
// while the learning rate and the step number change -- read from device memory, where a one-thread kernel
// enqueued in front of the step has put them.
struct HyperArg {
    Hyper h;
    const Hyper* dev;       // non-null: use *dev
};
__device__ __forceinline__ Hyper resolve(const HyperArg& a) { return a.dev ? *a.dev : a.h; }

// the host's make_hyper on the device: lr and the step number come from device memory
__global__ void hyper_prepare_kernel(const float* lr_dev, const int64_t* step_dev, float beta1, float beta2, float eps,
                                     float wd, Hyper* out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double lr = double(*lr_dev);
    int64_t t = *step_dev;
    if (t < 1) t = 1;
    Hyper h;
    h.beta1 = beta1;
    h.beta2 = beta2;
    h.omb1 = 1.0f - beta1;
    h.omb2 = 1.0f - beta2;
    h.eps = eps;
    const double bc1 = 1.0 - pow(double(beta1), double(t));
    const double bc2 = 1.0 - pow(double(beta2), double(t));
    h.step_size = float(lr / bc1);
    h.inv_sqrt_bc2 = float(1.0 / sqrt(bc2));
    h.lr_wd = float(lr * double(wd));
    *out = h;
}
__global__ void sgdm_hyper_prepare_kernel(const float* lr_dev, float momentum, Hyper* out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    Hyper h{};
    h.beta1 = momentum;
    h.step_size = *lr_dev;
    *out = h;
}

struct Segment {        // a run of workgroups that work on one tensor
    int wg_begin;       // first workgroup of the run, in its kind's numbering
    int tensor;         // index into the tensor table
};

// Tensors per kind in one phase; the tables travel as kernel arguments (3 KiB of the 4 KiB a launch may carry).
// As many as fit: sets of a few hundred small tensors run fastest as a single group (the 108 M-parameter set of 197
// tensors by phases: 0.361 ms per step as one group against 0.397 as two with their passes overlapped).
constexpr int kMaxSeg = 192;

struct Phase {
    const Tensor4Table* tensors;
    int n_seg_a, n_seg_b;
    int n_a, n_b;           // workgroups of each kind
    int skew_a, skew_b;     // of a launch of one kind, see logical_wg
    Segment seg_a[kMaxSeg];
    Segment seg_b[kMaxSeg];
};

static_assert(sizeof(Phase) + sizeof(HyperArg) <= 4000, "kernel arguments of a phase launch");

// the hyper-parameters as they apply to one tensor of a plan
__device__ __forceinline__ Hyper for_tensor(const Hyper& h, const Tensor4& a) {
    Hyper t = h;
    if (a.no_decay) t.lr_wd = 0.0f;
    return t;
}

// last segment whose first workgroup is <= wg (segments are sorted by wg_begin, seg[0].wg_begin = 0;
// a uniform binary search on scalar registers)
__device__ __forceinline__ Segment find_segment(const Segment* seg, int n_seg, int wg) {
    int lo = 0, hi = n_seg;                 // answer in [lo, hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg[mid].wg_begin <= wg) lo = mid; else hi = mid;
    }
    return seg[lo];
}

// ROLES: 0 = A and B work interleaved in one launch; 1 = A work only; 2 = B work only; 3 = A work
// only of a group without rank-1 tensors (block-wise and fp32-state tensors: no rank-1 code); 4 = B work only of tensors on
// the general tiles.  The single-role kernels exist because a kernel's register and LDS footprint is that of its heaviest
// path.  PLAIN: for plans with rows of whole blocks only, without the ragged and the general tiles, of which the ragged statistics take 89
// registers (fp32; bf16 92) where the plain ones take 73 (78), and the factorized form's 74 (78) where 66 (62) do.  Sets of a few matrices, where latency
// counts, us with them and without, bf16: rank-1 4 of 1024 x 1024 18.1, 17.9, 2 of 512 x 512 11.7, 11.2, a layer of width 1024 35.9, 35.5;
// factorized 20.8, 19.5, 12.1, 11.3, 38.4, 37.5; 8 of 4096 x 4096 the same.  Long factorized launches keep the second pass with them
// (the host's rule has the figures).
template <bool BF16, int ROLES, bool PLAIN = false>
__global__ __launch_bounds__(kThreads) void phase_kernel(const Phase ph, const HyperArg ha) {
    const Hyper h = resolve(ha);
    constexpr bool kOnlyA = ROLES == 1 || ROLES == 3;
    constexpr bool kOnlyB = ROLES == 2 || ROLES == 4;
    __shared__ std::conditional_t<kOnlyA, Lds, LdsRank1> s;
    const int x = ROLES == 2 ? logical_wg_or_dealt(ph.skew_b) : logical_wg(kOnlyB ? ph.skew_b : ph.skew_a);
    const int n = (kOnlyB ? 0 : ph.n_a) + (kOnlyA ? 0 : ph.n_b);
    if (x >= n) return;
    // B workgroups sit at the positions where floor(x * n_b / n) steps up
    const int b_before = kOnlyA ? 0 : (kOnlyB ? x : int((int64_t(x) * ph.n_b) / n));
    const int b_after = kOnlyA ? 0 : (kOnlyB ? x + 1 : int((int64_t(x + 1) * ph.n_b) / n));
    if (!kOnlyA && b_after > b_before) {
        __shared__ int s_last[2];
        const Segment sg = find_segment(ph.seg_b, ph.n_seg_b, b_before);
        const Tensor4 a = from_table(ph.tensors[sg.tensor]);
        const Hyper ht = for_tensor(h, a);
        const int wg = b_before - sg.wg_begin;
        TicketSync sync{a.counter, unsigned(wg), 0u};
        if (ROLES == 4 || (!PLAIN && a.kind == kQuantGeneral)) {
            pass2_general_chunk<BF16>(a, h, int64_t(wg) * kGenChunkElems);
            __syncthreads();
            sync.staged();
        } else if constexpr (!kOnlyA && ROLES != 4) {
            if (PLAIN || a.kind == kQuantFast) update_tile<BF16, false>(a, ht, wg, s, sync);
            else update_ragged<BF16, false>(a, ht, wg, s, sync);
        }
        finish_rank1(a, unsigned(wg), unsigned(a.n_wg2), sync.ticket, s_last);
    } else if (!kOnlyB) {
        const int xa = x - b_before;
        const Segment sg = find_segment(ph.seg_a, ph.n_seg_a, xa);
        const Tensor4 a = from_table(ph.tensors[sg.tensor]);
        const Hyper ht = for_tensor(h, a);
        const int wg = xa - sg.wg_begin;
        if (a.kind == kFp32State) {
            adamw32_tile<BF16>(a.p, a.g, reinterpret_cast<float*>(a.mq), reinterpret_cast<float*>(a.vq), a.P, ht, wg);
        } else if (a.kind == kQuantBlockV) {
            b128_work<BF16>(a, ht, wg, s);
        } else if (ROLES == 3) {
            // not reached: the host launches this variant only for groups without rank-1 tensors
        } else if (PLAIN || a.kind == kQuantFast) {
            maxima_tile<BF16>(a, ht, wg, s);
        } else if (a.kind == kQuantRagged) {
            maxima_ragged<BF16>(a, ht, wg, s);
        } else {
            pass1_general_tile<BF16>(a, ht, wg, s);
        }
    }
}

// =====================================================================================================
// Rank-1 normalization of a tensor with more than two dimensions (App. F Alg. 4): one statistic per
// index of every dimension, an element's scale is the minimum of its statistics.  Seen as a matrix of
// d_1 rows and d_2 * ... * d_p columns, the scale is min(mu_1[i], colscale[col]) with colscale[col] =
// min over the other dimensions of their statistic at the column's index: the two passes of the
// matrix step run unchanged on (mu_1, colscale), and two small kernels between them turn the column
// maxima of v_t into the new statistics (reduce) and those into the new colscale (expand).
// =====================================================================================================

constexpr int kMaxInnerDims = 7;

struct InnerDims {                  // dimensions 2..p
    int n;
    int64_t d[kMaxInnerDims];       // sizes
    int64_t first[kMaxInnerDims];   // where each dimension's statistics start in the statistics array
};

// One workgroup per statistic: mu_new[first[r] + j] = max of colmax over the columns whose index in inner
// dimension r is j (cols / d_r of them: col = a * d_r * inner + j * inner + b).  No atomics: with a small
// dimension (a 3 x 3 kernel) thousands of columns share a statistic, and atomics on one address queue up.
// `stat` = which statistic this workgroup computes (0 .. d_2 + ... + d_p - 1).
__device__ __forceinline__ void nd_reduce_one(const float* colmax, float* mu_new, int64_t cols, const InnerDims& dm,
                                              int64_t stat, float* s_part) {
    int r = 0;
    int64_t j = stat;
    while (r < dm.n - 1 && j >= dm.d[r]) { j -= dm.d[r]; ++r; }
    int64_t inner = 1;
    for (int q = r + 1; q < dm.n; ++q) inner *= dm.d[q];
    const int64_t count = cols / dm.d[r];
    float m = 0.0f;
    for (int64_t k = threadIdx.x; k < count; k += kThreads) {
        const int64_t a = k / inner, b = k - a * inner;
        m = fmaxf(m, colmax[(a * dm.d[r] + j) * inner + b]);
    }
    m = row16_allmax(m);                    // values are >= +0
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) mu_new[dm.first[r] + j] = fmaxf(fmaxf(s_part[0], s_part[1]), fmaxf(s_part[2], s_part[3]));
}

// colscale[col] = min over the inner dimensions of mu[first[r] + idx_r(col)]
__device__ __forceinline__ void nd_expand_one(const float* mu, float* colscale, int64_t cols, const InnerDims& dm,
                                              int64_t col) {
    if (col >= cols) return;
    int64_t rest = col;
    float m = 0.0f;
    for (int r = dm.n - 1; r >= 0; --r) {
        const int64_t idx = rest % dm.d[r];
        rest /= dm.d[r];
        const float v = mu[dm.first[r] + idx];
        m = (r == dm.n - 1) ? v : fminf(m, v);
    }
    colscale[col] = m;
}

__global__ __launch_bounds__(kThreads) void nd_reduce_kernel(const float* colmax, float* mu_new, int64_t cols,
                                                             const InnerDims dm) {
    __shared__ float s_part[kThreads / 64];
    nd_reduce_one(colmax, mu_new, cols, dm, blockIdx.x, s_part);
}

__global__ __launch_bounds__(kThreads) void nd_expand_kernel(const float* mu, float* colscale, int64_t cols,
                                                             const InnerDims dm) {
    nd_expand_one(mu, colscale, cols, dm, int64_t(blockIdx.x) * kThreads + threadIdx.x);
}

// The two small kernels between the passes for all tensors with more than two dimensions of one group of a plan.
struct NdPhase {
    const Tensor4Table* tensors;
    const InnerDims* dims;          // device table, indexed by Tensor4::nd_index
    int n_seg, n_r, n_e;            // tensors; workgroups of the reduce and of the expand kernel
    Segment seg_r[kMaxSeg];         // per tensor: first workgroup of the reduce kernel (one per statistic)
    Segment seg_e[kMaxSeg];         // per tensor: first workgroup of the expand kernel (one per 256 columns)
};

static_assert(sizeof(NdPhase) <= 4000, "kernel arguments of the reduce / expand launches");

__global__ __launch_bounds__(kThreads) void nd_plan_reduce(const NdPhase ph) {
    __shared__ float s_part[kThreads / 64];
    const int x = blockIdx.x;
    if (x >= ph.n_r) return;
    const Segment sg = find_segment(ph.seg_r, ph.n_seg, x);
    const Tensor4 a = from_table(ph.tensors[sg.tensor]);
    const InnerDims dm = ph.dims[a.nd_index];
    nd_reduce_one(a.c_new, a.c_new + a.cols, a.cols, dm, x - sg.wg_begin, s_part);
}

__global__ __launch_bounds__(kThreads) void nd_plan_expand(const NdPhase ph) {
    const int x = blockIdx.x;
    if (x >= ph.n_e) return;
    const Segment sg = find_segment(ph.seg_e, ph.n_seg, x);
    const Tensor4 a = from_table(ph.tensors[sg.tensor]);
    const InnerDims dm = ph.dims[a.nd_index];
    nd_expand_one(a.c_new + a.cols, a.c_new, a.cols, dm, int64_t(x - sg.wg_begin) * kThreads + threadIdx.x);
}

// The reduce and totals steps for all tensors with deterministic sums of one group of a plan.
struct DetPhase {
    const Tensor4Table* tensors;
    int n_seg, n_r;                 // tensors; workgroups of the reduce kernel
    Segment seg_r[kMaxSeg];         // per tensor: first workgroup of the reduce kernel
};

__global__ __launch_bounds__(kThreads) void factor_plan_reduce(const DetPhase ph) {
    __shared__ float s_part[kThreads / 64];
    const int x = blockIdx.x;
    if (x >= ph.n_r) return;
    const Segment sg = find_segment(ph.seg_r, ph.n_seg, x);
    factor_reduce_one(from_table(ph.tensors[sg.tensor]), x - sg.wg_begin, s_part);
}

__global__ __launch_bounds__(kThreads) void factor_plan_totals(const DetPhase ph) {
    __shared__ float s_part[kThreads / 64];
    if (int(blockIdx.x) >= ph.n_seg) return;
    factor_totals_one(from_table(ph.tensors[ph.seg_r[blockIdx.x].tensor]), s_part);
}

// The same for a plan whose 2-dimensional tensors keep a factorized second moment: "A" work is the
// statistics pass (next to block-wise and fp32-state tensors, which are complete after it), "B" work
// the update pass.  ROLES: 0 = both interleaved, 1 = A only, 2 = B only.  Separate kernels, so that the
// rank-1 kernels above keep their register footprint.
template <bool BF16, int ROLES, bool PLAIN = false>
__global__ __launch_bounds__(kThreads) void factor_phase_kernel(const Phase ph, const HyperArg ha) {
    const Hyper h = resolve(ha);
    __shared__ Lds s;
    const int x = logical_wg(ROLES == 2 ? ph.skew_b : ph.skew_a);
    const int n = (ROLES == 2 ? 0 : ph.n_a) + (ROLES == 1 ? 0 : ph.n_b);
    if (x >= n) return;
    const int b_before = ROLES == 1 ? 0 : (ROLES == 2 ? x : int((int64_t(x) * ph.n_b) / n));
    const int b_after = ROLES == 1 ? 0 : (ROLES == 2 ? x + 1 : int((int64_t(x + 1) * ph.n_b) / n));
    if (ROLES != 1 && b_after > b_before) {
        __shared__ int s_last;
        const Segment sg = find_segment(ph.seg_b, ph.n_seg_b, b_before);
        const Tensor4 a = from_table(ph.tensors[sg.tensor]);
        const Hyper ht = for_tensor(h, a);
        const int wg = b_before - sg.wg_begin;
        NoSync sync;            // the ticket at the end: six of 1024 x 1024 fp32 26.1 us, 26.5 with it in the tile's middle
        if (PLAIN || a.kind == kFactorFast) {
            factor_update_tile_down<BF16, false>(a, ht, wg, s, sync);
        } else if (a.kind == kFactorRagged) {
            factor_update_ragged<BF16>(a, ht, wg, s);
        } else {
            load_tables(s);
            factor_update_general_tile<BF16>(a, ht, wg, s);
        }
        if (last_to_arrive(a.counter, unsigned(wg), unsigned(a.n_wg2), s_last)) factor_publish(a, h);
    } else if (ROLES != 2) {
        const int xa = x - b_before;
        const Segment sg = find_segment(ph.seg_a, ph.n_seg_a, xa);
        const Tensor4 a = from_table(ph.tensors[sg.tensor]);
        const int wg = xa - sg.wg_begin;
        const Hyper ht = for_tensor(h, a);
        if (a.kind == kFp32State)
            adamw32_tile<BF16>(a.p, a.g, reinterpret_cast<float*>(a.mq), reinterpret_cast<float*>(a.vq), a.P, ht, wg);
        else if (a.kind == kQuantBlockV) b128_work<BF16>(a, ht, wg, s);
        else if (PLAIN || a.kind == kFactorFast) factor_stats_tile<BF16>(a, wg, s);
        else if (a.kind == kFactorRagged) factor_stats_ragged<BF16>(a, wg, s);
        else factor_stats_general_tile<BF16>(a, wg, a.n_wg, s);
    }
}

// A plan of SGD-with-momentum tensors (App. E Alg. 2): everything is one pass, so only "A" work exists.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void sgdm_phase_kernel(const Phase ph, const HyperArg ha) {
    const Hyper h = resolve(ha);
    __shared__ Lds s;
    const int x = logical_wg(ph.skew_a);
    if (x >= ph.n_a) return;
    const Segment sg = find_segment(ph.seg_a, ph.n_seg_a, x);
    const Tensor4 a = from_table(ph.tensors[sg.tensor]);
    const int wg = x - sg.wg_begin;
    if (a.kind == kSgdmFp32) sgdm32_tile<BF16>(a.p, a.g, reinterpret_cast<float*>(a.mq), a.P, h, wg);
    else b128_work<BF16, true>(a, h, wg, s);
}

// =====================================================================================================
// The zero state.
// =====================================================================================================

// fill `n` bytes at dst with `value`, and force the byte at index `last_index` (if >= 0) to `last`
__global__ __launch_bounds__(kThreads) void fill_bytes_kernel(uint8_t* dst, int64_t n, uint8_t value,
                                                              int64_t last_index, uint8_t last) {
    const int64_t stride = int64_t(gridDim.x) * kThreads;
    for (int64_t i = int64_t(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride)
        dst[i] = (i == last_index) ? last : value;
}

}  // namespace lpmm

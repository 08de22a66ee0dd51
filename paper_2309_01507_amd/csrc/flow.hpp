// One launch for a whole plan step.
//
// The rank-1 and the factorized step read every gradient twice, once per pass (2 or 4 of their 13 to 19 bytes per
// parameter).  As launches of their own the passes of a large group are gigabytes apart and the second reading comes from
// HBM.  Here both passes of all tensors are ONE launch whose work list (built with the plan) puts pass 2 of a tensor a
// little behind its pass 1: the gradient and the codes of a tensor of a few million parameters are then still in the
// memory-side cache, whose reads cost nothing beside the HBM traffic of the following tensors' pass 1.  (Probe without
// arithmetic: an in-place stream of 8 GB takes 1.575 ms, with 4.3 GB of re-reads from a region of at most 128 MB beside it
// 1.58, from HBM 2.26; pass 1's and pass 2's streams over 2^31 parameters in tensors of at most 8.4 M 4.98 ms, of 50 M 5.2, of
// 134 M 5.65, the same as by phases.)  It also spares the step the starts and the tails of its launches, and tiles of unequal
// cost do not leave XCDs idle.
//
// Order inside the launch.  Pass 2 of a tensor needs its complete maxima (sums): a workgroup of pass 1 waits for its own
// atomics and then raises the tensor's count, a workgroup of pass 2 polls that count.  Workgroups are started in the order
// of their ids as far as the hardware is known to do it, so the count is usually complete long before; but nothing
// promises that order, so the polling is BOUNDED and no workgroup ever waits for one that might not run: a workgroup that
// has polled `spin_limit` times writes its tile to the tensor's list of deferred tiles and leaves.  The last workgroup of
// the tensor to finish -- of either pass: `final` counts "pass 1 complete" and "pass 2 complete" -- does the deferred
// tiles, then publishes the new statistics and clears the workspace.  Every workgroup ends after a bounded time in any
// order of execution, and the results do not depend on it.
//
// What crosses workgroups inside the launch is only the workspace (maxima, sums, counters): written with device-scope
// atomics that have completed (s_waitcnt) before the count is raised, and read with agent-scope loads (ld_ws).  Codes and
// parameters are read and written by one workgroup each per pass; pass 2 overwrites codes that pass 1 of the tensor has
// finished reading.
#pragma once

#include "launch.hpp"

namespace lpmm {

struct FlowItem {       // one workgroup's work
    int what;           // index of the tensor, kFlowSecond added for its second pass; -1: nothing
    int wg;             // the workgroup's number in that pass
};
constexpr int kFlowSecond = 1 << 30;

struct FlowArgs {
    const Tensor4Table* tensors;
    const FlowItem* items;
    const InnerDims* dims;
    int* deferred;          // per tensor n_wg2 entries, from Tensor4::deferred on
    int n_items;            // a multiple of 8
    int spin_limit;
};

// words in the last line of a tensor's counter block (plans use one line for the factorized sums)
__device__ __forceinline__ unsigned int* flow_word(const Tensor4& a, int k) {
    return a.counter + (1 + kTicketLanes + kMaxTotSlots - 1) * kTicketStride + k;
}
enum { kFlowFinal = 0, kFlowDeferred = 1 };
// The finished workgroups of pass 1 are counted in two levels like those of pass 2, in words of their own next to theirs.
// All of them on one word, the one that pass 2 polls, made the memory system serve the polls of several hundred waiting
// workgroups between the counts: one 4096 x 4096 matrix 147 us, 69 this way, and 90 us more than now in any plan whose last
// tensors are of that size.
__device__ __forceinline__ unsigned int* flow_done(const Tensor4& a) { return a.counter + kTicketStride / 2; }

__device__ __forceinline__ unsigned int flow_peek(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tensors with more than two dimensions, between the passes, by the workgroup that completes pass 1: statistics of the
// inner dimensions from the column maxima (LDS atomics), then the new column scales in place of the maxima.
constexpr int kFlowNdCols = 16384;                    // columns up to which one workgroup does this
constexpr int kFlowNdStats = 2 * kColSlots;           // statistics that fit s.col and s.cold
__device__ __forceinline__ void flow_nd(const Tensor4& a, const InnerDims& dm, Lds& s) {
    unsigned int* mu = reinterpret_cast<unsigned int*>(s.col);
    for (int k = threadIdx.x; k < a.c_extra; k += kThreads) mu[k] = 0u;
    __syncthreads();
    const int cols = int(a.cols);
    // the whole chip may be waiting for this one workgroup: eight columns per thread at a time, so that their loads (which
    // no cache on this side serves) are in flight together
    constexpr int kBatch = 8;
    auto put = [](float* p, unsigned int v) {
        __hip_atomic_store(reinterpret_cast<unsigned int*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // calls f(u, statistic) for the batch's columns and every inner dimension.  x / d = mulhi(x, floor(2^32 / d) + 1): exact
    // for x * d < 2^32, and both are at most kFlowNdCols here; d = 1 has no such factor and needs no division.
    auto walk = [&](int base, auto&& f) {
        uint32_t rest[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) rest[u] = uint32_t(base + u * kThreads);
        for (int r = dm.n - 1; r >= 0; --r) {
            const uint32_t d = uint32_t(dm.d[r]), first = uint32_t(dm.first[r]);
            const uint32_t inv = 0xFFFFFFFFu / d + (d == 1u ? 0u : 1u);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const uint32_t q = d == 1u ? rest[u] : __umulhi(rest[u], inv);
                f(u, first + (rest[u] - q * d));
                rest[u] = q;
            }
        }
    };
    for (int base = threadIdx.x; base < cols; base += kThreads * kBatch) {
        unsigned int v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            v[u] = base + u * kThreads < cols ? __float_as_uint(ld_ws<true>(a.c_new + base + u * kThreads)) : 0u;
        walk(base, [&](int u, uint32_t k) {
            if (base + u * kThreads < cols)
                (void)__hip_atomic_fetch_max(mu + k, v[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        });
    }
    __syncthreads();
    for (int base = threadIdx.x; base < cols; base += kThreads * kBatch) {
        unsigned int m[kBatch];                       // non-negative floats order like their bits
#pragma unroll
        for (int u = 0; u < kBatch; ++u) m[u] = 0xFFFFFFFFu;
        walk(base, [&](int u, uint32_t k) {
            const unsigned int v = base + u * kThreads < cols ? mu[k] : 0u;
            m[u] = v < m[u] ? v : m[u];
        });
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (base + u * kThreads < cols) put(a.c_new + base + u * kThreads, m[u]);
    }
    for (int k = threadIdx.x; k < a.c_extra; k += kThreads) put(a.c_new + cols + k, mu[k]);
}

// every memory operation of this workgroup has been performed when thread 0 returns from here
__device__ __forceinline__ void flow_drain() {
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
}

template <bool BF16, bool FACTOR>
__global__ __launch_bounds__(kThreads) void flow_kernel(const FlowArgs f, const HyperArg ha) {
    __shared__ Lds s;
    __shared__ int s_flag;
    const Hyper h = resolve(ha);
    const FlowItem it = f.items[blockIdx.x];
    if (it.what < 0) return;
    const bool second = it.what & kFlowSecond;
    const Tensor4 a = from_table(f.tensors[it.what & (kFlowSecond - 1)]);
    const Hyper ht = for_tensor(h, a);
    const bool nd = !FACTOR && a.nd_index >= 0 && a.kind != kFp32State && a.kind != kQuantBlockV;
    const unsigned int target = lanes_used(unsigned(a.n_wg)) + (nd ? 1u : 0u);

    if (!second) {
        if (a.kind == kFp32State) {
            adamw32_tile<BF16>(a.p, a.g, reinterpret_cast<float*>(a.mq), reinterpret_cast<float*>(a.vq), a.P, ht, it.wg);
            return;
        }
        if (a.kind == kQuantBlockV) {
            b128_work<BF16>(a, ht, it.wg, s);
            return;
        }
        if constexpr (FACTOR) {
            if (a.kind == kFactorFast) factor_stats_tile<BF16>(a, it.wg, s);
            else factor_stats_general_tile<BF16>(a, it.wg, a.n_wg, s);
        } else {
            if (a.kind == kQuantFast) {
                if (a.flat) pass1_flat_tile<BF16>(a, ht, it.wg, s);
                else pass1_fast_tile<BF16>(a, ht, it.wg, s);
            } else if (a.kind == kQuantRagged) {
                pass1_ragged<BF16>(a, ht, it.wg, s);
            } else {
                pass1_general_tile<BF16>(a, ht, it.wg, s);
            }
        }
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);          // the maxima and sums have been sent: count this workgroup
        if (!last_to_arrive(flow_done(a), unsigned(it.wg), unsigned(a.n_wg), s_flag)) return;
        if (nd) {
            flow_nd(a, f.dims[a.nd_index], s);
            flow_drain();
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            if (nd) (void)atomicAdd(flow_done(a), 1u);
            s_flag = atomicAdd(flow_word(a, kFlowFinal), 1u) == 1u;
        }
        __syncthreads();
        if (!s_flag) return;
    }
    // Second pass: this workgroup's tile if it is one of that pass, and, in the workgroup that finishes the tensor, the
    // tiles that were deferred.
    int wg = it.wg, n_left = 0;
    bool mine = second;
    int* deferred = f.deferred + a.deferred;
    // the same value in every lane: say so, the tile functions address through scalar registers
    auto n_deferred = [&] { return __builtin_amdgcn_readfirstlane(int(flow_peek(flow_word(a, kFlowDeferred)))); };
    auto take = [&](int k) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(deferred + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    if (!second) {
        n_left = n_deferred();
        if (n_left > 0) wg = take(n_left - 1);
    }
    while (mine || n_left > 0) {
        // polls for the tensor's first pass (a deferred tile's is complete); the same answer in every thread
        auto ready = [&]() -> bool {
            if (!mine) return true;
            if (threadIdx.x == 0) {
                int ok = 0;
                for (int k = 0; k <= f.spin_limit; ++k) {
                    ok = flow_peek(flow_done(a)) == target;
                    if (ok) break;
                    __builtin_amdgcn_s_sleep(64);
                }
                s_flag = ok;
            }
            __syncthreads();
            return s_flag != 0;
        };
        if constexpr (FACTOR) {
            if (a.kind == kFactorFast) {
                factor_update_tile<BF16, true>(a, ht, wg, s, ready);
            } else if (ready()) {
                load_tables(s);
                factor_update_general_tile<BF16, true>(a, ht, wg, s);
            }
        } else {
            if (a.kind == kQuantFast) pass2_tile<BF16, false, true>(a, h, wg, ready, s);
            else if (a.kind == kQuantRagged) pass2_ragged<BF16, true>(a, h, wg, ready, s);
            else if (ready()) pass2_general_chunk<BF16, true>(a, h, int64_t(wg) * kGenChunkElems);
        }
        if (mine) {
            mine = false;
            if (!s_flag && threadIdx.x == 0) {
                const unsigned int k = atomicAdd(flow_word(a, kFlowDeferred), 1u);
                __hip_atomic_store(deferred + k, wg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            }
            if (!last_to_arrive(a.counter, unsigned(wg), unsigned(a.n_wg2), s_flag)) return;
            __syncthreads();                              // every wave has read the flag before it is written again
            if (threadIdx.x == 0) s_flag = atomicAdd(flow_word(a, kFlowFinal), 1u) == 1u;
            __syncthreads();
            if (!s_flag) return;
            n_left = n_deferred();
        } else {
            --n_left;
            __syncthreads();                              // LDS of the tile just done is free again
        }
        if (n_left > 0) wg = take(n_left - 1);
    }
    if constexpr (FACTOR) {
        ema_and_clear<true>(h, a.r, a.r_new, a.rows);
        ema_and_clear<true>(h, a.c, a.c_new, a.cols);
        if (int(threadIdx.x) < a.tot_slots) {
            a.counter[tot_new_word(threadIdx.x)] = 0u;
            a.counter[tot_old_word(threadIdx.x)] = 0u;
        }
    } else {
        move_and_clear<true>(a.r, a.r_new, a.rows);
        move_and_clear<true>(a.c, a.c_new, a.cols + a.c_extra);
    }
    if (threadIdx.x == 0) {
        *a.counter = 0u;
        *flow_done(a) = 0u;
        *flow_word(a, kFlowFinal) = 0u;
        *flow_word(a, kFlowDeferred) = 0u;
    }
}

}  // namespace lpmm

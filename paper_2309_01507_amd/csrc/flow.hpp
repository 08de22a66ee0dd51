// One launch for a whole plan step.
//
// The rank-1 and the factorized step read every gradient twice, once per pass (2 or 4 of their 13 to 19 bytes per parameter).
// As launches of their own the passes of a large group are gigabytes apart and the second reading comes from HBM.  Here both
// passes of all tensors are ONE launch whose work list (built with the plan) puts the first pass of a tensor, which only reads
// gradients and codes and leaves its statistics, a little ahead of its second one, which does everything else: what the first
// one read is still in the memory-side cache then, where the parameters' streams leave no trace (non-temporal).  (Probe without
// arithmetic, 2^31 parameters with bf16 gradients: second passes alone 3.98 ms, first ones 0.83, both in turn 4.10 to 4.43 for
// tensors of 2^22 to 2^26, 4.67 for 2^27; the update first and the codes 2^23 parameters behind 4.83.)  It also spares the step
// the starts and the tails of its launches, and tiles of unequal cost do not leave XCDs idle.
//
// Order inside the launch.  The second pass of a tensor needs its complete maxima (sums): a workgroup of the first waits for its own
// atomics and then raises the tensor's count, a workgroup of the second polls that count.  Workgroups are started in the order
// of their ids as far as the hardware is known to do it, so the count is usually complete long before; but nothing
// promises that order, so the polling is BOUNDED and no workgroup ever waits for one that might not run: a workgroup that
// has polled `spin_limit` times writes its tile to the tensor's list of deferred tiles and leaves.  The last workgroup of
// the tensor to finish -- of either pass: `final` counts "first pass complete" and "second pass complete" -- does the deferred
// tiles, then publishes the new statistics and clears the workspace.  Every workgroup ends after a bounded time in any
// order of execution, and the results do not depend on it.
//
// What crosses workgroups inside the launch is only the workspace (maxima, sums, counters): written with device-scope
// atomics that have completed (s_waitcnt) before the count is raised, and read with agent-scope loads (ld_ws).  Codes and
// parameters are read and written by one workgroup each per pass; pass 2 overwrites codes that pass 1 of the tensor has
// finished reading.
#pragma once

#include <type_traits>

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
// The finished workgroups of first passes are counted in two levels like those of second ones, in words of their own next to theirs.
// All of them on one word, the one that is polled, made the memory system serve the polls of several hundred waiting
// workgroups between the counts: one 4096 x 4096 matrix 147 us, 69 this way, and 90 us more than now in any plan whose last
// tensors are of that size.
__device__ __forceinline__ unsigned int* flow_done(const Tensor4& a) { return a.counter + kTicketStride / 2; }

__device__ __forceinline__ unsigned int flow_peek(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tensors with more than two dimensions, between the passes, by the workgroup that completes the first: statistics of the
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

// FORM: which tensors the plan has.  Rank-1 plans without ragged matrices and without rows shorter than 128 elements take
// a kernel of their own: with the tiles of those in it, it needs 128 registers in place of 96, four waves on a SIMD in place
// of five.  (Launch bounds: at 80 registers and six waves the plain form spills, 8 llama-like layers 4.44 ms, 4.27 at five,
// 4.31 at four; the other form at 96 registers 597 us for rows of 1088, 576 at 128.)
enum { kFlowFactor = 0, kFlowRank1 = 1, kFlowRank1Any = 2 };
template <bool BF16, int FORM>
__global__ __launch_bounds__(kThreads, FORM == kFlowRank1 ? 5 : FORM == kFlowRank1Any ? 4 : 6) void flow_kernel(const FlowArgs f, const HyperArg ha) {
    constexpr bool FACTOR = FORM == kFlowFactor;
    constexpr bool kAny = FORM == kFlowRank1Any;
    __shared__ std::conditional_t<FACTOR, Lds, LdsRank1> s;
    __shared__ int s_flag;
    // what lies in LDS differs from lane to lane as far as the compiler knows: say that it does not, so that branches on it
    // are scalar and what the tiles address with stays in scalar registers
    auto flag = [&] { return __builtin_amdgcn_readfirstlane(s_flag) != 0; };
    const Constant<FlowItem> item = as_constant(f.items + blockIdx.x);
    const FlowItem it{item->what, item->wg};
    if (it.what < 0) return;
    const bool second = it.what & kFlowSecond;
    // Read again wherever it is needed, not kept: a tile needs most of the scalar registers for itself.
    auto tensor = [&] {
        Constant<Tensor4Table> entry = as_constant(f.tensors + (it.what & (kFlowSecond - 1)));
        asm volatile("" : "+s"(entry));
        return from_table(*entry);
    };
    auto is_nd = [](const Tensor4& a) { return !FACTOR && a.nd_index >= 0 && a.kind != kFp32State && a.kind != kQuantBlockV; };

    if (!second) {
        {
            const Tensor4 a = tensor();
            const Hyper h = for_tensor(resolve(ha), a);
            if (a.kind == kFp32State) {
                adamw32_tile<BF16>(a.p, a.g, reinterpret_cast<float*>(a.mq), reinterpret_cast<float*>(a.vq), a.P, h, it.wg);
                return;
            }
            if (a.kind == kQuantBlockV) {
                b128_work<BF16>(a, h, it.wg, s);
                return;
            }
            if constexpr (FACTOR) {
                if (a.kind == kFactorFast) factor_stats_tile<BF16>(a, it.wg, s);
                else factor_stats_general_tile<BF16>(a, it.wg, a.n_wg, s);
            } else {
                if (!kAny || a.kind == kQuantFast) maxima_tile<BF16>(a, h, it.wg, s);
                else if (a.kind == kQuantRagged) maxima_ragged<BF16>(a, h, it.wg, s);
                else pass1_general_tile<BF16>(a, h, it.wg, s);
            }
        }
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);          // the maxima and sums have been sent: count this workgroup
        const Tensor4 a = tensor();
        if (!last_to_arrive(flow_done(a), unsigned(it.wg), unsigned(a.n_wg), s_flag)) return;
        const bool nd = is_nd(a);
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
        if (!flag()) return;
    }
    // Second pass: this workgroup's tile if it is one of that pass, and, in the workgroup that finishes the tensor, the
    // tiles that were deferred.
    int wg = it.wg, n_left = 0;
    bool mine = second;
    // the same value in every lane: say so, the tile functions address through scalar registers
    auto n_deferred = [&](const Tensor4& a) { return __builtin_amdgcn_readfirstlane(int(flow_peek(flow_word(a, kFlowDeferred)))); };
    auto take = [&](const Tensor4& a, int k) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(f.deferred + a.deferred + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    if (!second) {
        const Tensor4 a = tensor();
        n_left = n_deferred(a);
        if (n_left > 0) wg = take(a, n_left - 1);
    }
    while (mine || n_left > 0) {
        // ready(): the tensor's first pass is complete (a deferred tile's is); the same answer in every thread.  It usually is long
        // before, and the word read when the tile began says so; only else it is polled.  spin_limit < 0: never, every tile is deferred.
        struct Sync {
            const Tensor4& a;
            const FlowArgs& f;
            int& s_flag;
            const bool mine;
            const int wg;
            const unsigned int target, early;
            bool done = true;
            unsigned int ticket = 0u;
            __device__ __forceinline__ bool ready() {
                if (!mine) return true;
                if (threadIdx.x == 0) s_flag = f.spin_limit >= 0 && early == target;
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(s_flag) != 0) return true;
                __syncthreads();                          // every wave has read the flag before it is written again
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
                done = __builtin_amdgcn_readfirstlane(s_flag) != 0;
                return done;
            }
            __device__ __forceinline__ void staged() {
                if (mine) ticket = take_ticket(a.counter, unsigned(wg));
            }
        };
        unsigned int ticket;
        bool done;
        {
            const Tensor4 a = tensor();
            const Hyper h = for_tensor(resolve(ha), a);
            Sync sync{a, f, s_flag, mine, wg, lanes_used(unsigned(a.n_wg)) + (is_nd(a) ? 1u : 0u), flow_peek(flow_done(a))};
            auto behind = [&](auto tile) {                // tiles that read the statistics all along
                if (!sync.ready()) return;
                tile();
                __syncthreads();
                sync.staged();
            };
            if constexpr (FACTOR) {
                if (a.kind == kFactorFast) factor_update_tile_down<BF16, true>(a, h, wg, s, sync);
                else behind([&] {
                    load_tables(s);
                    factor_update_general_tile<BF16, true>(a, h, wg, s);
                });
            } else {
                if (!kAny || a.kind == kQuantFast) update_tile<BF16, true>(a, h, wg, s, sync);
                else if (a.kind == kQuantRagged) update_ragged<BF16, true>(a, h, wg, s, sync);
                else behind([&] { pass2_general_chunk<BF16, true>(a, h, int64_t(wg) * kGenChunkElems); });
            }
            ticket = sync.ticket;
            done = sync.done;
        }
        const Tensor4 a = tensor();
        if (mine) {
            mine = false;
            if (!done) {
                __syncthreads();                          // every wave has read the answer in s_flag before the ticket writes it
                if (threadIdx.x == 0) {
                    const unsigned int k = atomicAdd(flow_word(a, kFlowDeferred), 1u);
                    __hip_atomic_store(f.deferred + a.deferred + k, wg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
                }
                ticket = take_ticket(a.counter, unsigned(wg));
            }
            if (!ticket_is_last(a.counter, unsigned(wg), unsigned(a.n_wg2), ticket, s_flag)) return;
            __syncthreads();                              // every wave has read the flag before it is written again
            if (threadIdx.x == 0) s_flag = atomicAdd(flow_word(a, kFlowFinal), 1u) == 1u;
            __syncthreads();
            if (!flag()) return;
            n_left = n_deferred(a);
        } else {
            --n_left;
            __syncthreads();                              // LDS of the tile just done is free again
        }
        if (n_left > 0) wg = take(a, n_left - 1);
    }
    const Tensor4 a = tensor();
    if constexpr (FACTOR) {
        const Hyper h = resolve(ha);
        ema_and_clear<true>(h, a.r, a.r_new, a.rows);
        ema_and_clear<true>(h, a.c, a.c_new, a.cols);
        if (int(threadIdx.x) < a.tot_slots) {
            a.counter[tot_new_word(threadIdx.x)] = 0u;
            a.counter[tot_old_word(threadIdx.x)] = 0u;
        }
    } else {
        move_statistics<true>(a, request_statistics<true>(a, 0));
    }
    if (threadIdx.x == 0) {
        *a.counter = 0u;
        *flow_done(a) = 0u;
        *flow_word(a, kFlowFinal) = 0u;
        *flow_word(a, kFlowDeferred) = 0u;
    }
}

}  // namespace lpmm

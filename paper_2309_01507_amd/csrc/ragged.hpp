// Both passes of the rank-1 and of the factorized step for matrices whose rows are no multiple of 128 elements long (or
// whose column maxima are not 16-byte aligned).  First-moment blocks are 128 elements of the row-major FLATTENING, so here
// they start anywhere in a row and may straddle the end of one.
//
// What bounds the step is memory, as on the fast path, so the second pass' work unit is the fast path's: 32 lanes own one
// block, 4 consecutive elements per lane, and every access is aligned because blocks start at multiples of 128 elements.  A
// block belongs to the row and to the strip of columns in which it STARTS.  Positions inside a tile are counted from
// the strip's first column, p = 0 .. width + 127: a block that starts in the strip may reach up to 127 columns beyond
// it, and beyond the end of the row position p continues with the next row's first columns.  The strip's column vectors sit in
// LDS indexed by p, so only the row of an element needs a compare per element.  (1024 x 50257 with bf16 gradients: 779 us per
// step on the general kernels, 170 with the maxima taken per element in the update, 140 with the passes as they are.)
//
// Two ways to cut a matrix (chosen by the host):
//   cols <= 1024:  one strip; a tile is a run of a.rw consecutive blocks, each of the 8 groups of a workgroup takes an
//                  eighth of the run.  Every unit is a whole block, whatever the row length.
//   wider:         strips of a.sw columns (a multiple of 128, at most 1024) x a.rw rows; a group walks along the blocks
//                  of its row that start in the strip.  In the last strip their number varies by one from row to row;
//                  a unit that does not exist gets an offset beyond the tile, where loads return zeros and stores are
//                  dropped.
// The partial last block of a tensor whose size is no multiple of 128 is left to one workgroup with exact arithmetic.
// The first pass needs none of this: nothing in it is reduced over a block, see maxima_ragged_tile.
#pragma once

#include <type_traits>

#include "kernels.hpp"

namespace lpmm {

constexpr int kRagRowSlots = kMaxRowSlots / 2;            // s.blk_vmax: old row maxima, then the new ones

struct RagTile {
    int64_t e0;          // first element of the tile's first block (a multiple of 128)
    int64_t row0;        // row of position 0 of the tile's first row
    int f0;              // first row's position 0, relative to e0
    int n_blocks;        // contiguous tiling: blocks of the tile
    int n_rows;          // rows whose statistics the tile touches (one more than it owns where blocks straddle)
    int own_rows;        // strip tiling: rows of the tile
    int c0, width;       // the strip's first column and its width
    int lim;             // positions at or beyond this belong to the next row
    int per_row;         // strip tiling: units per row
    int end;             // strip tiling: blocks of the tensor behind e0
    uint32_t inv_cols;   // contiguous tiling: x / cols == umulhi(x, inv_cols) for the positions of a tile
    uint32_t bytes4;     // bytes of the tile in an fp32 array (its whole blocks)
};

struct RagUnit {         // one block
    uint32_t off4;       // byte offset of the block in the tile's fp32 array, kNowhere if it does not exist
    int il;              // its row in the tile
    int p;               // position of its first element in that row
    int slot;            // its slot among the staged block scales
};

template <bool ONE_STRIP>
__device__ __forceinline__ RagTile rag_tile(const Tensor4& a, int wg) {
    RagTile t;
    const int64_t nb = a.nb;                                             // whole blocks of the tensor
    if constexpr (ONE_STRIP) {
        const int64_t b0 = int64_t(wg) * a.rw;
        t.n_blocks = nb - b0 < a.rw ? int(nb - b0) : a.rw;
        t.e0 = b0 * 128;
        t.row0 = t.e0 / a.cols;
        t.f0 = int(t.row0 * a.cols - t.e0);                              // <= 0
        t.c0 = 0;
        t.width = t.lim = int(a.cols);
        t.inv_cols = uint32_t((uint64_t(1) << 32) / uint32_t(a.cols)) + 1u;
        t.n_rows = int((uint32_t(t.n_blocks) * 128u - uint32_t(t.f0) - 1u) / uint32_t(a.cols)) + 1;
        t.own_rows = t.per_row = t.end = 0;
        t.bytes4 = uint32_t(t.n_blocks) * 512u;
    } else {
        const int strip = wg % a.strips;
        t.row0 = int64_t(wg / a.strips) * a.rw;
        t.own_rows = a.rows - t.row0 < a.rw ? int(a.rows - t.row0) : a.rw;
        t.n_rows = t.own_rows + 1;
        t.c0 = strip * a.sw;
        t.lim = int(a.cols) - t.c0;
        t.width = t.lim < a.sw ? t.lim : a.sw;
        const int64_t f = t.row0 * a.cols + t.c0;
        t.e0 = (f + 127) / 128 * 128;
        t.f0 = int(f - t.e0);                                            // -127 .. 0
        t.per_row = (t.width + 127) / 128;
        const int64_t left = nb - t.e0 / 128;                            // may be negative: no whole block starts here
        t.end = int(left < (1 << 24) ? (left > 0 ? left : 0) : (1 << 24));
        t.inv_cols = 0;
        t.n_blocks = 0;
        // the blocks that start before the end of the tile's last row of the strip
        const int64_t last = (int64_t(t.own_rows - 1) * a.cols + t.f0 + t.width + 127) >> 7;
        t.bytes4 = uint32_t(last < t.end ? last : t.end) * 512u;
    }
    return t;
}

// unit q of group grp, in the order the group takes them
template <bool ONE_STRIP>
__device__ __forceinline__ RagUnit rag_unit(const RagTile& t, const Tensor4& a, int grp, int q) {
    RagUnit u;
    if constexpr (ONE_STRIP) {
        const int run = a.rw / kGroups;
        const int b = grp * run + q;
        const bool ok = q < run && b < t.n_blocks;
        const uint32_t x = ok ? uint32_t(b) * 128u - uint32_t(t.f0) : 0u;
        u.il = int(__umulhi(x, t.inv_cols));
        u.p = int(x) - u.il * t.width;
        u.off4 = ok ? uint32_t(b) * 512u : kNowhere;
        u.slot = b;
    } else {
        const int k = int((uint32_t(q) * ((65536u + uint32_t(t.per_row) - 1u) / uint32_t(t.per_row))) >> 16);   // q / per_row
        const int j = q - k * t.per_row;
        u.il = k * kGroups + grp;
        const int f = t.f0 + int(row_offset(u.il, a.cols, 0u));          // < 2^29 for rows of the tile
        const int b = ((f + 127) >> 7) + j;
        u.p = b * 128 - f;
        const bool ok = u.il < t.own_rows && u.p < t.width && b < t.end;
        u.off4 = ok ? uint32_t(b) * 512u : kNowhere;
        u.slot = u.il * kFlatBlocks + j;
    }
    return u;
}
// units a group runs through (the same for all groups of the workgroup)
template <bool ONE_STRIP>
__device__ __forceinline__ int rag_units(const RagTile& t, const Tensor4& a) {
    if constexpr (ONE_STRIP) return a.rw / kGroups;
    else return (t.own_rows + kGroups - 1) / kGroups * t.per_row;
}

// the four column-vector entries of a lane: position p of the strip, 4-byte aligned
__device__ __forceinline__ void lds_load4(const float* s, float out[4]) {
    typedef float v4f_l __attribute__((ext_vector_type(4), aligned(4)));
    const v4f_l v = *reinterpret_cast<const v4f_l*>(s);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}
__device__ __forceinline__ int rag_col(const RagTile& t, int64_t cols, int p) { return p < t.lim ? t.c0 + p : p - t.lim; }

template <bool BF16>
__device__ __forceinline__ TileBase rag_base(const Tensor4& a, const RagTile& t) {
    TileBase b;
    const int64_t e = t.e0;
    b.ms = a.ms + e / 128;
    b.rp = tile_rsrc(a.p + e, t.bytes4);
    b.rg = tile_rsrc(reinterpret_cast<const char*>(a.g) + e * (BF16 ? 2 : 4), BF16 ? t.bytes4 / 2 : t.bytes4);
    b.rmq = tile_rsrc(reinterpret_cast<const uint8_t*>(a.mq) + (e >> 1), t.bytes4 / 8);
    b.rvq = tile_rsrc(reinterpret_cast<const uint8_t*>(a.vq) + (e >> 1), t.bytes4 / 8);
    return b;
}

// Statistics tiles (the maxima of the rank-1 form, the sums of the factorized one): strips of 256 columns by rw2 rows, a multiple
// of 8.  A half-wave of 32 lanes takes 256 consecutive columns of one row, a lane 8 elements aligned in the flattening (one
// 16-byte load of a bf16 gradient, 4 bytes of codes): the lanes of row i start at the first multiple of 8 at or behind i * cols,
// `shift` = -i * cols mod 8 columns into the row, and that shift is the same for all rows a half-wave takes (they are 8 apart), so
// that a lane's columns are fixed down the tile.  Columns are counted on through the end of a row: positions cols .. cols + 6 are
// the next row's first ones, whose statistics the row's last lane collects for that row.  Only a tile that has that lane (`edge`)
// looks at which row an element belongs to.
// Bound by the latency of memory: few and wide accesses, and one round trip in front of the loop.  With 4 elements a lane, a wave per
// row and two dependent round trips at the start the maxima of 1024 x 50257 bf16 took 42 us (3.1 TB/s), 31 this way.
constexpr int kSpan = 264;                                        // positions of a strip: 256, and a shift of at most 7
static_assert(offsetof(Lds, cold) == offsetof(Lds, col) + sizeof(float) * kColSlots && kGroups * kSpan <= 2 * kColSlots,
              "col and cold hold the half-waves' column statistics");
static_assert(kMaxRw2 + kGroups + 1 < kMaxRowSlots && kMaxRw2 + kGroups + 1 < 512, "a tile's row statistics are staged in LDS");

template <bool BF16>
struct RagStats {
    static constexpr uint32_t kBytes = BF16 ? 2u : 4u;
    static constexpr int kDepth = BF16 ? 3 : 2;                   // about the same bytes in flight
    int strip, tile, grp, l, n, n_stat, rounds;
    int64_t row0;
    uint32_t cols, at, col0;      // the lane's first position in the strip and column
    int n_lane;                   // rows whose group of the lane's columns is whole: n, or n - 1 at the tensor's end
    bool live, edge;
    Rsrc rg, rv;
    uint32_t off_g, off_v;        // byte offsets of the lane's elements in the half-wave's first row

    __device__ __forceinline__ RagStats(const Tensor4& a, int wg) {
        strip = wg % a.strips2, tile = wg / a.strips2;
        grp = threadIdx.x >> 5, l = threadIdx.x & 31;
        row0 = int64_t(tile) * a.rw2;
        const int64_t left = class_rows(a) - row0;
        n = left < a.rw2 ? int(left) : a.rw2;
        n_stat = row0 + n < a.rows ? n + 1 : n;
        rounds = (n + kGroups - 1) / kGroups;
        cols = uint32_t(a.cols);
        at = uint32_t(l) * 8u + ((0u - uint32_t(grp) * cols) & 7u);
        col0 = uint32_t(strip) * 256u + at;
        live = col0 < cols;
        edge = uint32_t(strip) * 256u + 262u >= cols;
        const int64_t e0 = row0 * a.cols;
        // what the tile's lanes own: up to where the lanes of the row behind its last one begin, so that those read zeros; up to the
        // last whole group of the tensor
        uint32_t elems = (uint32_t(n) * cols + 7u) / 8u * 8u;
        if (e0 + elems > a.P) elems -= 8u;
        n_lane = uint32_t(n - 1) * cols + col0 < elems ? n : n - 1;
        rg = tile_rsrc(reinterpret_cast<const char*>(a.g) + e0 * int(kBytes), elems * kBytes);
        const uint32_t e = uint32_t(grp) * cols + col0;
        off_g = live ? e * kBytes : kNowhere;
        off_v = live ? e >> 1 : kNowhere;
        if (a.vq) rv = tile_rsrc(reinterpret_cast<const uint8_t*>(a.vq) + (e0 >> 1), elems >> 1);
    }
    __device__ __forceinline__ bool next_row(int e) const { return col0 + uint32_t(e) >= cols; }      // of element e, if edge
    __device__ __forceinline__ void load_grad(int k, float4 (&g)[BF16 ? 1 : 2]) const {
        const uint32_t off = off_g + uint32_t(k) * (cols * 8u * kBytes);
        g[0] = buf_ld_f4(rg, off);
        if constexpr (!BF16) g[1] = buf_ld_f4(rg, off + 16u);
    }
    __device__ __forceinline__ uint32_t load_codes(int k) const {
        return __builtin_amdgcn_raw_buffer_load_b32(rv, int(off_v + uint32_t(k) * (cols * 4u)), 0, 0);
    }
    // the positions that a half-wave of some other shift has and one of this has not, in each half-wave's kSpan column statistics
    static __device__ __forceinline__ void clear_ends(float* span) {
        const int t = threadIdx.x;
        if (t < kGroups * 16) span[(t >> 4) * kSpan + ((t & 15) < 8 ? t & 15 : 248 + (t & 15))] = 0.0f;
    }
    // one(set, k) for the half-wave's rows k = 0 .. rounds - 1, of which the first kDepth have been fetched; a register set is
    // reloaded right after its row
    template <class Row, class Fetch, class One>
    __device__ __forceinline__ void run(Row (&r)[kDepth], Fetch fetch, One one) const {
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);          // loop start-up state: nothing outstanding
        int k = 0;
        while (k + kDepth - 1 < rounds) {
#pragma unroll
            for (int u = 0; u < kDepth; ++u) {
                one(r[u], k + u);
                __builtin_amdgcn_sched_barrier(0);
                r[u] = fetch(k + kDepth + u);
                __builtin_amdgcn_sched_barrier(0);
            }
            k += kDepth;
        }
#pragma unroll
        for (int u = 0; u < kDepth - 1; ++u)
            if (k + u < rounds) one(r[u], k + u);
    }
};

template <bool BF16>
__device__ __forceinline__ void maxima_ragged_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    const RagStats<BF16> t(a, wg);
    auto fetch = [&](int k) {
        Row8<BF16> r;
        t.load_grad(k, r.g);
        r.vq = t.load_codes(k);
        return r;
    };
    Row8<BF16> r[t.kDepth];
#pragma unroll
    for (int u = 0; u < t.kDepth; ++u) r[u] = fetch(u);
    // Old statistics, requested with the first rows, so that one round trip to the memory stands in front of the loop: thread p takes
    // position p of the strip (and 256 + p) and row p.  Lanes without columns get zeros: their moments are zero then.
    float* const stage = reinterpret_cast<float*>(s.search);
    float* const rows = stage + kSpan;                            // for the exact route
    static_assert(kBucketsPadded * sizeof(SearchEntry) >= (kSpan + kThreads + 1) * sizeof(float) && kSpan <= 2 * kThreads, "old statistics");
    auto col = [&](uint32_t c) { return c < t.cols ? c : c - t.cols; };
    const int tid = threadIdx.x;
    const uint32_t c_own = uint32_t(t.strip) * 256u + uint32_t(tid);
    const float c_a = c_own < t.cols + 7u ? a.c[col(c_own)] : 0.0f;
    const float c_b = tid < kSpan - kThreads && c_own + 256u < t.cols + 7u ? a.c[col(c_own + 256u)] : 0.0f;
    const Rsrc rr = tile_rsrc(a.r + t.row0, uint32_t(t.n_stat) * 4u);
    const float r_a = buf_ld_f1(rr, uint32_t(tid) * 4u), r_b = tid == 0 ? buf_ld_f1(rr, kThreads * 4u) : 0.0f;
    __builtin_amdgcn_sched_barrier(0);
    float* const next = reinterpret_cast<float*>(s.deq);          // maxima of rows' first elements, from the row in front
    stage[tid] = c_a;
    if (tid < kSpan - kThreads) stage[tid + kThreads] = c_b;
    rows[tid] = r_a;
    s.blk_scale[tid] = r_a * 0.0625f;
    s.blk_vmax[tid] = next[tid] = 0.0f;
    static_assert(kMaxRw2 == kThreads, "rows of a tile and the one behind");
    if (tid == 0) {
        rows[kThreads] = r_b;
        s.blk_scale[kThreads] = r_b * 0.0625f;
        s.blk_vmax[kThreads] = next[kThreads] = 0.0f;
    }
    t.clear_ends(s.col);
    const bool lane_tame = scale_is_tame(c_a) && scale_is_tame(c_b) && scale_is_tame(r_a) && scale_is_tame(r_b);
    const bool tame = all_threads(s, lane_tame);         // else the exact route for the whole tile
    float c16[8], cmax[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        c16[e] = t.live ? stage[t.at + e] * 0.0625f : 0.0f;
        cmax[e] = 0.0f;
    }
    auto one = [&](const Row8<BF16>& x, int k, auto edge) {
        constexpr bool kEdge = decltype(edge)::value;
        const int il = t.grp + k * kGroups;
        const bool in = il < t.n_lane;                            // behind the tile: zeros
        float g[8], vt[8];
        unpack_grad8<BF16>(x.g, g);
        if (__builtin_expect(tame, 1)) {
            float qf[8];
            codes_to_float8(x.vq, qf);
            const float ra = in ? s.blk_scale[il] : 0.0f, rb = kEdge && in ? s.blk_scale[il + 1] : 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) vt[e] = dequant_v16(qf[e], min_nonneg(kEdge && t.next_row(e) ? rb : ra, c16[e]));
        } else {
            const float ra = in ? rows[il] : 0.0f, rb = kEdge && in ? rows[il + 1] : 0.0f;
            uint32_t at = t.at;
            asm volatile("" : "+v"(at));                          // these columns are not worth registers all along
#pragma unroll
            for (int e = 0; e < 8; ++e)
                vt[e] = dequant_v((x.vq >> (4 * e)) & 15u, t.live ? fminf(kEdge && t.next_row(e) ? rb : ra, stage[at + e]) : 0.0f);
        }
        float own = 0.0f, behind = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            vt[e] = moment_v(h, vt[e], g[e]);
            cmax[e] = fmaxf(cmax[e], vt[e]);                      // a NaN raises no maximum
        }
        if constexpr (kEdge) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                own = fmaxf(own, t.next_row(e) ? 0.0f : vt[e]);
                behind = fmaxf(behind, t.next_row(e) ? vt[e] : 0.0f);
            }
            if (t.live && t.next_row(7)) next[il + 1] = behind;   // one lane of the row
        } else {
#pragma unroll
            for (int e = 0; e < 8; e += 2) own = fmaxf(fmaxf(own, vt[e]), vt[e + 1]);
        }
        own = group32_allmax(own);
        if (t.l == 0) s.blk_vmax[il] = own;
    };
    if (t.edge) t.run(r, fetch, [&](const Row8<BF16>& x, int k) { one(x, k, std::true_type{}); });
    else t.run(r, fetch, [&](const Row8<BF16>& x, int k) { one(x, k, std::false_type{}); });
#pragma unroll
    for (int e = 0; e < 8; ++e) s.col[t.grp * kSpan + int(t.at) + e] = cmax[e];
    __syncthreads();
    for (int k = threadIdx.x; k < t.n_stat; k += kThreads) {
        const float m = fmaxf(s.blk_vmax[k], next[k]);
        if (m > 0.0f) atomic_max_nonneg(a.r_new + t.row0 + k, m);
    }
    for (int k = threadIdx.x; k < kSpan; k += kThreads) {
        const uint32_t c = uint32_t(t.strip) * 256u + uint32_t(k);
        float m = 0.0f;
#pragma unroll
        for (int y = 0; y < kGroups; ++y) m = fmaxf(m, s.col[y * kSpan + k]);
        if (m > 0.0f && c < t.cols + 7u) atomic_max_nonneg(a.c_new + (c < t.cols ? c : c - t.cols), m);
    }
}

// The elements that the tiles leave out, all in the last row.  A workgroup requests its elements all at once (one after the other, two
// round trips each, a last row was the end of the pass: 847 x 4973 bf16 9.1 us, 6.7 so).
constexpr int kLastEach = kLastRowElems / kThreads;
template <bool BF16>
struct Tail {
    int64_t first, col0, left;      // first element, its column, elements from there on
    __device__ __forceinline__ Tail(const Tensor4& a, int part) {
        first = tail_begin(a) + int64_t(part) * kLastRowElems;
        col0 = first - (a.rows - 1) * a.cols;
        left = a.P - first;
    }
    __device__ __forceinline__ int at(int u) const { return u * kThreads + int(threadIdx.x); }
    __device__ __forceinline__ bool on(int u) const { return at(u) < left; }
    __device__ __forceinline__ void grads(const Tensor4& a, uint32_t raw[kLastEach]) const {      // zeros behind the end
        const Rsrc r = tile_rsrc(reinterpret_cast<const char*>(a.g) + first * (BF16 ? 2 : 4), uint32_t(left) * (BF16 ? 2u : 4u));
#pragma unroll
        for (int u = 0; u < kLastEach; ++u) {
            if constexpr (BF16) raw[u] = uint16_t(__builtin_amdgcn_raw_buffer_load_b16(r, at(u) * 2, 0, 0));
            else raw[u] = __builtin_amdgcn_raw_buffer_load_b32(r, at(u) * 4, 0, 0);
        }
    }
    static __device__ __forceinline__ float value(uint32_t raw) { return __uint_as_float(BF16 ? raw << 16 : raw); }
};

template <bool BF16>
__device__ __forceinline__ void maxima_tail(const Tensor4& a, const Hyper& h, int part) {
    const Tail<BF16> t(a, part);
    const float r_old = a.r[a.rows - 1];
    float c[kLastEach], rmax = 0.0f;
    uint32_t g[kLastEach], q[kLastEach];
    t.grads(a, g);
    const Rsrc rc = tile_rsrc(a.c + t.col0, uint32_t(t.left) * 4u), rq = tile_rsrc(reinterpret_cast<const uint8_t*>(a.vq) + (t.first >> 1), uint32_t(t.left + 1) / 2u);
#pragma unroll
    for (int u = 0; u < kLastEach; ++u) {
        c[u] = buf_ld_f1(rc, uint32_t(t.at(u)) * 4u);
        q[u] = uint8_t(__builtin_amdgcn_raw_buffer_load_b8(rq, t.at(u) >> 1, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kLastEach; ++u) {
        const float v = dequant_v((q[u] >> (4 * (threadIdx.x & 1))) & 15u, fminf(r_old, c[u]));      // behind the end: 0
        const float vt = fmaxf(moment_v(h, v, t.value(g[u])), 0.0f);
        if (vt > 0.0f) atomic_max_nonneg(a.c_new + t.col0 + t.at(u), vt);
        rmax = fmaxf(rmax, vt);
    }
    for (int d = 1; d < 64; d <<= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, d));
    if ((threadIdx.x & 63) == 0 && rmax > 0.0f) atomic_max_nonneg(a.r_new + a.rows - 1, rmax);
}

template <bool BF16>
__device__ __forceinline__ void maxima_ragged(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    const int tiles = int((class_rows(a) + a.rw2 - 1) / a.rw2) * a.strips2;
    if (wg < tiles) maxima_ragged_tile<BF16>(a, h, wg, s);
    else maxima_tail<BF16>(a, h, wg - tiles);
}

// One block of the second pass.  l = lane of the group.
template <bool BF16, class Mid>
__device__ __forceinline__ void update_ragged_unit(const Tensor4& a, const Hyper& h, const TileBase& tb, const RagTile& t, LdsRank1& s,
                                                   const Row1<BF16>& cur, const RagUnit& u, int l, bool tame, Mid mid) {
    float w[4] = {cur.p.x, cur.p.y, cur.p.z, cur.p.w};
    float g[4];
    unpack_grad4<BF16>(cur.g, g);
    const bool ok = u.off4 != kNowhere;
    // a unit that does not exist works on the tile's first slots; its stores are dropped
    const int il = ok ? u.il : 0, p4 = ok ? u.p + 4 * l : 0;
    const float s_old = ok ? s.blk_scale[u.slot] : 0.0f;
    const float2 ra = row_scalars(s, il), rb = row_scalars(s, il + 1);
    float mt[4], vt[4], amax = 0.0f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float2 d = s.deq[(uint32_t(cur.mq) >> (8 * k)) & 255u];
        mt[2 * k] = d.x * s_old;
        mt[2 * k + 1] = d.y * s_old;
    }
    if (__builtin_expect(tame, 1)) {
        float qf[4], c16[4];
        codes_to_float4(cur.vq, qf);
        lds_load4(&s.cold[p4], c16);
#pragma unroll
        for (int e = 0; e < 4; ++e) vt[e] = dequant_v16(qf[e], min_nonneg(p4 + e < t.lim ? ra.x : rb.x, c16[e]));
    } else {
        const float r_a = a.r[t.row0 + il], r_b = t.row0 + il + 1 < a.rows ? a.r[t.row0 + il + 1] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            vt[e] = dequant_v((uint32_t(cur.vq) >> (4 * e)) & 15u, fminf(p4 + e < t.lim ? r_a : r_b, a.c[rag_col(t, a.cols, p4 + e)]));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        mt[e] = moment_m(h, mt[e], g[e]);
        vt[e] = moment_v(h, vt[e], g[e]);
        w[e] = param_update(h, w[e], mt[e], vt[e]);
        amax = fmaxf(amax, fabsf(mt[e]));
    }
    __builtin_amdgcn_sched_barrier(0);
    mid();
    __builtin_amdgcn_sched_barrier(0);
    const float s_new = group32_allmax(amax);
    uint32_t vq_new = 0;
    bool sure = false;
    if (__builtin_expect(tame, 1)) {
        float inv[4];
        lds_load4(&s.col[p4], inv);
#pragma unroll
        for (int e = 0; e < 4; ++e) inv[e] = max_nonneg(p4 + e < t.lim ? ra.y : rb.y, inv[e]);
        vq_new = compress_v4(vt, inv, sure);
    }
    if (__builtin_expect(!sure, 0)) {
        vq_new = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            vq_new |= quant_v_code(vt[e], fminf(row_new(s, p4 + e < t.lim ? il : il + 1), s.cnew[p4 + e])) << (4 * e);
    }
    const uint32_t off4 = ok ? u.off4 + 16u * l : kNowhere;
    store_row1(tb, off4, w, compress_m4(s.search, mt, s_new));
    store_vq(tb, off4, vq_new);
    if (l == 0 && ok) s.blk_scale[u.slot] = s_new;
}

// Positions of a strip as a thread takes them, kThreads apart; rows and block scales likewise.
constexpr int kRagPos = (kFlatBlocks * 128 + 128 + kThreads - 1) / kThreads;
static_assert(kRowSlots <= kThreads && kRagPos * kThreads >= kFlatBlocks * 128 + 128, "start-up of a ragged update tile");

template <bool BF16, bool ONE_STRIP, bool SAME_LAUNCH, class Sync>
__device__ __forceinline__ void update_ragged_tile(const Tensor4& a, const Hyper& h, int wg, LdsRank1& s, Sync& sync) {
    const TableRegs tables = request_tables();
    const RagTile t = rag_tile<ONE_STRIP>(a, wg);
    const TileBase tb = rag_base<BF16>(a, t);
    const int grp = threadIdx.x >> 5, l = threadIdx.x & 31, tid = threadIdx.x;
    auto unit = [&](int q) { return rag_unit<ONE_STRIP>(t, a, grp, q); };
    auto fetch = [&](const RagUnit& u) { return load_row1<BF16, kPolicyNt>(tb, u.off4 == kNowhere ? kNowhere : u.off4 + 16u * l); };
    const int n = rag_units<ONE_STRIP>(t, a);
    // start-up as in update_tile
    float c_old[kRagPos], c_new[kRagPos];
#pragma unroll
    for (int u = 0; u < kRagPos; ++u) {
        const int k = tid + u * kThreads;
        c_old[u] = k < t.width + 128 ? a.c[rag_col(t, a.cols, k)] : 0.0f;
    }
    const bool row_in = tid < t.n_rows && t.row0 + tid < a.rows;  // a unit looks at its row and the next
    const float r_old = row_in ? a.r[t.row0 + tid] : 0.0f;
    // old block scales into the slots of the new ones
    float ms_old = 0.0f;
    if constexpr (ONE_STRIP) {
        if (tid < t.n_blocks) ms_old = tb.ms[tid];
    } else if (tid < t.own_rows * kFlatBlocks) {
        const int b = ((t.f0 + int(row_offset(tid / kFlatBlocks, a.cols, 0u)) + 127) >> 7) + tid % kFlatBlocks;
        if (tid % kFlatBlocks < t.per_row && b < t.end) ms_old = tb.ms[b];
    }
    float r_new;
    auto request_new = [&] {
#pragma unroll
        for (int u = 0; u < kRagPos; ++u) {
            const int k = tid + u * kThreads;
            c_new[u] = k < t.width + 128 ? ld_ws<SAME_LAUNCH>(a.c_new + rag_col(t, a.cols, k)) : 0.0f;
        }
        r_new = row_in ? ld_ws<SAME_LAUNCH>(a.r_new + t.row0 + tid) : 0.0f;
    };
    if constexpr (!SAME_LAUNCH) request_new();
    RagUnit u0 = unit(0), u1 = unit(1), u2;
    Row1<BF16> r0 = fetch(u0), r1 = fetch(u1), r2;
    put_tables(s, tables);
    bool lane_tame = true;
    auto tame_too = [&](float x) { lane_tame = bool(int(lane_tame) & int(scale_is_tame(x))); return x; };
#pragma unroll
    for (int u = 0; u < kRagPos; ++u) {
        const int k = tid + u * kThreads;
        if (k < t.width + 128) s.cold[k] = tame_too(c_old[u]) * 0.0625f;
    }
    if (tid <= t.n_rows) stage_row_old(s, tid, tame_too(r_old));
    s.blk_scale[tid] = ms_old;
    if (!sync.ready()) return;
    if constexpr (SAME_LAUNCH) request_new();
#pragma unroll
    for (int u = 0; u < kRagPos; ++u) {
        const int k = tid + u * kThreads;
        if (k < t.width + 128) {
            s.cnew[k] = tame_too(c_new[u]);
            s.col[k] = approx_inv16(c_new[u]);
        }
    }
    if (tid <= t.n_rows) stage_row_new(s, tid, tame_too(r_new));
    const bool tame = all_threads(s, lane_tame);
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);              // loop start-up state: nothing outstanding (see update_tile)
    if (tame) sync.staged();
    auto none = [] {};
    auto work = [&](const Row1<BF16>& cur, const RagUnit& u, auto mid) { update_ragged_unit<BF16>(a, h, tb, t, s, cur, u, l, tame, mid); };
    int q = 0;
    while (q + 2 < n) {                                   // rounds of three units, no exit in the middle
        work(r0, u0, [&] { u2 = unit(q + 2); r2 = fetch(u2); });
        work(r1, u1, [&] { u0 = unit(q + 3); r0 = fetch(u0); });
        work(r2, u2, [&] { u1 = unit(q + 4); r1 = fetch(u1); });
        q += 3;
    }
    if (q < n) {
        work(r0, u0, none);
        if (q + 1 < n) work(r1, u1, none);
    }
    __syncthreads();
    if (!tame) sync.staged();
    if constexpr (ONE_STRIP) {
        for (int k = threadIdx.x; k < t.n_blocks; k += kThreads) tb.ms[k] = s.blk_scale[k];
    } else {
        for (int k = threadIdx.x; k < t.own_rows * kFlatBlocks; k += kThreads) {
            const int f = t.f0 + int(row_offset(k / kFlatBlocks, a.cols, 0u));
            const int b = ((f + 127) >> 7) + k % kFlatBlocks;
            if (b * 128 - f < t.width && b < t.end) tb.ms[b] = s.blk_scale[k];
        }
    }
}

// The partial last block of a tensor whose size is no multiple of 128: a thread per byte of codes, exact arithmetic.
template <bool BF16, bool SAME_LAUNCH>
__device__ __forceinline__ void update_last_block(const Tensor4& a, const Hyper& h, LdsRank1& s) {
    const int64_t e0 = int64_t(a.nb) * 128;
    const int t = threadIdx.x;
    const float s_old = a.ms[a.nb];
    const bool on = e0 + 2 * t < a.P;                     // fewer than 64 threads
    uint32_t bm = 0, bv = 0;
    float mt[2] = {0.0f, 0.0f}, vt[2] = {0.0f, 0.0f};
    if (on) {
        bm = reinterpret_cast<const uint8_t*>(a.mq)[(e0 >> 1) + t];
        bv = reinterpret_cast<const uint8_t*>(a.vq)[(e0 >> 1) + t];
    }
    auto each = [&](auto f) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t e = e0 + 2 * t + k;
            if (e < a.P) f(k, e, e / a.cols, e % a.cols);
        }
    };
    each([&](int k, int64_t e, int64_t i, int64_t j) {
        const float2 dq = s.deq[bm];
        const float g = load_grad1<BF16>(a.g, e);
        mt[k] = moment_m(h, (k ? dq.y : dq.x) * s_old, g);
        vt[k] = moment_v(h, dequant_v((bv >> (4 * k)) & 15u, fminf(a.r[i], a.c[j])), g);
        a.p[e] = param_update(h, a.p[e], mt[k], vt[k]);
    });
    s.col[t] = fmaxf(fabsf(mt[0]), fabsf(mt[1]));
    __syncthreads();
    float s_new = 0.0f;
    for (int i = 0; i < 64; ++i) s_new = fmaxf(s_new, s.col[i]);
    uint32_t qm = 0, qv = 0;
    each([&](int k, int64_t, int64_t i, int64_t j) {
        qm |= quant_m_code(s.search, mt[k], s_new) << (4 * k);
        qv |= quant_v_code(vt[k], fminf(ld_ws<SAME_LAUNCH>(a.r_new + i), ld_ws<SAME_LAUNCH>(a.c_new + j))) << (4 * k);
    });
    if (on) {
        reinterpret_cast<uint8_t*>(a.mq)[(e0 >> 1) + t] = uint8_t(qm);
        reinterpret_cast<uint8_t*>(a.vq)[(e0 >> 1) + t] = uint8_t(qv);
    }
    if (t == 0) a.ms[a.nb] = s_new;
}

// Workgroups [0, n_wg2) of the second pass; the last one takes the partial block, if any.
template <bool BF16, bool SAME_LAUNCH, class Sync>
__device__ __forceinline__ void update_ragged(const Tensor4& a, const Hyper& h, int wg, LdsRank1& s, Sync& sync) {
    if ((a.P & 127) && wg == a.n_wg2 - 1) {
        load_tables(s);
        if (!sync.ready()) return;
        update_last_block<BF16, SAME_LAUNCH>(a, h, s);
        __syncthreads();
        sync.staged();
    } else if (a.strips == 1) {
        update_ragged_tile<BF16, true, SAME_LAUNCH>(a, h, wg, s, sync);
    } else {
        update_ragged_tile<BF16, false, SAME_LAUNCH>(a, h, wg, s, sync);
    }
}

// ---- the factorized step on the same tiles ------------------------------------------------------------------------
//
// Memory-bound like the rank-1 form.  (Before, on the general tiles: a float atomic in LDS per element for the column sums,
// an exact division and four loads of statistics per element for the update.  General / these, us per step: 4096 x 4000
// bf16 907 / 49, 1024 x 50257 bf16 1747 / 147, 30000 x 1000 fp32 361 / 107, 600 x 147 fp32 15.7 / 13.9.)

// Statistics pass: the tiles of maxima_ragged_tile, sums of squares in place of maxima.
template <bool BF16>
__device__ __forceinline__ void factor_stats_ragged_tile(const Tensor4& a, int wg, Lds& s) {
    const RagStats<BF16> t(a, wg);
    struct Row { float4 g[BF16 ? 1 : 2]; };
    auto fetch = [&](int k) {
        Row r;
        t.load_grad(k, r.g);
        return r;
    };
    Row r[t.kDepth];
#pragma unroll
    for (int u = 0; u < t.kDepth; ++u) r[u] = fetch(u);
    float* const next = reinterpret_cast<float*>(s.deq);          // sums of rows' first elements, from the row in front
    for (int k = threadIdx.x; k <= t.n; k += kThreads) { s.blk_scale[k] = 0.0f; next[k] = 0.0f; }
    t.clear_ends(s.col);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float old = 0.0f;                                             // of the tile's rows, once per row
    if (wave == 1 && t.strip == 0)
        for (int k = lane; k < t.n; k += 64) old += a.r[t.row0 + k];
    __syncthreads();
    float cacc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    auto one = [&](const Row& x, int k, auto edge) {
        constexpr bool kEdge = decltype(edge)::value;
        const int il = t.grp + k * kGroups;
        float g[8], sq[8], own[8];
        unpack_grad8<BF16>(x.g, g);                               // zeros in lanes without columns and behind the tile
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            sq[e] = g[e] * g[e];
            cacc[e] += sq[e];
            own[e] = kEdge && t.next_row(e) ? 0.0f : sq[e];
        }
        auto sum8 = [](const float (&v)[8]) { return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])); };
        if constexpr (kEdge) {
            if (t.live && t.next_row(7)) {                        // one lane of the row
#pragma unroll
                for (int e = 0; e < 8; ++e) sq[e] = t.next_row(e) ? sq[e] : 0.0f;
                next[il + 1] = sum8(sq);
            }
        }
        const float sum = group32_sum(sum8(own));
        if (t.l == 0) s.blk_scale[il] = sum;
    };
    if (t.edge) t.run(r, fetch, [&](const Row& x, int k) { one(x, k, std::true_type{}); });
    else t.run(r, fetch, [&](const Row& x, int k) { one(x, k, std::false_type{}); });
#pragma unroll
    for (int e = 0; e < 8; ++e) s.col[t.grp * kSpan + int(t.at) + e] = cacc[e];
    __syncthreads();
    for (int k = threadIdx.x; k < t.n_stat; k += kThreads) atomic_add_f32(a.r_new + t.row0 + k, s.blk_scale[k] + next[k]);
    for (int k = threadIdx.x; k < kSpan; k += kThreads) {
        const uint32_t c = uint32_t(t.strip) * 256u + uint32_t(k);
        auto at = [&](int y) { return s.col[y * kSpan + k]; };
        const float sum = ((at(0) + at(1)) + (at(2) + at(3))) + ((at(4) + at(5)) + (at(6) + at(7)));
        if (sum != 0.0f && c < t.cols + 7u) atomic_add_f32(a.c_new + (c < t.cols ? c : c - t.cols), sum);
    }
    float* tot = reinterpret_cast<float*>(a.counter);
    if (wave == 0) {
        float part = 0.0f;
        for (int k = lane; k < t.n_stat; k += 64) part += s.blk_scale[k] + next[k];
        part = wave_sum(part);
        if (lane == 0) atomic_add_f32(tot + tot_new_word(wg & (a.tot_slots - 1)), part);
    } else if (wave == 1 && t.strip == 0) {
        old = wave_sum(old);
        if (lane == 0) atomic_add_f32(tot + tot_old_word(t.tile & (a.tot_slots - 1)), old);
    }
}

// The elements that the tiles leave out.
template <bool BF16>
__device__ __forceinline__ void factor_stats_tail(const Tensor4& a, int part, Lds& s) {
    const Tail<BF16> t(a, part);
    const int lane = threadIdx.x & 63;
    uint32_t g[kLastEach];
    float sum = 0.0f;
    t.grads(a, g);
#pragma unroll
    for (int u = 0; u < kLastEach; ++u) {
        const float sq = t.value(g[u]) * t.value(g[u]);
        if (t.on(u)) atomic_add_f32(a.c_new + t.col0 + t.at(u), sq);
        sum += sq;
    }
    sum = wave_sum(sum);
    if (lane == 0) s.col[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float* tot = reinterpret_cast<float*>(a.counter);
        const float all = (s.col[0] + s.col[1]) + (s.col[2] + s.col[3]);
        atomic_add_f32(a.r_new + a.rows - 1, all);
        atomic_add_f32(tot + tot_new_word(part & (a.tot_slots - 1)), all);
        if (part == 0 && class_rows(a) == 0) atomic_add_f32(tot + tot_old_word(0), a.r[a.rows - 1]);
    }
}

template <bool BF16>
__device__ __forceinline__ void factor_stats_ragged(const Tensor4& a, int wg, Lds& s) {
    const int tiles = int((class_rows(a) + a.rw2 - 1) / a.rw2) * a.strips2;
    if (wg < tiles) factor_stats_ragged_tile<BF16>(a, wg, s);
    else factor_stats_tail<BF16>(a, wg - tiles, s);
}

// Update pass: the blocks of update_ragged_tile; s.cold holds the columns' new statistics by position, s.blk_vmax the rows'
// over their total.
template <bool BF16, bool ONE_STRIP>
__device__ __forceinline__ void factor_update_ragged_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    // start-up as in update_ragged_tile: everything is requested before any of it is waited for
    const TableRegs tables = request_tables();
    const RagTile t = rag_tile<ONE_STRIP>(a, wg);
    const TileBase tb = rag_base<BF16>(a, t);
    const int grp = threadIdx.x >> 5, l = threadIdx.x & 31, tid = threadIdx.x;
    auto unit = [&](int q) { return rag_unit<ONE_STRIP>(t, a, grp, q); };
    auto fetch = [&](const RagUnit& u) { return load_rowf<BF16>(tb, u.off4 == kNowhere ? kNowhere : u.off4 + 16u * l); };
    const int n = rag_units<ONE_STRIP>(t, a);
    float c_old[kRagPos], c_sum[kRagPos];
#pragma unroll
    for (int u = 0; u < kRagPos; ++u) {
        const int k = tid + u * kThreads;
        const bool in = k < t.width + 128;
        const int c = in ? rag_col(t, a.cols, k) : 0;
        c_old[u] = in ? a.c[c] : 0.0f;
        c_sum[u] = in ? a.c_new[c] : 0.0f;
    }
    const bool row_in = tid < t.n_rows && t.row0 + tid < a.rows;
    const float r_old = row_in ? a.r[t.row0 + tid] : 0.0f, r_sum = row_in ? a.r_new[t.row0 + tid] : 0.0f;
    float ms_old = 0.0f;
    if constexpr (ONE_STRIP) {
        if (tid < t.n_blocks) ms_old = tb.ms[tid];
    } else if (tid < t.own_rows * kFlatBlocks) {
        const int b = ((t.f0 + int(row_offset(tid / kFlatBlocks, a.cols, 0u)) + 127) >> 7) + tid % kFlatBlocks;
        if (tid % kFlatBlocks < t.per_row && b < t.end) ms_old = tb.ms[b];
    }
    RagUnit u0 = unit(0), u1 = unit(1), u2;
    RowF<BF16> r0 = fetch(u0), r1 = fetch(u1), r2;
    const float inv_total = factor_inv_total(a, h);
    __builtin_amdgcn_sched_barrier(0);
    put_tables(s, tables);
#pragma unroll
    for (int u = 0; u < kRagPos; ++u) {
        const int k = tid + u * kThreads;
        if (k < t.width + 128) s.cold[k] = stat_ema(h, c_old[u], c_sum[u]);
    }
    static_assert(kRagRowSlots == kThreads, "a thread per row");
    s.blk_vmax[tid] = stat_ema(h, r_old, r_sum) * inv_total;
    s.blk_scale[tid] = ms_old;
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);              // loop start-up state: nothing outstanding (see update_tile)
    auto none = [] {};
    auto work = [&](const RowF<BF16>& cur, const RagUnit& u, auto mid) {
        float w[4] = {cur.p.x, cur.p.y, cur.p.z, cur.p.w};
        float g[4], ct[4], mt[4], amax = 0.0f;
        unpack_grad4<BF16>(cur.g, g);
        const bool ok = u.off4 != kNowhere;            // a unit that does not exist: all moments zero
        const float s_old = ok ? s.blk_scale[u.slot] : 0.0f;
        const float r_a = ok ? s.blk_vmax[u.il] : 0.0f, r_b = ok ? s.blk_vmax[u.il + 1] : 0.0f;
        const int p4 = ok ? u.p + 4 * l : 0;
        lds_load4(&s.cold[p4], ct);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float2 d = s.deq[(uint32_t(cur.mq) >> (8 * k)) & 255u];
            mt[2 * k] = d.x * s_old;
            mt[2 * k + 1] = d.y * s_old;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mt[e] = moment_m(h, mt[e], g[e]);
            w[e] = param_update(h, w[e], mt[e], (p4 + e < t.lim ? r_a : r_b) * ct[e]);
            amax = fmaxf(amax, fabsf(mt[e]));
        }
        __builtin_amdgcn_sched_barrier(0);
        mid();
        __builtin_amdgcn_sched_barrier(0);
        const float s_new = group32_allmax(amax);
        store_row1(tb, ok ? u.off4 + 16u * l : kNowhere, w, compress_m4(s.search, mt, s_new));
        if (l == 0 && ok) s.blk_scale[u.slot] = s_new;
    };
    int q = 0;
    while (q + 2 < n) {                                   // rounds of three units, no exit in the middle
        work(r0, u0, [&] { u2 = unit(q + 2); r2 = fetch(u2); });
        work(r1, u1, [&] { u0 = unit(q + 3); r0 = fetch(u0); });
        work(r2, u2, [&] { u1 = unit(q + 4); r1 = fetch(u1); });
        q += 3;
    }
    if (q < n) {
        work(r0, u0, none);
        if (q + 1 < n) work(r1, u1, none);
    }
    __syncthreads();
    if constexpr (ONE_STRIP) {
        for (int k = threadIdx.x; k < t.n_blocks; k += kThreads) tb.ms[k] = s.blk_scale[k];
    } else {
        for (int k = threadIdx.x; k < t.own_rows * kFlatBlocks; k += kThreads) {
            const int f = t.f0 + int(row_offset(k / kFlatBlocks, a.cols, 0u));
            const int b = ((f + 127) >> 7) + k % kFlatBlocks;
            if (b * 128 - f < t.width && b < t.end) tb.ms[b] = s.blk_scale[k];
        }
    }
}

// Workgroups [0, n_wg2) of the update pass; the last one takes the partial block, if any.
template <bool BF16>
__device__ __forceinline__ void factor_update_ragged(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    if ((a.P & 127) && wg == a.n_wg2 - 1) {
        load_tables(s);
        factor_update_general_tile<BF16>(a, h, a.nb / 16, s, a.nb);
    } else if (a.strips == 1) {
        factor_update_ragged_tile<BF16, true>(a, h, wg, s);
    } else {
        factor_update_ragged_tile<BF16, false>(a, h, wg, s);
    }
}

}  // namespace lpmm

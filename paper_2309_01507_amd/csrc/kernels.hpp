// Kernels of the 4-bit AdamW step (gfx950, wave64, 256-thread workgroups).
//
// Work unit: a group of lanes owns one 128-element block of the row-major flattening.  On the fast
// path (cols % 128 == 0) that is 32 lanes with 4 consecutive elements each; on the general path 16
// lanes (one DPP row) with 8 consecutive elements each.
//
// One step is two passes, because every v code needs the complete row and column maxima of the
// updated second moment (rank-1 normalization, paper Sec. 4.2):
//   first pass:  decompress v -> v_t (Eq. 1) -> row/column maxima of v_t into the workspace (LDS combine, then integer
//                atomic max on the float bits).  It reads the gradient and the codes, 2.5 or 4.5 bytes per parameter.
//   second pass: decompress m, v -> Adam moments -> parameter update -> block absmax of m_t, compress m_t (B128 + signed
//                dynamic-exponent map), compress v_t against min(r'_i, c'_j) (Linear map); the last workgroup publishes
//                r', c' as the new state and clears the workspace.
// (The other way about -- the update first, then the codes of v -- moves the same bytes, but leaves the gradient of a
// tensor behind 11.6 bytes per parameter of other traffic instead of 2.5, out of reach of the memory-side cache; it
// stays for rows shorter than 128 elements, the general path.)
// For 1-dimensional or flattened tensors the second moment is block-wise like the first (Sec. 4.2,
// last paragraph); then nothing crosses a block and the step is ONE pass (b128_*).  The same one-pass
// code without a second moment is SGD with momentum (App. E Alg. 2).  With a factorized second
// moment (Sec. 4.3, factor_*) the two passes are: row / column sums of g^2, then the update.  Tensors
// with more than two dimensions (App. F Alg. 4, nd_*) run the two matrix passes on derived column scales.
// The bodies are "tile" functions, here and (rows that are no multiple of 128 elements) in ragged.hpp.  Thin __global__
// wrappers run them for one tensor (two launches per step, one for the block-wise form); for many tensors they run from a
// work list in one launch with the first pass of a tensor ahead of its second one (flow.hpp), or by phases (launch.hpp).
#pragma once

#include <cstddef>

#include "device_math.hpp"

namespace lpmm {

// Lookup tables, uploaded once per device at init.
__device__ __align__(16) float d_byte_decode[512];          // entry b: {T_DE[b & 15], T_DE[b >> 4]}
__device__ __align__(16) SearchEntry d_search[kBucketsPadded];    // nearest-entry search for the DE map

enum TensorKind : int { kQuantFast = 0, kQuantGeneral = 1, kFp32State = 2, kQuantBlockV = 3, kFactorFast = 4, kFactorGeneral = 5,
                        kSgdmBlock = 6, kSgdmFp32 = 7, kQuantRagged = 8, kFactorRagged = 9 };

struct Tensor4 {
    float* p;               // parameters, fp32 [P]
    const void* g;          // gradient, fp32 or bf16 [P]
    uint32_t* mq;           // first-moment codes, 8 per word   (kFp32State: float* m)
    float* ms;              // first-moment block scales
    uint32_t* vq;           // second-moment codes              (kFp32State: float* v)
    float* r;               // row maxima (state)               (kQuantBlockV: block scales of v; kFactor*: row statistics)
    float* c;               // column maxima (state)            (kFactor*: column statistics)
    float* r_new;           // workspace: row maxima of v_t (zero between steps)      (kFactor*: row sums of g^2)
    float* c_new;           // workspace: column maxima of v_t (zero between steps)   (kFactor*: column sums of g^2)
    unsigned int* counter;  // workspace: ticket counters of the second pass (zero between steps); kFactor*: also two float sums
    int64_t rows, cols, P;
    // second pass (update) of the fast path (cols % 128 == 0)
    int nb;                 // column blocks per row = cols / 128    (kQuantBlockV: whole blocks of the tensor)
    int gx, gy;             // kQuantFast: column blocks of a strip; kFactorFast: a workgroup's 8 groups are gx blocks x gy rows
    int rw;                 // rows per workgroup tile; rw * cols < 2^29   (kQuantBlockV, kSgdmBlock: blocks a group takes in
                            // a row; general path: chunks of 2048 elements a workgroup of the first pass takes;
                            // *Ragged: blocks of a tile if strips == 1, else rows of a tile)
    int strips;             // strips of gx blocks
    int n_wg;               // workgroups of the first pass (kQuantBlockV, kSgdmBlock: of the step)
    int kind;
    // first pass (maxima or sums): strips of 256 columns, rw2 rows per workgroup
    int strips2;            // ceil(nb / 2)
    int rw2;                // rw2 * cols < 2^29
    int n_wg2;              // workgroups of the second pass        (kQuantBlockV: workgroups on whole blocks)
    // log2 of the row spacing of the second / first pass: the groups (waves) that run side by side are 2^rs (2^rs2)
    // rows apart
    int rs, rs2;
    int tot_slots;          // kFactor*: slots that each of the two float sums is spread over (1, 2, 4 or 8)
    int no_decay;           // plans: this tensor takes no weight decay
    int c_extra;            // floats behind c_new (and room behind c) that the publishing workgroup moves and clears
                            // along with the column maxima (tensors with more than two dimensions)
    int nd_index;           // plans: index into the plan's table of inner dimensions, -1 for matrices
    int det;                // kFactorFast in a plan: the sums of g^2 are reduced in a fixed order (no float atomics);
                            // vq then points at the partial sums: float[strips2][round_up(rows, 64)] per strip and row,
                            // then float[tiles][round_up(cols, 64)] per row tile and column
    int sw;                 // kQuantRagged: columns of a strip
    int deferred;           // plans stepped in one launch: the tensor's first entry in the list of deferred tiles
    int skew, skew2;        // logical_wg's skew for the workgroups of the first and of the second pass
};

// The tensor table of a plan lives in device memory.  A pointer read from memory is a generic
// pointer to the compiler, and accesses through it would become flat instructions: slower, and
// counted together with LDS traffic, so that every wait for a table lookup would also wait for the
// rows being prefetched.  On the device the table is therefore read through a twin of Tensor4 whose
// pointer members are typed as global memory (same layout), and converted member by member.
#if defined(__HIP_DEVICE_COMPILE__)
#define LPMM_AS_GLOBAL __attribute__((address_space(1)))
struct Tensor4Table {
    float LPMM_AS_GLOBAL* p;
    const void LPMM_AS_GLOBAL* g;
    uint32_t LPMM_AS_GLOBAL* mq;
    float LPMM_AS_GLOBAL* ms;
    uint32_t LPMM_AS_GLOBAL* vq;
    float LPMM_AS_GLOBAL* r;
    float LPMM_AS_GLOBAL* c;
    float LPMM_AS_GLOBAL* r_new;
    float LPMM_AS_GLOBAL* c_new;
    unsigned int LPMM_AS_GLOBAL* counter;
    int64_t rows, cols, P;
    int nb, gx, gy, rw, strips, n_wg, kind, strips2, rw2, n_wg2, rs, rs2, tot_slots, no_decay, c_extra, nd_index, det, sw, deferred, skew, skew2;
};
static_assert(sizeof(Tensor4Table) == sizeof(Tensor4), "the table twin must mirror Tensor4");
template <class T>
__device__ __forceinline__ Tensor4 from_table(const T& t) {
    Tensor4 a;
    a.p = (float*)t.p;
    a.g = (const void*)t.g;
    a.mq = (uint32_t*)t.mq;
    a.ms = (float*)t.ms;
    a.vq = (uint32_t*)t.vq;
    a.r = (float*)t.r;
    a.c = (float*)t.c;
    a.r_new = (float*)t.r_new;
    a.c_new = (float*)t.c_new;
    a.counter = (unsigned int*)t.counter;
    a.rows = t.rows; a.cols = t.cols; a.P = t.P;
    a.nb = t.nb; a.gx = t.gx; a.gy = t.gy; a.rw = t.rw; a.strips = t.strips; a.n_wg = t.n_wg; a.kind = t.kind;
    a.strips2 = t.strips2; a.rw2 = t.rw2; a.n_wg2 = t.n_wg2; a.rs = t.rs; a.rs2 = t.rs2;
    a.tot_slots = t.tot_slots; a.no_decay = t.no_decay; a.c_extra = t.c_extra; a.nd_index = t.nd_index; a.det = t.det; a.sw = t.sw; a.deferred = t.deferred; a.skew = t.skew; a.skew2 = t.skew2;
    return a;
}
#else
typedef Tensor4 Tensor4Table;
__host__ __device__ inline Tensor4 from_table(const Tensor4& t) { return t; }   // host pass: only parsed, never run
#endif

// A pointer to memory that nothing writes while the kernel runs, typed so that the compiler reads it through the scalar cache
// wherever the address is uniform -- also behind stores, where it would take a vector load and vector registers otherwise.
#if defined(__HIP_DEVICE_COMPILE__)
template <class T> using Constant = const T __attribute__((address_space(4)))*;
template <class T> __device__ __forceinline__ Constant<T> as_constant(const T* p) { return (Constant<T>)(p); }
#else
template <class T> using Constant = const T*;
template <class T> __device__ __forceinline__ Constant<T> as_constant(const T* p) { return p; }
#endif

constexpr int kThreads = 256;
constexpr int kXcds = 8;
constexpr int kElemsPerWg32 = kThreads * 16;   // fp32-state path: elements per workgroup

// Workgroups are dealt to the 8 XCDs round-robin by their id.  Remap so that consecutive logical
// ids -- which touch neighbouring memory -- run on the same XCD and share its L2: XCD x works through the x-th eighth.
// It does not begin at its eighth's start but x * skew workgroups behind it, and comes to the start last: the XCDs keep pace
// with each other, and eight streams at equal distances that are a multiple of a large power of two get in each other's way
// in the memory system.  skew: the workgroups of 2^19 elements (2 MiB of parameters).  Block-wise step of 2^25, 2^26 and 2^27
// elements 5.72, 6.05 and 6.58 TB/s with skew 0, 6.15, 6.62, 6.80 with half of it, 6.43, 6.80, 6.92 with it, 6.45, 6.80, 6.94
// with the double; sizes whose eighths lie at other distances are the same with and without (45 M elements 6.45 / 6.49) or, where
// the skew itself brings them to such a distance, slower with it (the host's launch_skew).
constexpr int64_t kSkewElems = int64_t(1) << 19;
// skew < per_xcd (the host sees to it), so i + x * skew < 8 per_xcd and three conditional subtractions are the remainder: a
// division here, in front of everything else a workgroup does, cost every kernel 0.3 us (statistics pass of 512 x 512 5.80 us
// without a skew, 6.08 with the division, 5.64 as it is; step of 1024 x 1024 12.6 and 11.7).
__device__ __forceinline__ int logical_wg(int skew) {
    const unsigned x = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds;     // the grid is padded to a multiple of 8
    unsigned i = blockIdx.x / kXcds + x * unsigned(skew);
#pragma unroll
    for (unsigned f = kXcds / 2; f >= 1; f /= 2) i -= i >= f * per_xcd ? f * per_xcd : 0u;
    return int(x * per_xcd + i);
}
// Launches of workgroups of very unequal cost (kDealt in place of a skew) are dealt to the XCDs in runs of kDealRun instead; the
// grid is a multiple of 8 of them.
constexpr int kDealRun = 32, kDealt = -1;
__device__ __forceinline__ int logical_wg_or_dealt(int skew) {
    if (skew != kDealt) return logical_wg(skew);
    const int x = blockIdx.x % kXcds, i = blockIdx.x / kXcds;
    return (i / kDealRun * kXcds + x) * kDealRun + i % kDealRun;
}

constexpr int kWaitVmcnt0 = 0x0F70;   // s_waitcnt vmcnt(0) only: expcnt and lgkmcnt fields at their maxima
constexpr int kMaxRowSlots = 512;    // rows of a tile, or x column blocks of its strip (rw * gx) for the row walk

constexpr int kColSlots = 9 * 128;   // columns of a strip; a ragged strip's last block may reach 127 columns beyond it

struct alignas(16) Lds {
    float2 deq[256];
    SearchEntry search[kBucketsPadded];
    float col[kColSlots];
    float cold[kColSlots];      // update tiles: the strip's old column maxima / 16
    // per row and column block of the tile: new block scale of m and the block's maximum of v_t.
    // They leave for global memory at the end of the tile, so that the row loop issues the same
    // memory instructions on every path (loads, the parameter store, the code store) and nothing
    // that depends on the lane.
    float blk_scale[kMaxRowSlots];
    float blk_vmax[kMaxRowSlots];
    uint32_t not_all[kThreads / 64];     // all_threads
};
struct LdsRank1 : Lds {         // second pass of the rank-1 step
    float cnew[kColSlots];      // the strip's new column maxima (s.col: 16 / them, approximately)
};

// The lookup tables on their way to LDS: requested first and put down once the rest of a tile's start-up has been requested,
// too, so that a workgroup waits for one round trip and not for one per loop iteration.
struct TableRegs { uint4 deq, search, rest; };
constexpr int kDeqQuads = 512 / 4, kSearchQuads = kBucketsPadded / 2;
static_assert(kDeqQuads <= kThreads && kSearchQuads <= 2 * kThreads && kBucketsPadded % 2 == 0, "one thread, one 16-byte piece");
__device__ __forceinline__ TableRegs request_tables() {
    TableRegs r{};
    const int t = threadIdx.x;
    if (t < kDeqQuads) r.deq = reinterpret_cast<const uint4*>(d_byte_decode)[t];
    r.search = reinterpret_cast<const uint4*>(d_search)[t];
    if (t < kSearchQuads - kThreads) r.rest = reinterpret_cast<const uint4*>(d_search)[kThreads + t];
    return r;
}
__device__ __forceinline__ void put_tables(Lds& s, const TableRegs& r) {       // the caller's barrier publishes them
    const int t = threadIdx.x;
    if (t < kDeqQuads) reinterpret_cast<uint4*>(s.deq)[t] = r.deq;
    reinterpret_cast<uint4*>(s.search)[t] = r.search;
    if (t < kSearchQuads - kThreads) reinterpret_cast<uint4*>(s.search)[kThreads + t] = r.rest;
}
__device__ __forceinline__ void load_tables(Lds& s) {
    put_tables(s, request_tables());
    __syncthreads();
}

// Whether `ok` holds in every thread, the same answer in all of them, and a barrier: what was put into LDS before is there.  (The
// runtime's __syncthreads_or has three barriers and waits for a load of the workgroup's size: fp32 steps of 512 x 512 and 1024 x 1024
// 9.5 and 11.4 us, 9.1 and 11.0 so.)
// Between two calls there is another barrier.
__device__ __forceinline__ bool all_threads(Lds& s, bool ok) {
    static_assert(kThreads == 256, "one word per wave, four of them");
    const bool bad = __ballot(!ok) != 0;
    if ((threadIdx.x & 63) == 0) s.not_all[threadIdx.x >> 6] = bad;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(int((s.not_all[0] | s.not_all[1]) | (s.not_all[2] | s.not_all[3]))) == 0;
}

// ---- small helpers -----------------------------------------------------------------------------------

// min / max of two floats that are both >= +0, through the integer units (no NaN canonicalization)
__device__ __forceinline__ float min_nonneg(float a, float b) {
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float(x < y ? x : y);
}
__device__ __forceinline__ float max_nonneg(float a, float b) {
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float(x > y ? x : y);
}

// Streaming 128-bit access for the parameters: they are read and written exactly once per step.
// The loads carry the non-temporal hint; the stores go out with the nt and sc1 cache-policy bits (write
// through, do not keep the line).  Measured on the 7B-shaped set: about 9 % less time per step than plain
// accesses for nt on both, and a further 2-3 % of the update (then without v's codes) for sc1 on the
// store.
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));
constexpr int kPolicyNtSc1 = 2 | 16;            // gfx94x/gfx950 cache-policy bits: 1 = sc0, 2 = nt, 16 = sc1
constexpr int kRawBufferWord3 = 0x00020000;     // untyped 32-bit data format, no swizzle, offsets in bytes

// Bounds-checked loads of the fast path.  A tile's arrays are described by raw buffer resources
// whose length is the tile's; a load beyond it returns zero and touches no memory.  The row
// prefetch can therefore run unconditionally past the end of a tile: no branch around the loads, so
// the compiler counts outstanding loads exactly and never waits for a row it has just requested.
typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int kPolicyNt = 2;
constexpr uint32_t kNowhere = 0x7FFFFF00u;      // a byte offset beyond every tile (also after >> 1 and >> 3); the geometries see to it
__device__ __forceinline__ Rsrc tile_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), kRawBufferWord3);
}
__device__ __forceinline__ float4 buf_ld_f4_stream(Rsrc r, uint32_t off) {
    const v4f_t v = __builtin_bit_cast(v4f_t, __builtin_amdgcn_raw_buffer_load_b128(r, int(off), 0, kPolicyNt));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float buf_ld_f1(Rsrc r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, int(off), 0, 0));
}
template <int POLICY = 0>
__device__ __forceinline__ float4 buf_ld_f4(Rsrc r, uint32_t off) {
    const v4f_t v = __builtin_bit_cast(v4f_t, __builtin_amdgcn_raw_buffer_load_b128(r, int(off), 0, POLICY));
    return make_float4(v.x, v.y, v.z, v.w);
}
template <int POLICY = 0>
__device__ __forceinline__ uint2 buf_ld_u2(Rsrc r, uint32_t off) {
    const v2u_t v = __builtin_amdgcn_raw_buffer_load_b64(r, int(off), 0, POLICY);
    return make_uint2(v.x, v.y);
}
// Kept 16 bits wide until it is used: widening right here would put an instruction that needs the
// value directly behind the load, and with it a wait for a row that was only just requested.
__device__ __forceinline__ uint16_t buf_ld_u16(Rsrc r, uint32_t off) {
    return uint16_t(__builtin_amdgcn_raw_buffer_load_b16(r, int(off), 0, 0));
}

template <typename T>
__device__ __forceinline__ T ld(const void* base, uint32_t byte_off) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + byte_off);
}
template <typename T>
__device__ __forceinline__ void st(void* base, uint32_t byte_off, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

__device__ __forceinline__ void load8(const float* p, float out[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
}

// =====================================================================================================
// Fast path: cols % 128 == 0, so a block never straddles a row.  Here a lane owns FOUR consecutive
// elements of a row and a group of 32 lanes (half a wave) owns one 128-element block: a group's
// 128-bit parameter access is 512 contiguous bytes, and the per-lane register footprint lets five
// waves share a SIMD.  A group walks down rows of one column block with the old and the running new
// column maxima of its 4 columns in registers.  Loads go through bounds-checked buffer resources of
// the tile (uniform base, 32-bit lane offsets); the loads of the next two rows are in flight while a
// row is computed.
// =====================================================================================================

constexpr int kGroups = 8;          // 32-lane groups per workgroup

// maximum over the 32 lanes of a group of a value that is >= +0 everywhere, result in all 32 lanes
__device__ __forceinline__ float group32_allmax(float v) {
    uint32_t x = __float_as_uint(row16_allmax(v));
    // lane ^ 16 inside each half wave: swizzle in bit mode (and 0x1F, or 0, xor 0x10)
    const uint32_t y = uint32_t(__builtin_amdgcn_ds_swizzle(int(x), 0x401F));
    return __uint_as_float(x > y ? x : y);
}

template <bool BF16> struct GradRegs4;
template <> struct GradRegs4<true> { uint2 w; };
template <> struct GradRegs4<false> { float4 a; };

// gradient of a lane's 4 elements; off4 is the byte offset the elements have in an fp32 array.
// POLICY = kPolicyNt where the gradient is read for the last time in the step.
template <bool BF16, int POLICY = 0>
__device__ __forceinline__ GradRegs4<BF16> load_grad_regs4(Rsrc g_tile, uint32_t off4) {
    GradRegs4<BF16> r;
    if constexpr (BF16) r.w = buf_ld_u2<POLICY>(g_tile, off4 >> 1);
    else r.a = buf_ld_f4<POLICY>(g_tile, off4);
    return r;
}
template <bool BF16>
__device__ __forceinline__ void unpack_grad4(const GradRegs4<BF16>& r, float out[4]) {
    if constexpr (BF16) {
        out[0] = bf16_lo(r.w.x); out[1] = bf16_hi(r.w.x);
        out[2] = bf16_lo(r.w.y); out[3] = bf16_hi(r.w.y);
    } else {
        out[0] = r.a.x; out[1] = r.a.y; out[2] = r.a.z; out[3] = r.a.w;
    }
}

// float(code) of a lane's 4 codes (16 bits): split into low and high nibbles (kept opaque so that
// the byte-to-float converts are used), then one convert per element
__device__ __forceinline__ void codes_to_float4(uint32_t w, float qf[4]) {
    uint32_t lo = w & 0x0F0Fu, hi = (w >> 4) & 0x0F0Fu;
    asm("" : "+v"(lo));
    asm("" : "+v"(hi));
    qf[0] = float(lo & 255u);
    qf[1] = float(hi & 255u);
    qf[2] = float((lo >> 8) & 255u);
    qf[3] = float((hi >> 8) & 255u);
}

// il * pitch + x for a row index and a pitch that both fit 24 bits (rows of a tile; cols <= 2^24).
// The 24-bit multiply-add is a single 32-bit instruction; a full 32-bit multiply-add would go through
// the 64-bit one, whose unused upper addend register the compiler may alias with a register that a
// prefetch is still loading into, which turns into a wait for that prefetch.
__device__ __forceinline__ uint32_t row_offset(int il, int64_t pitch, uint32_t x) {
    return __umul24(uint32_t(il), uint32_t(pitch)) + x;
}

struct Geo {            // where this group works
    int strip, grp, l, gxi, gyi, cb;
    int64_t row0;
    int n_rows;         // rows of this tile
    uint32_t col0;      // first of the lane's 4 columns
};

// The rows of a tile that the groups (waves) side by side take one after the other: group g takes rows (g << rs) +
// walk(k), k = 0, 1, ...  walk(k) and the number of rounds are the same for all groups -- for group 0, which has the
// most rows in a cut-off tile -- so the loop counter and everything derived from it stay in scalar registers; a group
// whose row lies behind the tile's end reads zeros (with zero scales: see the tiles) and its stores are dropped by the
// bounds check.  With a loop bound of its own per group the counter was a vector value and index arithmetic a fifth of
// the vector instructions.
struct RowWalk {
    int rs, hop;        // hop = groups << rs
    __device__ __forceinline__ int at(int k) const { return (k & ((1 << rs) - 1)) + (k >> rs) * hop; }
    __device__ __forceinline__ int rounds(int n) const {          // number of k with at(k) < n
        const int rest = n % hop, run = 1 << rs;
        return (n / hop) * run + (rest < run ? rest : run);
    }
};

__device__ __forceinline__ Geo geometry(const Tensor4& a, int wg) {
    Geo g;
    g.strip = wg % a.strips;
    const int tile = wg / a.strips;
    g.grp = threadIdx.x >> 5;
    g.l = threadIdx.x & 31;
    g.gxi = g.grp % a.gx;
    g.gyi = g.grp / a.gx;
    g.cb = g.strip * a.gx + g.gxi;
    g.row0 = int64_t(tile) * a.rw;
    const int64_t left = a.rows - g.row0;
    g.n_rows = left < a.rw ? int(left) : a.rw;
    g.col0 = uint32_t(g.cb) * 128u + uint32_t(g.l) * 4u;
    return g;
}

// uniform base pointers of a tile (row0 folded in), so that lane offsets fit 32 bits
struct TileBase {
    float* p;
    const char* g;
    uint8_t* mq;
    uint8_t* vq;
    float* ms;
    const float* r;
    float* r_new;
    // the same arrays as bounds-checked resources of n_rows rows, for the loads and the row stores
    Rsrc rp, rg, rmq, rvq;
};

template <bool BF16>
__device__ __forceinline__ TileBase tile_base(const Tensor4& a, int64_t row0, int n_rows) {
    TileBase b;
    const int64_t e = row0 * a.cols;
    const uint32_t elems = uint32_t(n_rows) * uint32_t(a.cols);       // < 2^29
    b.p = a.p + e;
    b.g = reinterpret_cast<const char*>(a.g) + e * (BF16 ? 2 : 4);
    b.mq = reinterpret_cast<uint8_t*>(a.mq) + (e >> 1);
    b.vq = reinterpret_cast<uint8_t*>(a.vq) + (e >> 1);
    b.ms = a.ms + row0 * a.nb;
    b.r = a.r + row0;
    b.r_new = a.r_new + row0;
    b.rp = tile_rsrc(b.p, elems * 4u);
    b.rg = tile_rsrc(b.g, elems * (BF16 ? 2u : 4u));
    b.rmq = tile_rsrc(b.mq, elems >> 1);
    b.rvq = tile_rsrc(b.vq, elems >> 1);
    return b;
}

__device__ __forceinline__ void load4(const float* p, float out[4]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
}

template <bool BF16>
struct Row1 {                      // everything the second pass prefetches for one unit of one lane
    float4 p;
    GradRegs4<BF16> g;
    uint16_t mq, vq;               // the lane's 4 codes of each moment
};

// The old block scales of m and the old row maxima of v of a tile are not prefetched per row (each would be a
// load of 4 bytes that all 32 lanes of a group share): the tile stages them in LDS once, in the slots that
// later take the new block scales and the new row maxima (s.blk_scale, s.blk_vmax).  A slot's old value is
// read by the same group that replaces it, earlier in program order.

// parameters and first-moment codes of a lane's 4 elements, through the tile's bounds-checked resources (no
// registers for a second set of base addresses)
__device__ __forceinline__ void store_row1(const TileBase& tb, uint32_t off4, const float w[4], uint32_t mq_new);

// off4: byte offset of the lane's 4 elements in the tile's fp32 array; offsets at or beyond the tile's end read as zeros.
// POLICY: of the gradient.
template <bool BF16, int POLICY = 0>
__device__ __forceinline__ Row1<BF16> load_row1(const TileBase& b, uint32_t off4) {
    Row1<BF16> r;
    r.p = buf_ld_f4_stream(b.rp, off4);
    r.g = load_grad_regs4<BF16, POLICY>(b.rg, off4);
    r.mq = buf_ld_u16(b.rmq, off4 >> 3);
    r.vq = buf_ld_u16(b.rvq, off4 >> 3);
    return r;
}

__device__ __forceinline__ void store_row1(const TileBase& tb, uint32_t off4, const float w[4], uint32_t mq_new) {
    const v4f_t v = {w[0], w[1], w[2], w[3]};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u_t, v), tb.rp, int(off4), 0, kPolicyNtSc1);
    __builtin_amdgcn_raw_buffer_store_b16(short(mq_new), tb.rmq, int(off4 >> 3), 0, 0);
}

// Raise a running maximum in global memory, reading it first: the value only grows during a kernel,
// so an atomic that cannot change it is skipped.  For the general path, which would otherwise send
// an atomic per element.
__device__ __forceinline__ void raise_max(float* addr, float v) {
    if (v > 0.0f && __float_as_uint(v) > __hip_atomic_load(reinterpret_cast<unsigned int*>(addr),
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomic_max_nonneg(addr, v);
}

// Codes of 4 first moments against their block's scale: reciprocal and guard; the wave recomputes with IEEE division if
// some lane came too close to a threshold or its block's scale is extreme.
__device__ __forceinline__ uint32_t compress_m4(const SearchEntry* s_search, const float mt[4], float s_new) {
    // an all-zero block (every mt is 0) takes any scale; with that out of the way one compare tells an extreme one
    const float s_div = s_new == 0.0f ? 1.0f : s_new;
    const float inv_s = __builtin_amdgcn_rcpf(s_div);
    uint32_t q = 0, dist = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
        uint32_t da, db;
        q |= quant_m_code_fast(s_search, mt[e], inv_s, da) << (4 * e);
        q |= quant_m_code_fast(s_search, mt[e + 1], inv_s, db) << (4 * e + 4);
        dist = min(min(dist, da), db);
    }
    if (__builtin_expect((__ballot(dist < kMinDistM) | __ballot(!scale_is_tame_nonzero(s_div))) != 0, 0)) {
        q = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) q |= quant_m_code(s_search, mt[e], s_new) << (4 * e);
    }
    return q;
}

constexpr int kFlatBlocks = 8;             // column blocks of an update tile's strip at most

// ---- first pass: row and column maxima of v_t ------------------------------------------------------------------------
// A workgroup takes a strip of 256 columns of rw2 rows.  A group's 32 lanes take 8 consecutive columns each of one row,
// so a row costs a lane one 4-byte load of codes and one or two 16-byte loads of the gradient.  Column maxima stay in
// registers down the tile, row maxima go through LDS; one atomic per row and column of the tile follows at its end.
template <bool BF16>
struct Row8 {
    float4 g[BF16 ? 1 : 2];
    uint32_t vq;
};

// a lane's 8 gradients, and float(code) of its 8 codes (see codes_to_float4)
template <bool BF16>
__device__ __forceinline__ void unpack_grad8(const float4 (&x)[BF16 ? 1 : 2], float g[8]) {
    if constexpr (BF16) {
        const float w[4] = {x[0].x, x[0].y, x[0].z, x[0].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            g[2 * q] = bf16_lo(__float_as_uint(w[q]));
            g[2 * q + 1] = bf16_hi(__float_as_uint(w[q]));
        }
    } else {
        g[0] = x[0].x; g[1] = x[0].y; g[2] = x[0].z; g[3] = x[0].w;
        g[4] = x[1].x; g[5] = x[1].y; g[6] = x[1].z; g[7] = x[1].w;
    }
}
__device__ __forceinline__ void codes_to_float8(uint32_t w, float qf[8]) {
    uint32_t lo = w & 0x0F0F0F0Fu, hi = (w >> 4) & 0x0F0F0F0Fu;
    asm("" : "+v"(lo));
    asm("" : "+v"(hi));
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[e] = float((e & 1 ? hi : lo) >> (8 * (e >> 1)) & 255u);
}

template <bool BF16>
__device__ __forceinline__ void maxima_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    static_assert(offsetof(Lds, cold) == offsetof(Lds, col) + sizeof(float) * kColSlots && 2 * kColSlots >= kGroups * 256,
                  "col and cold hold the groups' column maxima here");
    const int strip = wg % a.strips2, tile = wg / a.strips2;
    const int grp = threadIdx.x >> 5, l = threadIdx.x & 31;
    const int64_t row0 = int64_t(tile) * a.rw2, left = a.rows - row0;
    const int n = left < a.rw2 ? int(left) : a.rw2;
    // with an odd number of column blocks the upper half of the last strip repeats the lower half's columns
    const uint32_t col_own = uint32_t(strip) * 256u + uint32_t(l) * 8u;
    const uint32_t col0 = col_own < uint32_t(a.cols) ? col_own : col_own - 128u;
    const int64_t e0 = row0 * a.cols;
    const uint32_t elems = uint32_t(n) * uint32_t(a.cols);                    // < 2^29
    const Rsrc rg = tile_rsrc(reinterpret_cast<const char*>(a.g) + e0 * (BF16 ? 2 : 4), elems * (BF16 ? 2u : 4u));
    const Rsrc rv = tile_rsrc(reinterpret_cast<const uint8_t*>(a.vq) + (e0 >> 1), elems >> 1);
    const RowWalk walk{a.rs2, kGroups << a.rs2};
    const int rounds = walk.rounds(n);
    const int row_g = grp << a.rs2;
    const uint32_t lane_e = row_offset(row_g, a.cols, col0), pitch = uint32_t(a.cols);
    auto fetch = [&](int k) {
        const uint32_t e = lane_e + uint32_t(walk.at(k)) * pitch;             // behind the tile: zeros
        Row8<BF16> r;
        r.g[0] = buf_ld_f4(rg, e * (BF16 ? 2u : 4u));
        if constexpr (!BF16) r.g[1] = buf_ld_f4(rg, e * 4u + 16u);
        r.vq = __builtin_amdgcn_raw_buffer_load_b32(rv, int(e >> 1), 0, 0);
        return r;
    };
    constexpr int kDepth = BF16 ? 3 : 2;                  // about the same bytes in flight
    Row8<BF16> r[kDepth];
#pragma unroll
    for (int u = 0; u < kDepth; ++u) r[u] = fetch(u);
    // old statistics, requested with the first rows: one round trip to the memory in front of the loop.  Zeros for rows behind the
    // tile's end.
    float c16[8], cmax[8], r_old[kMaxRowSlots / kThreads];
    load8(a.c + col0, c16);
    const Rsrc rr = tile_rsrc(a.r + row0, uint32_t(n) * 4u);
#pragma unroll
    for (int u = 0; u < kMaxRowSlots / kThreads; ++u)
        r_old[u] = u * kThreads < a.rw2 + kGroups ? buf_ld_f1(rr, (threadIdx.x + u * kThreads) * 4u) : 0.0f;
    __builtin_amdgcn_sched_barrier(0);                    // the columns' wait does not move in front of the rows' request
    bool lane_tame = true;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lane_tame = bool(int(lane_tame) & int(scale_is_tame(c16[e])));
        c16[e] *= 0.0625f;
        cmax[e] = 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kMaxRowSlots / kThreads; ++u) {
        if (u * kThreads >= a.rw2 + kGroups) break;
        lane_tame = bool(int(lane_tame) & int(scale_is_tame(r_old[u])));
        s.blk_scale[threadIdx.x + u * kThreads] = r_old[u] * 0.0625f;
    }
    const bool tame = all_threads(s, lane_tame);                     // else the exact route for the whole tile
    auto one = [&](const Row8<BF16>& x, int k) {
        const int il = row_g + walk.at(k);
        const float r16 = s.blk_scale[il];
        float g[8], vt[8];
        unpack_grad8<BF16>(x.g, g);
        if (__builtin_expect(tame, 1)) {
            float qf[8];
            codes_to_float8(x.vq, qf);
#pragma unroll
            for (int e = 0; e < 8; ++e) vt[e] = dequant_v16(qf[e], min_nonneg(r16, c16[e]));
        } else {
            const float r_old = il < n ? a.r[row0 + il] : 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) vt[e] = dequant_v((x.vq >> (4 * e)) & 15u, fminf(r_old, a.c[col0 + e]));
        }
        float rmax = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            vt[e] = moment_v(h, vt[e], g[e]);
            cmax[e] = fmaxf(cmax[e], vt[e]);              // a NaN raises no maximum
        }
#pragma unroll
        for (int e = 0; e < 8; e += 2) rmax = fmaxf(fmaxf(rmax, vt[e]), vt[e + 1]);
        rmax = group32_allmax(rmax);
        if (l == 0) s.blk_vmax[il] = rmax;
    };
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);              // loop start-up state: nothing outstanding
    int k = 0;
    while (k + kDepth - 1 < rounds) {                     // a register set is reloaded right after its row
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
#pragma unroll
    for (int e = 0; e < 8; ++e) s.col[grp * 256 + l * 8 + e] = cmax[e];
    __syncthreads();
    for (int t = threadIdx.x; t < n; t += kThreads) {
        const float m = s.blk_vmax[t];
        if (m > 0.0f) atomic_max_nonneg(a.r_new + row0 + t, m);
    }
    {
        const int t = threadIdx.x;
        const int64_t col = int64_t(strip) * 256 + t;
        float m = 0.0f;
#pragma unroll
        for (int y = 0; y < kGroups; ++y) m = fmaxf(m, s.col[y * 256 + t]);
        if (col < a.cols && m > 0.0f) atomic_max_nonneg(a.c_new + col, m);
    }
}

// The workgroup of a tensor's second pass that takes the last ticket makes r', c' the state and clears the
// workspace.  Every other workgroup has read the old r, c before it took its ticket, so
// overwriting them is safe.  Tickets are taken in two levels (kTicketLanes first-level counters, one
// cache line apart, then one top counter) so that thousands of workgroups do not queue up on a
// single address.  `me` / `participants`: this workgroup's index among, and the number of,
// workgroups that call this for the tensor.
constexpr int kTicketLanes = 32;
constexpr int kTicketStride = 32;                                  // in 32-bit words: 128 bytes
constexpr int kMaxTotSlots = 8;                                    // lines behind the ticket counters, for the
                                                                   // factorized step's two float sums
constexpr int kCounterWords = (1 + kTicketLanes + kMaxTotSlots) * kTicketStride;  // per tensor
// first-level counters that `participants` workgroups use = what the top counter ends at
__device__ __forceinline__ unsigned int lanes_used(unsigned int participants) {
    return participants < kTicketLanes ? participants : unsigned(kTicketLanes);
}

// A word of the workspace (the new maxima or sums) as the second pass reads it.  SAME_LAUNCH: the first pass of the
// tensor ran in the same launch, on other XCDs, so the load has to see what their atomics left (agent scope: it does not
// take the line from this XCD's L2); between launches the kernel boundary has done that and plain loads will do.
template <bool SAME_LAUNCH>
__device__ __forceinline__ float ld_ws(const float* p) {
    if constexpr (SAME_LAUNCH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}

// The same for four consecutive words at a byte offset of a bounds-checked array of the workspace: a 16-byte load with the
// cache policy of an agent-scope one.
constexpr int kPolicySc1 = 16;
template <bool SAME_LAUNCH>
__device__ __forceinline__ float4 ld_ws4(Rsrc r, uint32_t off) { return buf_ld_f4<SAME_LAUNCH ? kPolicySc1 : 0>(r, off); }

// The new statistics become the state and the workspace is cleared, by one workgroup: dst[i] = src[i]; src[i] = 0 for the rows and
// the columns.  (src is 16-byte aligned and padded to whole quads; dst takes whole quads where it is 16-byte aligned: 4 x
// 1048576 fp32 400 us per step with single words a lane, 305 so.)  It runs alone at the end of a tensor's step, so what counts is
// latency: 16 words of the rows and 16 of the columns per thread are on their way before the first store, and finish_rank1
// requests those of the first chunk before it is known that this workgroup is the one.
struct StatRegs { float4 r[4], c[4]; };
constexpr int kStatChunk = kThreads * 4 * 4;
template <bool SAME_LAUNCH>
__device__ __forceinline__ StatRegs request_statistics(const Tensor4& a, int64_t base) {
    auto quads = [&](int64_t n) { return n <= base ? 0u : uint32_t(n - base < kStatChunk ? int(n - base + 3) / 4 : kStatChunk / 4); };
    const Rsrc rr = tile_rsrc(a.r_new + base, quads(a.rows) * 16u), rc = tile_rsrc(a.c_new + base, quads(a.cols + a.c_extra) * 16u);
    StatRegs v;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t off = uint32_t(u * kThreads + int(threadIdx.x)) * 16u;
        v.r[u] = ld_ws4<SAME_LAUNCH>(rr, off);
        v.c[u] = ld_ws4<SAME_LAUNCH>(rc, off);
    }
    return v;
}
template <bool SAME_LAUNCH>
__device__ __forceinline__ void move_statistics(const Tensor4& a, StatRegs v) {
    const int64_t cols = a.cols + a.c_extra;
    const bool quad_r = (reinterpret_cast<uintptr_t>(a.r) & 15) == 0, quad_c = (reinterpret_cast<uintptr_t>(a.c) & 15) == 0;
    for (int64_t base = 0;;) {
        auto put = [&](float* dst, float* src, int64_t n, bool quad, const float4& x, int64_t i) {
            if (i >= n) return;
            if (quad && i + 3 < n) {
                *reinterpret_cast<float4*>(dst + i) = x;
            } else {
                dst[i] = x.x;
                if (i + 1 < n) dst[i + 1] = x.y;
                if (i + 2 < n) dst[i + 2] = x.z;
                if (i + 3 < n) dst[i + 3] = x.w;
            }
            *reinterpret_cast<float4*>(src + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        };
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = base + (u * kThreads + int(threadIdx.x)) * 4;
            put(a.r, a.r_new, a.rows, quad_r, v.r[u], i);
            put(a.c, a.c_new, cols, quad_c, v.c[u], i);
        }
        base += kStatChunk;
        if (base >= a.rows && base >= cols) return;
        v = request_statistics<SAME_LAUNCH>(a, base);
    }
}

// Tickets in two steps.  take_ticket: thread 0 raises the first-level counter and returns what it held; the answer is not
// needed before ticket_is_last, so a tile that is done with the old and new statistics takes its ticket and works on.
__device__ __forceinline__ unsigned int take_ticket(unsigned int* counter, unsigned int me) {
    return threadIdx.x == 0 ? atomicAdd(counter + (1 + me % kTicketLanes) * kTicketStride, 1u) : 0u;
}
// true in every thread of the one workgroup that took the last ticket; `counter`: the top counter, the first-level ones on
// the following lines
__device__ __forceinline__ bool ticket_is_last(unsigned int* counter, unsigned int me, unsigned int participants,
                                               unsigned int ticket, int& s_last) {
    if (threadIdx.x == 0) {
        const unsigned int lane = me % kTicketLanes;
        const unsigned int in_lane = participants / kTicketLanes + (lane < participants % kTicketLanes ? 1u : 0u);
        int last = 0;
        if (ticket == in_lane - 1) {
            // this lane is complete: reset it (past the L2: its line holds words that other workgroups still count on)
            __hip_atomic_store(counter + (1 + lane) * kTicketStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = atomicAdd(counter, 1u) == lanes_used(participants) - 1;
        }
        s_last = last;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(s_last) != 0;       // a scalar branch: the same in every lane
}
__device__ __forceinline__ bool last_to_arrive(unsigned int* counter, unsigned int me, unsigned int participants,
                                               int& s_last) {
    // No fence: the ticket orders nothing but "this workgroup's loads of r, c have returned", which holds once its waves
    // have computed with them and reached the barrier.  (An agent-scope release here would write back the XCD's whole L2
    // once per workgroup.)
    __syncthreads();
    return ticket_is_last(counter, me, participants, take_ticket(counter, me), s_last);
}

// The end of a second pass that is a launch of its own: every workgroup calls this with its ticket, and the one with the last
// makes r', c' the state.  A workgroup whose ticket completed a first-level counter (32 of them at most) requests what is to be
// published, final since the first pass ended, beside the top counter's answer: one round trip to the memory less in the chain
// at the step's end (fp32, us per step: 768 x 3072 15.2 -> 14.6, 4096 x 1024 19.7 -> 18.8).  Not below four workgroups to a
// first-level counter: there most workgroups would request it in vain (200 tensors of 256 x 512, bf16 gradients: 87.8 us, without 85.0).  The
// factorized form, which reads the old statistics, too, gains nothing from it.
constexpr unsigned int kFinishMany = 4 * kTicketLanes;
__device__ __forceinline__ void finish_rank1(const Tensor4& a, unsigned int me, unsigned int participants, unsigned int ticket,
                                             int (&s_last)[2]) {
    StatRegs v;
    if (participants < kFinishMany) {
        if (!ticket_is_last(a.counter, me, participants, ticket, s_last[0])) return;
        v = request_statistics<false>(a, 0);
    } else {
        const unsigned int lane = me % kTicketLanes;
        const unsigned int in_lane = participants / kTicketLanes + (lane < participants % kTicketLanes ? 1u : 0u);
        if (threadIdx.x == 0) s_last[0] = ticket == in_lane - 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_last[0]) == 0) return;
        unsigned int top = 0u;
        if (threadIdx.x == 0) {
            __hip_atomic_store(a.counter + (1 + lane) * kTicketStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            top = atomicAdd(a.counter, 1u);
        }
        v = request_statistics<false>(a, 0);
        if (threadIdx.x == 0) s_last[1] = top == lanes_used(participants) - 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_last[1]) == 0) return;
    }
    move_statistics<false>(a, v);
    if (threadIdx.x == 0) *a.counter = 0u;
}

// What a tile of a second pass is told and tells.  ready(): called once by every thread, after everything that does not
// depend on the first pass has been requested; false leaves the tile undone.  staged(): called once by every thread, behind a
// barrier, when the workgroup has read all it needs of the old and the new statistics.
// nothing of both
struct NoSync {
    __device__ __forceinline__ bool ready() { return true; }
    __device__ __forceinline__ void staged() {}
};
// a launch of its own: the ticket of the publishing workgroup
struct TicketSync {
    unsigned int* counter;
    unsigned int me, ticket;
    __device__ __forceinline__ bool ready() { return true; }
    __device__ __forceinline__ void staged() { ticket = take_ticket(counter, me); }
};

// ---- second pass: the whole update ----------------------------------------------------------------------------------
// decompress m and v, Eq. 1, parameter update, compress m against its block's maximum and v against min(r', c').
// A workgroup's tile is gx (1..8) column blocks of rw rows; a group takes rw / 8 consecutive rows and walks ALONG each, block
// after block, so that it reads and writes runs of up to 4 KiB.  The groups' rows are 2^rs rows apart, 32 KiB of parameters
// where rows of a power of two of elements allow it: a super-tile of 8 << rs rows is dealt to (8 << rs) / rw workgroups.  The
// memory system serves accesses side by side at exactly that distance fastest (this pass by itself, bf16 gradients, 246 M
// parameters: 8192 columns 6.5 TB/s 32 KiB apart, 5.9 next to each other's double distance or farther; 4096 columns 6.4, 6.0 at 16
// KiB, 5.8 at 64 KiB; 11008 columns, whose rows never are that far apart, 5.8 for neighbouring rows and 5.5 at 32 of them).
// What a lane needs of its 4 columns (old maxima / 16, approximate inverses of the new ones) sits in LDS, and so do the rows'
// scalars and the blocks' scales.  The loads of two units (one block of one row) are in flight while a third is computed
// (three register sets take turns, the loop is unrolled by three); the prefetch is unconditional, units behind the tile come
// back as zeros or are never used.

// The rows' scalars of an update tile, in s.blk_vmax: {old maximum / 16, approx. 16 / new maximum} per row, then the new maxima.
constexpr int kRowSlots = 160;
static_assert(3 * kRowSlots <= kMaxRowSlots, "row scalars of an update tile");
__device__ __forceinline__ void stage_row_old(Lds& s, int t, float r) { s.blk_vmax[2 * t] = r * 0.0625f; }
__device__ __forceinline__ void stage_row_new(Lds& s, int t, float r) {
    s.blk_vmax[2 * t + 1] = approx_inv16(r);
    s.blk_vmax[2 * kRowSlots + t] = r;
}
__device__ __forceinline__ float2 row_scalars(const Lds& s, int t) { return *reinterpret_cast<const float2*>(&s.blk_vmax[2 * t]); }
__device__ __forceinline__ float row_new(const Lds& s, int t) { return s.blk_vmax[2 * kRowSlots + t]; }

// Codes of 4 second moments against their scales, inv[e] = 16 / scale approximately; false in `sure` if some lane of the wave
// came too close to a boundary.
__device__ __forceinline__ uint32_t compress_v4(const float vt[4], const float inv[4], bool& sure) {
    // even elements collect in the bytes of `lo`, odd ones in `hi`; word = lo | hi << 4
    uint32_t lo = 0, hi = 0;
    float closest = 0.5f, fa, fb;
#define LPMM_V2(K)                                                                                        \
    lo = quant_v_code_fast<K>(vt[2 * K], inv[2 * K], lo, fa);                                             \
    hi = quant_v_code_fast<K>(vt[2 * K + 1], inv[2 * K + 1], hi, fb);                                     \
    closest = fminf(fminf(closest, fabsf(fa)), fabsf(fb));
    LPMM_V2(0) LPMM_V2(1)
#undef LPMM_V2
    sure = __ballot(closest < kMarginV) == 0;
    return lo | (hi << 4);
}

__device__ __forceinline__ void store_vq(const TileBase& tb, uint32_t off4, uint32_t vq_new) {
    __builtin_amdgcn_raw_buffer_store_b16(short(vq_new), tb.rvq, int(off4 >> 3), 0, 0);
}

// One unit.  off4: byte offset of the lane's elements in the tile; row, il: the row, in the tensor and in the tile; j = block inside the strip (the same for all
// lanes), cb0 = the strip's first column block.
template <bool BF16, class Mid>
__device__ __forceinline__ void update_unit(const Tensor4& a, const Hyper& h, const TileBase& tb, LdsRank1& s,
                                            const Row1<BF16>& cur, uint32_t off4, int64_t row, int il, int j, int cb0, int l,
                                            bool tame, Mid mid) {
    float w[4] = {cur.p.x, cur.p.y, cur.p.z, cur.p.w};
    float g[4];
    unpack_grad4<BF16>(cur.g, g);
    float mt[4], vt[4], amax = 0.0f;
    const float s_old = s.blk_scale[il * kFlatBlocks + j];     // staged by the tile; replaced below
    const float2 rs = row_scalars(s, il);
    const int at = j * 128 + l * 4;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float2 t = s.deq[(uint32_t(cur.mq) >> (8 * k)) & 255u];
        mt[2 * k] = t.x * s_old;              // decompress: T_DE[code] * block scale
        mt[2 * k + 1] = t.y * s_old;
    }
    if (__builtin_expect(tame, 1)) {          // no old or new scale of the tile is extreme
        float qf[4];
        codes_to_float4(cur.vq, qf);
        const float4 c16 = *reinterpret_cast<const float4*>(&s.cold[at]);
        const float cold16[4] = {c16.x, c16.y, c16.z, c16.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) vt[e] = dequant_v16(qf[e], min_nonneg(rs.x, cold16[e]));
    } else {
        const float r_old = row < a.rows ? a.r[row] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) vt[e] = dequant_v((uint32_t(cur.vq) >> (4 * e)) & 15u, fminf(r_old, a.c[cb0 * 128 + at + e]));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        mt[e] = moment_m(h, mt[e], g[e]);
        vt[e] = moment_v(h, vt[e], g[e]);
        w[e] = param_update(h, w[e], mt[e], vt[e]);
        amax = fmaxf(amax, fabsf(mt[e]));
    }
    // the caller's prefetch of a later unit is issued here, in the middle of the arithmetic: by now the previous unit's
    // stores have been acknowledged, and loads queue behind older stores
    __builtin_amdgcn_sched_barrier(0);
    mid();
    __builtin_amdgcn_sched_barrier(0);
    const float s_new = group32_allmax(amax);     // block absmax of m_t
    uint32_t vq_new = 0;
    bool sure = false;
    if (__builtin_expect(tame, 1)) {
        const float4 ic = *reinterpret_cast<const float4*>(&s.col[at]);
        const float inv[4] = {max_nonneg(rs.y, ic.x), max_nonneg(rs.y, ic.y), max_nonneg(rs.y, ic.z), max_nonneg(rs.y, ic.w)};
        vq_new = compress_v4(vt, inv, sure);
    }
    if (__builtin_expect(!sure, 0)) {
        const float r_new = row_new(s, il);
        vq_new = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) vq_new |= quant_v_code(vt[e], fminf(r_new, s.cnew[at + e])) << (4 * e);
    }
    store_row1(tb, off4, w, compress_m4(s.search, mt, s_new));
    store_vq(tb, off4, vq_new);
    if (l == 0) s.blk_scale[il * kFlatBlocks + j] = s_new;
}

// Where a workgroup of an update works, and the units in the order its groups take them: unit q = block q % nbk of the group's row
// number q / nbk.
struct FlatTile {
    int cb0, nbk;                // the strip's first column block, and its blocks, 1..8
    int pl, per, rs, slice0;     // rows of a group, a power of two; 2^(rs - pl) workgroups share a super-tile
    int n;                       // rows of the super-tile
    int grp, l, row_g, nq;
    int64_t row0;
    uint32_t inv_nbk, lane4, pitch4;
    __device__ __forceinline__ FlatTile(const Tensor4& a, int wg) {
        const int strip = wg % a.strips, tile = wg / a.strips;
        grp = threadIdx.x >> 5, l = threadIdx.x & 31;
        cb0 = strip * a.gx;
        nbk = a.nb - cb0 < a.gx ? a.nb - cb0 : a.gx;
        pl = __builtin_ctz(a.rw) - 3, per = 1 << pl, rs = a.rs;
        row0 = int64_t(tile >> (rs - pl)) << (rs + 3);
        slice0 = (tile & ((1 << (rs - pl)) - 1)) << pl;
        const int64_t left = a.rows - row0;
        n = left < (kGroups << rs) ? int(left) : kGroups << rs;
        nq = per * nbk;
        inv_nbk = (65536u + uint32_t(nbk) - 1u) / uint32_t(nbk);         // q / nbk == (q * inv_nbk) >> 16 for q < 9000
        row_g = grp * per;
        lane4 = row_offset((grp << rs) + slice0, a.cols, uint32_t(cb0) * 128u + uint32_t(l) * 4u) * 4u;
        pitch4 = uint32_t(a.cols) * 4u;
    }
    // of the tile's il-th row, in the super-tile
    __device__ __forceinline__ int row_of(int il) const { return (il >> pl << rs) + slice0 + (il & (per - 1)); }
    __device__ __forceinline__ int krow(int q) const { return int((uint32_t(q) * inv_nbk) >> 16); }
    __device__ __forceinline__ uint32_t off(int q) const {
        return q < nq ? lane4 + (uint32_t(krow(q)) * pitch4 + uint32_t(q - krow(q) * nbk) * 512u) : kNowhere;
    }
};

// SAME_LAUNCH: the first pass of the tensor runs in the same launch.
template <bool BF16, bool SAME_LAUNCH, class Sync>
__device__ __forceinline__ void update_tile(const Tensor4& a, const Hyper& h, int wg, LdsRank1& s, Sync& sync) {
    const TableRegs tables = request_tables();
    const FlatTile f(a, wg);
    const int cb0 = f.cb0, nbk = f.nbk, n = f.n, nq = f.nq, l = f.l, row_g = f.row_g;
    const int64_t row0 = f.row0;
    const TileBase tb = tile_base<BF16>(a, row0, n);
    auto row_of = [&](int il) { return f.row_of(il); };
    auto krow = [&](int q) { return f.krow(q); };
    auto off = [&](int q) { return f.off(q); };
    auto fetch = [&](int q) { return load_row1<BF16, kPolicyNt>(tb, off(q)); };        // the gradient's last use in the step
    // Start-up: everything a workgroup needs before its first unit is requested before any of it is waited for, one round
    // trip in front of ready() and one behind it.  Thread t takes columns 4t .. 4t+3 of the strip, blocks t and t + 256 and row t.
    const int t = threadIdx.x;
    static_assert(kFlatBlocks * 128 <= 4 * kThreads && 64 * kFlatBlocks <= 2 * kThreads, "start-up of an update tile");
    const uint32_t strip_bytes = uint32_t(nbk) * 512u;
    const float4 c_old = buf_ld_f4(tile_rsrc(a.c + cb0 * 128, strip_bytes), uint32_t(t) * 16u);
    float ms_old[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int il = (t + u * kThreads) / kFlatBlocks, j = t % kFlatBlocks, row = row_of(il);
        ms_old[u] = il < a.rw && row < n && j < nbk ? tb.ms[row_offset(row, a.nb, uint32_t(cb0 + j))] : 0.0f;
    }
    const bool row_in = t < a.rw && row_of(t) < n;
    const float r_old = row_in ? tb.r[row_of(t)] : 0.0f;
    float4 c_new;
    float r_new;
    auto request_new = [&] {
        c_new = ld_ws4<SAME_LAUNCH>(tile_rsrc(a.c_new + cb0 * 128, strip_bytes), uint32_t(t) * 16u);
        r_new = row_in ? ld_ws<SAME_LAUNCH>(tb.r_new + row_of(t)) : 0.0f;
    };
    if constexpr (!SAME_LAUNCH) request_new();
    Row1<BF16> r0 = fetch(0);
    Row1<BF16> r1 = fetch(1);
    Row1<BF16> r2;
    put_tables(s, tables);
    bool lane_tame = true;
    auto tame_too = [&](float x) { lane_tame = bool(int(lane_tame) & int(scale_is_tame(x))); return x; };
    reinterpret_cast<float4*>(s.cold)[t] = make_float4(tame_too(c_old.x) * 0.0625f, tame_too(c_old.y) * 0.0625f,
                                                       tame_too(c_old.z) * 0.0625f, tame_too(c_old.w) * 0.0625f);
    // old block scales of m into the slots of the new ones; zeros for rows behind the tile's end
    s.blk_scale[t] = ms_old[0];
    s.blk_scale[t + kThreads] = ms_old[1];
    if (t < a.rw) stage_row_old(s, t, tame_too(r_old));
    if (!sync.ready()) return;
    if constexpr (SAME_LAUNCH) request_new();
    reinterpret_cast<float4*>(s.cnew)[t] = make_float4(tame_too(c_new.x), tame_too(c_new.y), tame_too(c_new.z), tame_too(c_new.w));
    reinterpret_cast<float4*>(s.col)[t] = make_float4(approx_inv16(c_new.x), approx_inv16(c_new.y), approx_inv16(c_new.z), approx_inv16(c_new.w));
    if (t < a.rw) stage_row_new(s, t, tame_too(r_new));
    const bool tame = all_threads(s, lane_tame);     // an extreme scale anywhere: the exact route for the whole tile
    // Everything requested so far has to be here before the first unit anyway.  Saying so with an explicit wait gives the
    // loop a start-up state with nothing outstanding; otherwise the start-up's own (tight) wait counts are merged into
    // the loop head and drain the prefetch in every round.
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    if (tame) sync.staged();                                  // the exact route reads old statistics all along
    auto none = [] {};
    auto unit = [&](const Row1<BF16>& cur, int qq, auto mid) {
        const int k = krow(qq);
        update_unit<BF16>(a, h, tb, s, cur, off(qq), row0 + row_of(row_g + k), row_g + k, qq - k * nbk, cb0, l, tame, mid);
    };
    // Rounds of three units while all three exist; the loop has no exit in its middle, so that every path through it sees
    // the same queue of outstanding loads and the compiler's wait counts are exact (an early exit would join a path on
    // which the newest prefetch is still pending, and the loop head would then wait for it).  At most two units remain.
    int q = 0;
    while (q + 2 < nq) {
        unit(r0, q, [&] { r2 = fetch(q + 2); });
        unit(r1, q + 1, [&] { r0 = fetch(q + 3); });
        unit(r2, q + 2, [&] { r1 = fetch(q + 4); });
        q += 3;
    }
    if (q < nq) {
        unit(r0, q, none);
        if (q + 1 < nq) unit(r1, q + 1, none);
    }
    __syncthreads();
    if (!tame) sync.staged();
    for (int k = t; k < a.rw * kFlatBlocks; k += kThreads) {
        const int row = row_of(k / kFlatBlocks), j = k % kFlatBlocks;
        if (row < n && j < nbk) st<float>(tb.ms, row_offset(row, a.nb, uint32_t(cb0 + j)) * 4u, s.blk_scale[k]);
    }
}

constexpr int kWaves = kThreads / 64;
constexpr int kMaxRw2 = 64 * kWaves;      // rows of a statistics tile of the ragged and the factorized forms

// Statistics tiles of ragged matrices (rows that are no multiple of 128 elements long) take groups of 8 consecutive elements,
// aligned in the flattening; the last such group of a row may reach up to 7 elements into the next row.  Where that would
// reach beyond the tensor (its size is no multiple of 8) its last elements are left to a workgroup of their own, and a single row to
// workgroups that take kLastRowElems elements each.  (A last row left to them, every element of it with an atomic of its own, made short
// tensors of 4 modulo 8 elements slower than with groups of 4: rank-1 4 x 50257 bf16 22.7 us with those, 23.8, 23.1 so; 28 x 50257 27.3, 28.3, 27.2; 4 x 1000003
// 260, 283, 260.)
__host__ __device__ __forceinline__ int64_t class_rows(const Tensor4& a) { return a.rows == 1 && (a.P & 7) ? 0 : a.rows; }
constexpr int kLastRowElems = kThreads * 8;
__host__ __device__ __forceinline__ int64_t tail_begin(const Tensor4& a) { return a.rows == 1 ? 0 : a.P & ~int64_t(7); }

// =====================================================================================================
// Block-wise second moment (1-dimensional or flattened tensors; Sec. 4.2, last paragraph): both
// moments are normalized per block of 128 elements, nothing crosses a block, and the whole step is
// ONE pass.  Same lane layout as update_tile (4 elements per lane, 32 lanes per block).  The 8 groups of a
// workgroup work 64 blocks = 32 KiB of parameters apart (the distance the memory system serves
// fastest, as for the rows there): the tensor is cut into super-tiles of 8 x 64 blocks, group g
// owns blocks [64 g, 64 g + 64) of a super-tile, and a workgroup takes `rounds` consecutive blocks of
// each of the 8 ranges, so 64 / rounds workgroups share a super-tile.  The tensor is a.P elements,
// a.r holds the second moment's block scales.  The tile routine covers whole blocks; a ragged last
// block is done by b128_tail_block.
// =====================================================================================================

struct TileB {
    float* p;
    uint8_t* mq;
    uint8_t* vq;
    float* ms;
    float* vs;
    Rsrc rp, rg, rmq, rvq;                // bounds-checked views of the tile, for the loads and stores
};

template <bool BF16>
__device__ __forceinline__ TileB tile_b128(const Tensor4& a, int64_t blk0, int n_blk) {
    TileB b;
    const int64_t e = blk0 * 128;
    const uint32_t elems = uint32_t(n_blk) * 128u;
    b.p = a.p + e;
    b.mq = reinterpret_cast<uint8_t*>(a.mq) + (e >> 1);
    b.vq = reinterpret_cast<uint8_t*>(a.vq) + (e >> 1);
    b.ms = a.ms + blk0;
    b.vs = a.r + blk0;
    b.rp = tile_rsrc(b.p, elems * 4u);
    b.rg = tile_rsrc(reinterpret_cast<const char*>(a.g) + e * (BF16 ? 2 : 4), elems * (BF16 ? 2u : 4u));
    b.rmq = tile_rsrc(b.mq, elems >> 1);
    b.rvq = tile_rsrc(b.vq, elems >> 1);
    return b;
}

template <bool BF16>
struct RowB {                      // everything the step reads for one block, per lane
    float4 p;
    GradRegs4<BF16> g;
    uint16_t mq, vq;               // the lane's 4 codes of each moment
};                                 // (the block's two old scales come from LDS, staged by the tile)

constexpr uint32_t kNoBlock = 1u << 30;     // a byte offset beyond any tile: loads return zeros, stores are dropped

// off4: byte offset of the lane's elements in the (super-)tile; offsets at or beyond its end read as zeros
// SGDM: the tensor has no second moment (SGD with momentum, App. E Alg. 2)
template <bool BF16, bool SGDM = false>
__device__ __forceinline__ RowB<BF16> load_rowb(const TileB& b, uint32_t off4) {
    RowB<BF16> r;
    r.p = buf_ld_f4_stream(b.rp, off4);
    r.g = load_grad_regs4<BF16, kPolicyNt>(b.rg, off4);              // read once per step
    r.mq = buf_ld_u16(b.rmq, off4 >> 3);
    if constexpr (SGDM) r.vq = 0;
    else r.vq = buf_ld_u16(b.rvq, off4 >> 3);
    return r;
}

template <bool BF16, bool SGDM, class Mid>
__device__ __forceinline__ void b128_row(const Hyper& h, const TileB& tb, Lds& s, const RowB<BF16>& cur,
                                         uint32_t off4, int slot, int l, bool tame, Mid mid) {
    float w[4] = {cur.p.x, cur.p.y, cur.p.z, cur.p.w};
    float g[4];
    unpack_grad4<BF16>(cur.g, g);
    float mt[4], vt[4], amax = 0.0f, vmax = 0.0f;
    const float sm_old = s.blk_scale[slot];
    const float sv_old = SGDM ? 0.0f : s.blk_vmax[slot];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float2 t = s.deq[(uint32_t(cur.mq) >> (8 * k)) & 255u];
        mt[2 * k] = t.x * sm_old;             // decompress: T_DE[code] * block scale
        mt[2 * k + 1] = t.y * sm_old;
    }
    if constexpr (SGDM) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mt[e] = moment_sgdm(h, mt[e], g[e]);
            w[e] = param_sgdm(h, w[e], mt[e]);
            amax = fmaxf(amax, fabsf(mt[e]));
            vt[e] = 0.0f;
        }
    } else {
        if (__builtin_expect(tame, 1)) {                      // no old scale of the tile is extreme
            float qf[4];
            codes_to_float4(cur.vq, qf);
            const float s16 = sv_old * 0.0625f;
#pragma unroll
            for (int e = 0; e < 4; ++e) vt[e] = dequant_v16(qf[e], s16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) vt[e] = dequant_v((uint32_t(cur.vq) >> (4 * e)) & 15u, sv_old);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mt[e] = moment_m(h, mt[e], g[e]);
            vt[e] = moment_v(h, vt[e], g[e]);
            w[e] = param_update(h, w[e], mt[e], vt[e]);
            amax = fmaxf(amax, fabsf(mt[e]));
            vmax = max_nonneg(vmax, vt[e]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    mid();                                        // the caller's prefetch of a later block
    __builtin_amdgcn_sched_barrier(0);
    const float sm_new = group32_allmax(amax);    // block absmax of m_t
    const float sv_new = SGDM ? 0.0f : group32_allmax(vmax);    // block maximum of v_t

    const uint32_t mq_new = compress_m4(s.search, mt, sm_new);
    uint32_t vq_new = 0;
    if constexpr (!SGDM) {
        const float inv_s = approx_inv16(sv_new);
        uint32_t lo = 0, hi = 0;
        float closest = scale_is_tame(sv_new) ? 0.5f : 0.0f, fa, fb;
#define LPMM_VB(K)                                                               \
        lo = quant_v_code_fast<K>(vt[2 * K], inv_s, lo, fa);                     \
        hi = quant_v_code_fast<K>(vt[2 * K + 1], inv_s, hi, fb);                 \
        closest = fminf(fminf(closest, fabsf(fa)), fabsf(fb));
        LPMM_VB(0) LPMM_VB(1)
#undef LPMM_VB
        vq_new = lo | (hi << 4);
        if (__builtin_expect(__ballot(closest < kMarginV) != 0, 0)) {
            vq_new = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) vq_new |= quant_v_code(vt[e], sv_new) << (4 * e);
        }
    }

    {   // through the tile's bounds-checked resources: no registers for a second set of base addresses
        const v4f_t v = {w[0], w[1], w[2], w[3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u_t, v), tb.rp, int(off4), 0, kPolicyNtSc1);
        __builtin_amdgcn_raw_buffer_store_b16(short(mq_new), tb.rmq, int(off4 >> 3), 0, 0);
        if constexpr (!SGDM) __builtin_amdgcn_raw_buffer_store_b16(short(vq_new), tb.rvq, int(off4 >> 3), 0, 0);
    }
    if (l == 0) {
        s.blk_scale[slot] = sm_new;
        if constexpr (!SGDM) s.blk_vmax[slot] = sv_new;
    }
}

constexpr int kB128Stride = 64;                            // blocks between the groups of a workgroup
constexpr int kB128Super = kGroups * kB128Stride;          // blocks of a super-tile
constexpr int kB128MaxRounds = kB128Stride;                // block results of a tile are staged in LDS
static_assert(kGroups * kB128MaxRounds <= kMaxRowSlots, "LDS staging of block results");

// workgroup `wg` of a tensor: super-tile wg / slices, slice wg % slices of each group's range, where
// slices = 64 / a.rw and a.rw = rounds (a power of two); a.nb = whole blocks of the tensor
template <bool BF16, bool SGDM = false>
__device__ __forceinline__ void b128_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    const int rounds = a.rw, slices = kB128Stride / rounds;
    const int64_t sup0 = int64_t(wg / slices) * kB128Super;
    const int64_t left = int64_t(a.nb) - sup0;
    const int n_sup = left < kB128Super ? int(left) : kB128Super;      // blocks of this super-tile that exist
    const TileB tb = tile_b128<BF16>(a, sup0, n_sup > 0 ? n_sup : 0);
    const int grp = threadIdx.x >> 5, l = threadIdx.x & 31;
    const int slice0 = (wg % slices) * rounds;
    // The group's blocks are grp * 64 + slice0 + k, k < rounds; those behind the tensor's last block lie beyond the tile's
    // resources, and a prefetch past the group's share (a real block of another workgroup) gets an offset that does.  The
    // round is the same for all groups and stays in scalar registers.
    const uint32_t lane4 = uint32_t(grp * kB128Stride + slice0) * 512u + uint32_t(l) * 16u;
    auto off = [&](int k) { return lane4 + (k < rounds ? uint32_t(k) * 512u : kNoBlock); };
    auto fetch = [&](int k) { return load_rowb<BF16, SGDM>(tb, off(k)); };
    const int slot0 = grp * rounds;
    int k = 0;
    const TableRegs tables = request_tables();
    RowB<BF16> r0 = fetch(0);
    RowB<BF16> r1 = fetch(1);
    RowB<BF16> r2;
    bool lane_tame = true;
    for (int t = threadIdx.x; t < kGroups * rounds; t += kThreads) {   // old block scales into the slots of the new ones
        const int b = (t / rounds) * kB128Stride + slice0 + t % rounds;
        s.blk_scale[t] = b < n_sup ? tb.ms[b] : 0.0f;
        if constexpr (!SGDM) {
            const float v = b < n_sup ? tb.vs[b] : 0.0f;
            s.blk_vmax[t] = v;
            lane_tame = bool(int(lane_tame) & int(scale_is_tame(v)));
        }
    }
    put_tables(s, tables);
    __syncthreads();                               // the first blocks' loads are in flight meanwhile
    bool tame = true;
    if constexpr (!SGDM) tame = all_threads(s, lane_tame);
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);       // loop start-up state: nothing outstanding (see update_tile)
    auto none = [] {};
    auto work = [&](const RowB<BF16>& cur, int kk, auto mid) { b128_row<BF16, SGDM>(h, tb, s, cur, off(kk), slot0 + kk, l, tame, mid); };
    while (k + 2 < rounds) {                       // rounds of three blocks, no exit in the middle
        work(r0, k, [&] { r2 = fetch(k + 2); });
        work(r1, k + 1, [&] { r0 = fetch(k + 3); });
        work(r2, k + 2, [&] { r1 = fetch(k + 4); });
        k += 3;
    }
    if (k < rounds) {
        work(r0, k, none);
        if (k + 1 < rounds) work(r1, k + 1, none);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kGroups * rounds; t += kThreads) {   // new block scales: 8 contiguous runs
        const int b = (t / rounds) * kB128Stride + slice0 + t % rounds;
        if (b < n_sup) {
            tb.ms[b] = s.blk_scale[t];
            if constexpr (!SGDM) tb.vs[b] = s.blk_vmax[t];
        }
    }
}

// The last, partial block of a tensor whose size is not a multiple of 128 (a.P - 128 * a.nb
// elements, an even number).  One lane per element pair, exact arithmetic, reductions through LDS.
template <bool BF16, bool SGDM = false>
__device__ __forceinline__ void b128_tail_block(const Tensor4& a, const Hyper& h, Lds& s) {
    const int64_t e0 = int64_t(a.nb) * 128;
    const int n = int(a.P - e0);                   // 1..127
    const int t = threadIdx.x;
    const bool on = t < (n + 1) / 2;               // this lane's pair: elements e0 + 2t, e0 + 2t + 1
    float mt[2] = {0.0f, 0.0f}, vt[2] = {0.0f, 0.0f};
    const float sm_old = a.ms[a.nb], sv_old = SGDM ? 0.0f : a.r[a.nb];
    uint32_t bm = 0, bv = 0;
    if (on) {
        bm = reinterpret_cast<const uint8_t*>(a.mq)[(e0 >> 1) + t];
        if constexpr (!SGDM) bv = reinterpret_cast<const uint8_t*>(a.vq)[(e0 >> 1) + t];
    }
    for (int k = 0; k < 2; ++k) {
        const int64_t e = e0 + 2 * t + k;
        if (on && e < a.P) {
            const float2 dq = s.deq[bm];
            const float g = load_grad1<BF16>(a.g, e);
            if constexpr (SGDM) {
                mt[k] = moment_sgdm(h, (k ? dq.y : dq.x) * sm_old, g);
                a.p[e] = param_sgdm(h, a.p[e], mt[k]);
            } else {
                mt[k] = moment_m(h, (k ? dq.y : dq.x) * sm_old, g);
                vt[k] = moment_v(h, dequant_v((bv >> (4 * k)) & 15u, sv_old), g);
                a.p[e] = param_update(h, a.p[e], mt[k], vt[k]);
            }
        }
    }
    s.col[t] = fmaxf(fabsf(mt[0]), fabsf(mt[1]));
    s.col[kThreads + t] = fmaxf(vt[0], vt[1]);
    __syncthreads();
    float sm_new = 0.0f, sv_new = 0.0f;
    for (int i = 0; i < 64; ++i) {                 // every lane reduces the 64 pairs itself
        sm_new = fmaxf(sm_new, s.col[i]);
        sv_new = fmaxf(sv_new, s.col[kThreads + i]);
    }
    if (on) {
        uint32_t qm = 0, qv = 0;
        for (int k = 0; k < 2; ++k)
            if (e0 + 2 * t + k < a.P) {
                qm |= quant_m_code(s.search, mt[k], sm_new) << (4 * k);
                if constexpr (!SGDM) qv |= quant_v_code(vt[k], sv_new) << (4 * k);
            }
        reinterpret_cast<uint8_t*>(a.mq)[(e0 >> 1) + t] = uint8_t(qm);
        if constexpr (!SGDM) reinterpret_cast<uint8_t*>(a.vq)[(e0 >> 1) + t] = uint8_t(qv);
    }
    if (t == 0) {
        a.ms[a.nb] = sm_new;
        if constexpr (!SGDM) a.r[a.nb] = sv_new;
    }
}

// workgroups [0, n_wg2) run tiles of whole blocks, workgroup n_wg2 (if n_wg > n_wg2) the partial block
template <bool BF16, bool SGDM = false>
__device__ __forceinline__ void b128_work(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    if (wg < a.n_wg2) {
        b128_tile<BF16, SGDM>(a, h, wg, s);
    } else {
        load_tables(s);
        b128_tail_block<BF16, SGDM>(a, h, s);
    }
}

// =====================================================================================================
// General path: any rows x cols.  Lane t owns flat elements [8t, 8t+8); a group is still one block
// of 128, but a lane's elements may lie in different rows, so row and column indices are tracked
// per element and the maxima go straight to atomics (skipped when they cannot raise the value).
// =====================================================================================================


struct LaneIo {
    int64_t base;   // first flat element of the lane
    int nv;         // valid elements, 0..8
    int64_t i;      // row of the first element
    int64_t j;      // column of the first element
};

__device__ __forceinline__ LaneIo lane_io(int64_t P, int64_t cols, int64_t lane_global) {
    LaneIo io;
    io.base = lane_global * 8;
    const int64_t left = P - io.base;
    io.nv = left >= 8 ? 8 : (left > 0 ? int(left) : 0);
    io.i = io.nv ? io.base / cols : 0;
    io.j = io.nv ? io.base - io.i * cols : 0;
    return io;
}

// code word of a lane: full lanes read one aligned word, the tail lane reads bytes
__device__ __forceinline__ uint32_t load_codes(const uint32_t* q, const LaneIo& io) {
    if (io.nv == 8) return q[io.base >> 3];
    const uint8_t* b = reinterpret_cast<const uint8_t*>(q) + (io.base >> 1);
    uint32_t w = 0;
    for (int k = 0; k < (io.nv + 1) / 2; ++k) w |= uint32_t(b[k]) << (8 * k);
    return w;
}
__device__ __forceinline__ void store_codes(uint32_t* q, const LaneIo& io, uint32_t w) {
    if (io.nv == 8) { q[io.base >> 3] = w; return; }
    uint8_t* b = reinterpret_cast<uint8_t*>(q) + (io.base >> 1);
    for (int k = 0; k < (io.nv + 1) / 2; ++k) b[k] = uint8_t(w >> (8 * k));
}

// A workgroup of the general first pass takes a.rw (1..16, chosen by the host) consecutive chunks of 2048 elements.  The maxima of v_t
// are first combined in LDS (integer atomics on the float bits), indexed by the column -- possible when the
// tensor has at most kGenColsLds columns, which is the usual case for shapes that miss the fast path (narrow
// matrices) -- and by the row relative to the workgroup's first row; one global atomic per column and row
// that the workgroup touched follows at its end.  Wider tensors, or rows shorter than 9 elements, send their
// maxima to global atomics directly (read first, skipped when they cannot raise the value).
constexpr int kGenChunkElems = kThreads * 8;             // a.rw chunks of this many elements per workgroup
constexpr int kGenMaxChunks = 16;
constexpr int kGenColsLds = 2048;                        // s.col and s.cold together
constexpr int kGenRowsLds = 2 * kMaxRowSlots;            // s.blk_scale and s.blk_vmax together

template <bool BF16>
__device__ __forceinline__ void pass1_general_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s) {
    const int64_t e_first = int64_t(wg) * a.rw * kGenChunkElems;
    const int64_t e_end = e_first + int64_t(a.rw) * kGenChunkElems < a.P ? e_first + int64_t(a.rw) * kGenChunkElems : a.P;
    static_assert(offsetof(Lds, cold) == offsetof(Lds, col) + sizeof(float) * kColSlots, "col and cold are one array here");
    static_assert(offsetof(Lds, blk_vmax) == offsetof(Lds, blk_scale) + sizeof(float) * kMaxRowSlots, "row slots");
    unsigned int* col_l = reinterpret_cast<unsigned int*>(s.col);          // [kGenColsLds]
    unsigned int* row_l = reinterpret_cast<unsigned int*>(s.blk_scale);    // [kGenRowsLds]
    const int n_chunks = int((e_end - e_first + kGenChunkElems - 1) / kGenChunkElems);
    const int64_t i0 = e_first / a.cols;                                   // first row this workgroup touches
    const int64_t n_rows_wg = (e_end - 1) / a.cols - i0 + 1;
    const bool cols_in_lds = a.cols <= kGenColsLds;
    const bool rows_in_lds = n_rows_wg <= kGenRowsLds;
    if (cols_in_lds)
        for (int t = threadIdx.x; t < int(a.cols); t += kThreads) col_l[t] = 0u;
    if (rows_in_lds)
        for (int t = threadIdx.x; t < int(n_rows_wg); t += kThreads) row_l[t] = 0u;
    load_tables(s);                                                        // its barrier covers the zeroing too
    auto raise_col = [&](int64_t j, float v) {
        if (cols_in_lds) (void)__hip_atomic_fetch_max(col_l + j, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else raise_max(a.c_new + j, v);
    };
    auto raise_row = [&](int64_t i, float v) {
        if (rows_in_lds) (void)__hip_atomic_fetch_max(row_l + (i - i0), __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else raise_max(a.r_new + i, v);
    };
    for (int c = 0; c < n_chunks; ++c) {
        const int64_t t = e_first / 8 + int64_t(c) * kThreads + threadIdx.x;
        const int64_t block = t >> 4;                       // uniform over the 16 lanes of a block
        const bool alive = block * 128 < a.P;               // dead lanes are the highest of the last chunk
        const LaneIo io = lane_io(a.P, a.cols, t);
        float w[8], g[8];
        if (io.nv == 8) {
            load8(a.p + io.base, w);
            load_grad8<BF16>(a.g, io.base, g);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                w[e] = e < io.nv ? a.p[io.base + e] : 0.0f;
                g[e] = e < io.nv ? load_grad1<BF16>(a.g, io.base + e) : 0.0f;
            }
        }
        const uint32_t mq = io.nv ? load_codes(a.mq, io) : 0u;
        const uint32_t vq = io.nv ? load_codes(a.vq, io) : 0u;
        const float s_old = alive ? a.ms[block] : 0.0f;

        float mt[8], amax = 0.0f;
        int64_t i = io.i, j = io.j;
        int64_t run_row = io.i;
        float run_max = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e < io.nv) {
                const float2 tt = s.deq[(mq >> (8 * (e >> 1))) & 255u];
                const float m_prev = ((e & 1) ? tt.y : tt.x) * s_old;
                const float v_prev = dequant_v((vq >> (4 * e)) & 15u, fminf(a.r[i], a.c[j]));
                mt[e] = moment_m(h, m_prev, g[e]);
                const float vt = moment_v(h, v_prev, g[e]);
                w[e] = param_update(h, w[e], mt[e], vt);
                amax = fmaxf(amax, fabsf(mt[e]));
                if (i != run_row) { raise_row(run_row, run_max); run_row = i; run_max = 0.0f; }
                run_max = fmaxf(run_max, vt);
                raise_col(j, vt);
                if (++j == a.cols) { j = 0; ++i; }
            } else {
                mt[e] = 0.0f;
            }
        }
        // The lane's last row usually is its neighbours' too (rows are contiguous runs of lanes): combine
        // over the wave first, one atomic per row and wave.
        {
            const int lane = threadIdx.x & 63;
            long long rr = io.nv ? (long long)run_row : -1ll - lane;
            float rm = run_max;
            for (int d = 1; d < 64; d <<= 1) {
                const float om = __shfl_down(rm, d);
                const long long orow = __shfl_down(rr, d);
                if (lane + d < 64 && orow == rr) rm = fmaxf(rm, om);
            }
            const long long prev = __shfl_up(rr, 1);
            if (io.nv && (lane == 0 || prev != rr)) raise_row(rr, rm);
        }

        const float s_new = row16_allmax(amax);
        uint32_t mq_new = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < io.nv) mq_new |= quant_m_code(s.search, mt[e], s_new) << (4 * e);

        if (io.nv == 8) {
            float4* pp = reinterpret_cast<float4*>(a.p + io.base);
            pp[0] = make_float4(w[0], w[1], w[2], w[3]);
            pp[1] = make_float4(w[4], w[5], w[6], w[7]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < io.nv) a.p[io.base + e] = w[e];
        }
        if (io.nv) store_codes(a.mq, io, mq_new);
        if (alive && (threadIdx.x & 15) == 0) a.ms[block] = s_new;
    }
    __syncthreads();
    if (cols_in_lds)
        for (int t = threadIdx.x; t < int(a.cols); t += kThreads) {
            const unsigned int m = col_l[t];
            if (m) atomicMax(reinterpret_cast<unsigned int*>(a.c_new) + t, m);
        }
    if (rows_in_lds)
        for (int t = threadIdx.x; t < int(n_rows_wg); t += kThreads) {
            const unsigned int m = row_l[t];
            if (m) atomicMax(reinterpret_cast<unsigned int*>(a.r_new) + i0 + t, m);
        }
}

// the 2048 elements from e_first (a multiple of 8) on
template <bool BF16, bool SAME_LAUNCH = false>
__device__ __forceinline__ void pass2_general_chunk(const Tensor4& a, const Hyper& h, int64_t e_first) {
    const LaneIo io = lane_io(a.P, a.cols, e_first / 8 + threadIdx.x);
    if (!io.nv) return;
    float g[8];
    if (io.nv == 8) {
        load_grad8<BF16>(a.g, io.base, g);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) g[e] = e < io.nv ? load_grad1<BF16>(a.g, io.base + e) : 0.0f;
    }
    const uint32_t vq = load_codes(a.vq, io);
    uint32_t vq_new = 0;
    int64_t i = io.i, j = io.j;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (e < io.nv) {
            const float v_prev = dequant_v((vq >> (4 * e)) & 15u, fminf(a.r[i], a.c[j]));
            const float vt = moment_v(h, v_prev, g[e]);
            vq_new |= quant_v_code(vt, fminf(ld_ws<SAME_LAUNCH>(a.r_new + i), ld_ws<SAME_LAUNCH>(a.c_new + j))) << (4 * e);
            if (++j == a.cols) { j = 0; ++i; }
        }
    }
    store_codes(a.vq, io, vq_new);
}

// =====================================================================================================
// Factorized second moment ("4-bit Factor", Sec. 4.3): for a rows x cols tensor the second moment is
// kept as row statistics R and column statistics C, moving averages (with beta2, as v_t in Eq. 1) of
// the row and column sums of g^2, and v_t[i][j] = R_i C_j / sum_i R_i takes the place of Eq. 1's v_t.
// The first moment is compressed as everywhere (B128 + signed dynamic-exponent map).
//
// Two passes, because every element's update needs the complete sums of its row and column:
//   statistics pass: reads the gradient only; row and column sums of g^2 into the workspace (float
//                    atomics), plus two scalars: the sum of all g^2 and the sum of the old R.
//   update pass:     R_t[i] = beta2 R[i] + (1-beta2) rowsum_i, C_t[j] likewise, sum R_t = beta2 sum R +
//                    (1-beta2) sum g^2; decompress m, Eq. 1 with the reconstructed v_t, parameter
//                    update, compress m_t.  The last workgroup writes R_t, C_t to the state (the same
//                    expression every workgroup evaluated) and clears the workspace.
// Nothing integer depends on the second moment here, so the sums are plain fp32 in whatever order
// the atomics arrive: R, C and the parameters vary in their last bits from run to run; the first
// moment's codes and scales do not.
// =====================================================================================================

// The two float sums live in the counter block, behind the ticket counters.  Each is spread over
// a.tot_slots slots (a power of two; a workgroup adds to slot = its index modulo the count), one slot
// per 128-byte line, because atomics on one line queue up behind each other even when their addresses
// differ; readers add the slots in a fixed order.  A tensor stepped on its own has all its workgroups
// arrive at once and takes 8 slots; in a plan the tensors' workgroups arrive spread out, one slot
// serves, and the update pass has fewer lines to read.
__device__ __forceinline__ int tot_new_word(int slot) { return (1 + kTicketLanes + slot) * kTicketStride; }      // sum of g^2
__device__ __forceinline__ int tot_old_word(int slot) { return (1 + kTicketLanes + slot) * kTicketStride + 1; }  // sum of the old R

__device__ __forceinline__ void atomic_add_f32(float* addr, float v) { (void)unsafeAtomicAdd(addr, v); }

// new statistic from the old one and this step's sum of squares
__device__ __forceinline__ float stat_ema(const Hyper& h, float old, float sum_sq) {
    return __builtin_fmaf(h.beta2, old, h.omb2 * sum_sq);
}
template <bool SAME_LAUNCH = false>
__device__ __forceinline__ float factor_inv_total(const Tensor4& a, const Hyper& h) {
    const float* tot = reinterpret_cast<const float*>(a.counter);
    float sum_new = 0.0f, sum_old = 0.0f;
    for (int k = 0; k < a.tot_slots; ++k) {
        sum_new += ld_ws<SAME_LAUNCH>(tot + tot_new_word(k));
        sum_old += ld_ws<SAME_LAUNCH>(tot + tot_old_word(k));
    }
    const float total = stat_ema(h, sum_old, sum_new);
    return total > 0.0f ? 1.0f / total : 0.0f;          // all-zero statistics: v_t = 0
}

template <int CTRL>
__device__ __forceinline__ float dpp_fadd(float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
// sum over the 32 lanes of a half-wave, the same value in every lane (fixed order)
__device__ __forceinline__ float group32_sum(float v) {
    v = dpp_fadd<0xB1>(v);      // lane ^ 1
    v = dpp_fadd<0x4E>(v);      // lane ^ 2
    v = dpp_fadd<0x141>(v);     // other quad of the half row
    v = dpp_fadd<0x140>(v);     // other half of the row of 16
    return v + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));     // lane ^ 16
}
// the same over the 64 lanes of a wave
__device__ __forceinline__ float wave_sum(float v) {
    v = group32_sum(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)) +
           __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
}

// Statistics pass, fast path (cols % 128 == 0): a wave works on 256 consecutive
// columns of one row, the four waves of a workgroup take rows w, w+4, ... of a tile of rw2 rows.  Row
// sums are staged in LDS, column sums are combined over the four waves in LDS; one atomic per row and
// per column of the tile.
template <bool BF16>
__device__ __forceinline__ void factor_stats_tile(const Tensor4& a, int wg, Lds& s) {
    const int strip = wg % a.strips2, tile = wg / a.strips2;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    const uint32_t col0 = uint32_t(strip) * 256u + uint32_t(lane) * 4u;
    const bool live = col0 < uint32_t(a.cols);      // odd number of column blocks: upper half of the last strip
    const int64_t row0 = int64_t(tile) * a.rw2;
    const int64_t left = a.rows - row0;
    const int n = left < a.rw2 ? int(left) : a.rw2;
    const Rsrc rg = tile_rsrc(reinterpret_cast<const char*>(a.g) + row0 * a.cols * (BF16 ? 2 : 4),
                              uint32_t(n) * uint32_t(a.cols) * (BF16 ? 2u : 4u));
    float cacc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto ld = [&](int il) { return load_grad_regs4<BF16>(rg, row_offset(il, a.cols, col0) * 4u); };
    auto one = [&](const GradRegs4<BF16>& r, int il) {
        float g[4];
        unpack_grad4<BF16>(r, g);
        float sq[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sq[e] = live ? g[e] * g[e] : 0.0f;
            cacc[e] += sq[e];
        }
        const float rsum = wave_sum((sq[0] + sq[1]) + (sq[2] + sq[3]));
        if (lane == 0) s.blk_scale[il] = rsum;
    };
    // the waves' rows are 2^rs2 rows apart; three register sets take turns: a set is reloaded right after its row has been
    // summed, so the loads of two rows are in flight while a third is summed (more sets in flight measured slower)
    const int rs = a.rs2;
    const int row_w = wave << rs, hop = kWaves << rs, low = (1 << rs) - 1;
    auto row = [&](int k) { return row_w + (k & low) + (k >> rs) * hop; };
    int k = 0;
    constexpr int kDepth = 3;
    GradRegs4<BF16> r[kDepth];
#pragma unroll
    for (int u = 0; u < kDepth; ++u) r[u] = ld(row(u));
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    if (row(k + kDepth - 1) < n) do {
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            one(r[u], row(k + u));
            __builtin_amdgcn_sched_barrier(0);
            r[u] = ld(row(k + kDepth + u));
            __builtin_amdgcn_sched_barrier(0);
        }
        k += kDepth;
    } while (row(k + kDepth - 1) < n);
#pragma unroll
    for (int u = 0; u < kDepth - 1; ++u)
        if (row(k + u) < n) one(r[u], row(k + u));
#pragma unroll
    for (int e = 0; e < 4; ++e) s.col[wave * 256 + lane * 4 + e] = cacc[e];
    __syncthreads();
    if (a.det) {
        // fixed order of summation: this tile's sums go to slots of their own; factor_reduce_one adds the strips
        // of a row and the tiles of a column in index order, factor_totals_one the rows
        const int64_t rows_pad = (a.rows + 63) / 64 * 64, cols_pad = (a.cols + 63) / 64 * 64;
        float* rowpart = reinterpret_cast<float*>(a.vq) + int64_t(strip) * rows_pad + row0;
        float* colpart = reinterpret_cast<float*>(a.vq) + int64_t(a.strips2) * rows_pad + int64_t(tile) * cols_pad;
        for (int t = threadIdx.x; t < n; t += kThreads) rowpart[t] = s.blk_scale[t];
        const int t = threadIdx.x;
        const float csum = (s.col[t] + s.col[256 + t]) + (s.col[512 + t] + s.col[768 + t]);
        const int64_t col = int64_t(strip) * 256 + t;
        if (col < a.cols) colpart[col] = csum;
        return;
    }
    for (int t = threadIdx.x; t < n; t += kThreads) atomic_add_f32(a.r_new + row0 + t, s.blk_scale[t]);
    {
        const int t = threadIdx.x;
        const float csum = (s.col[t] + s.col[256 + t]) + (s.col[512 + t] + s.col[768 + t]);
        const int64_t col = int64_t(strip) * 256 + t;
        if (col < a.cols) atomic_add_f32(a.c_new + col, csum);
    }
    float* tot = reinterpret_cast<float*>(a.counter);
    if (wave == 0) {                 // the tile's share of the sum of all g^2
        float part = 0.0f;
        for (int t = lane; t < n; t += 64) part += s.blk_scale[t];
        part = wave_sum(part);
        if (lane == 0) atomic_add_f32(tot + tot_new_word(wg & (a.tot_slots - 1)), part);
    } else if (wave == 1 && strip == 0) {   // the old statistics of the tile's rows, once per row
        float part = 0.0f;
        for (int t = lane; t < n; t += 64) part += a.r[row0 + t];
        part = wave_sum(part);
        if (lane == 0) atomic_add_f32(tot + tot_old_word(tile & (a.tot_slots - 1)), part);
    }
}

template <bool BF16>
struct RowF {                      // everything the update pass reads for one row of one lane
    float4 p;
    GradRegs4<BF16> g;
    uint16_t mq;
};

template <bool BF16>
__device__ __forceinline__ RowF<BF16> load_rowf(const TileBase& b, uint32_t off4) {
    RowF<BF16> r;
    r.p = buf_ld_f4_stream(b.rp, off4);
    r.g = load_grad_regs4<BF16, kPolicyNt>(b.rg, off4);     // last use of the gradient in this step
    r.mq = buf_ld_u16(b.rmq, off4 >> 3);
    return r;
}

// One unit (a row of one column block) of the update pass for one lane; ct[e] = C_t of the lane's columns.  The unit's old block scale
// and the row's R_t[i] / sum R_t (rn) come from LDS, where the tile staged them (see update_tile).
template <bool BF16, class Mid>
__device__ __forceinline__ void factor_unit(const Hyper& h, const TileBase& tb, Lds& s, const RowF<BF16>& cur, uint32_t off4, int slot,
                                            float rn, const float ct[4], int l, Mid mid) {
    float w[4] = {cur.p.x, cur.p.y, cur.p.z, cur.p.w};
    float g[4];
    unpack_grad4<BF16>(cur.g, g);
    float mt[4], amax = 0.0f;
    const float s_old = s.blk_scale[slot];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float2 t = s.deq[(uint32_t(cur.mq) >> (8 * k)) & 255u];
        mt[2 * k] = t.x * s_old;
        mt[2 * k + 1] = t.y * s_old;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        mt[e] = moment_m(h, mt[e], g[e]);
        w[e] = param_update(h, w[e], mt[e], rn * ct[e]);
        amax = fmaxf(amax, fabsf(mt[e]));
    }
    __builtin_amdgcn_sched_barrier(0);
    mid();                                    // the caller's prefetch (see update_unit)
    __builtin_amdgcn_sched_barrier(0);
    const float s_new = group32_allmax(amax);
    store_row1(tb, off4, w, compress_m4(s.search, mt, s_new));
    if (l == 0) s.blk_scale[slot] = s_new;
}

// Update pass, fast path, of a tensor stepped on its own: the tiles of update_tile.  s.cold holds C_t of the strip's columns, s.blk_vmax
// R_t[i] / sum R_t of the tile's rows.
template <bool BF16, class Sync>
__device__ __forceinline__ void factor_update_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s, Sync& sync) {
    const TableRegs tables = request_tables();
    const FlatTile f(a, wg);
    const TileBase tb = tile_base<BF16>(a, f.row0, f.n);
    auto fetch = [&](int q) { return load_rowf<BF16>(tb, f.off(q)); };
    // start-up as in update_tile: thread t takes columns 4t .. 4t+3 of the strip, blocks t and t + 256 and row t
    const int t = threadIdx.x;
    const uint32_t strip_bytes = uint32_t(f.nbk) * 512u;
    const float4 c_old = buf_ld_f4(tile_rsrc(a.c + f.cb0 * 128, strip_bytes), uint32_t(t) * 16u);
    float ms_old[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int il = (t + u * kThreads) / kFlatBlocks, j = t % kFlatBlocks, row = f.row_of(il);
        ms_old[u] = il < a.rw && row < f.n && j < f.nbk ? tb.ms[row_offset(row, a.nb, uint32_t(f.cb0 + j))] : 0.0f;
    }
    const bool row_in = t < a.rw && f.row_of(t) < f.n;
    const float r_old = row_in ? tb.r[f.row_of(t)] : 0.0f;
    const float4 c_sum = buf_ld_f4(tile_rsrc(a.c_new + f.cb0 * 128, strip_bytes), uint32_t(t) * 16u);
    const float r_sum = row_in ? tb.r_new[f.row_of(t)] : 0.0f;
    RowF<BF16> r0 = fetch(0), r1 = fetch(1), r2;
    put_tables(s, tables);
    s.blk_scale[t] = ms_old[0];
    s.blk_scale[t + kThreads] = ms_old[1];
    const float inv_total = factor_inv_total(a, h);
    reinterpret_cast<float4*>(s.cold)[t] = make_float4(stat_ema(h, c_old.x, c_sum.x), stat_ema(h, c_old.y, c_sum.y),
                                                       stat_ema(h, c_old.z, c_sum.z), stat_ema(h, c_old.w, c_sum.w));
    if (t < a.rw) s.blk_vmax[t] = stat_ema(h, r_old, r_sum) * inv_total;
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);              // loop start-up state: nothing outstanding (see update_tile)
    __syncthreads();
    sync.staged();
    auto none = [] {};
    auto unit = [&](const RowF<BF16>& cur, int q, auto mid) {
        const int k = f.krow(q), il = f.row_g + k, j = q - k * f.nbk;
        float ct[4];
        load4(&s.cold[j * 128 + f.l * 4], ct);
        factor_unit<BF16>(h, tb, s, cur, f.off(q), il * kFlatBlocks + j, s.blk_vmax[il], ct, f.l, mid);
    };
    int q = 0;
    while (q + 2 < f.nq) {                                // rounds of three units, no exit in the middle
        unit(r0, q, [&] { r2 = fetch(q + 2); });
        unit(r1, q + 1, [&] { r0 = fetch(q + 3); });
        unit(r2, q + 2, [&] { r1 = fetch(q + 4); });
        q += 3;
    }
    if (q < f.nq) {
        unit(r0, q, none);
        if (q + 1 < f.nq) unit(r1, q + 1, none);
    }
    __syncthreads();
    for (int k = t; k < a.rw * kFlatBlocks; k += kThreads) {
        const int row = f.row_of(k / kFlatBlocks), j = k % kFlatBlocks;
        if (row < f.n && j < f.nbk) st<float>(tb.ms, row_offset(row, a.nb, uint32_t(f.cb0 + j)) * 4u, s.blk_scale[k]);
    }
}

// The same in plans: a group walks down the rows of one column block.  (Along the rows, as above, a step takes in one launch with fp32
// gradients, us, down / along: 354 M parameters 877 / 891, 380 M 975 / 1007, bert-like, 131 M, 338 / 354, llama-like, 75 M, 192 / 201, with bf16
// ones 717 / 717, 821 / 816, 280 / 279; by phases, 640 wide, 71 / 74, 896 80 / 82, 1152 205 / 208, 512 75 / 72.5, 1280 369 / 354.)
template <bool BF16, bool SAME_LAUNCH, class Sync>
__device__ __forceinline__ void factor_update_tile_down(const Tensor4& a, const Hyper& h, int wg, Lds& s, Sync& sync) {
    const TableRegs tables = request_tables();
    const Geo geo = geometry(a, wg);
    const TileBase tb = tile_base<BF16>(a, geo.row0, geo.n_rows);
    const RowWalk walk{a.rs, a.gy << a.rs};
    const int n = walk.rounds(geo.n_rows);
    const uint32_t lane4 = row_offset(geo.gyi << a.rs, a.cols, geo.col0) * 4u, pitch4 = uint32_t(a.cols) * 4u;
    const int slot0 = (geo.gyi << a.rs) * a.gx + geo.gxi;
    auto off = [&](int k) { return lane4 + uint32_t(walk.at(k)) * pitch4; };
    auto fetch = [&](int k) { return load_rowf<BF16>(tb, off(k)); };
    float ct[4], csum[4];
    RowF<BF16> r0 = fetch(0), r1 = fetch(1), r2;
    load4(a.c + geo.col0, ct);
    if (!sync.ready()) return;
    float inv_total;
    if constexpr (SAME_LAUNCH) {                 // through LDS, one agent-scope load per word
        for (int t = threadIdx.x; t < a.gx * 128; t += kThreads) s.col[t] = ld_ws<true>(a.c_new + int64_t(geo.strip) * a.gx * 128 + t);
        if (threadIdx.x == 0) s.cold[0] = factor_inv_total<true>(a, h);
        __syncthreads();
        inv_total = s.cold[0];
#pragma unroll
        for (int e = 0; e < 4; ++e) csum[e] = s.col[geo.gxi * 128 + geo.l * 4 + e];
    } else {
        load4(a.c_new + geo.col0, csum);
        inv_total = factor_inv_total(a, h);
    }
    // per row of the tile: the old block scales of m, and R_t[i] / sum R_t once instead of in every lane; zeros for rows
    // behind its end
    for (int t = threadIdx.x; t < a.rw * a.gx; t += kThreads) {
        const int il = t / a.gx, cbi = geo.strip * a.gx + t % a.gx;
        const bool in = il < geo.n_rows;
        s.blk_scale[t] = in ? tb.ms[row_offset(il, a.nb, uint32_t(cbi))] : 0.0f;
        s.blk_vmax[t] = in ? stat_ema(h, tb.r[il], ld_ws<SAME_LAUNCH>(tb.r_new + il)) * inv_total : 0.0f;
    }
    put_tables(s, tables);
    // every thread's statistics are here before the ticket is taken; and nothing is outstanding when the loop starts (see
    // update_tile)
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) ct[e] = stat_ema(h, ct[e], csum[e]);
    sync.staged();
    auto none = [] {};
    auto work = [&](const RowF<BF16>& cur, int k, auto mid) {
        const int slot = slot0 + walk.at(k) * a.gx;
        factor_unit<BF16>(h, tb, s, cur, off(k), slot, s.blk_vmax[slot], ct, geo.l, mid);
    };
    int k = 0;
    while (k + 2 < n) {
        work(r0, k, [&] { r2 = fetch(k + 2); });
        work(r1, k + 1, [&] { r0 = fetch(k + 3); });
        work(r2, k + 2, [&] { r1 = fetch(k + 4); });
        k += 3;
    }
    if (k < n) {
        work(r0, k, none);
        if (k + 1 < n) work(r1, k + 1, none);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < geo.n_rows * a.gx; t += kThreads) {
        const int il = t / a.gx, cbi = geo.strip * a.gx + t % a.gx;
        st<float>(tb.ms, row_offset(il, a.nb, uint32_t(cbi)) * 4u, s.blk_scale[t]);
    }
}

// stat[i] = stat_ema(stat[i], sum[i]); sum[i] = 0, by one workgroup (see move_statistics; reading the sums four at a time, which
// takes the statistics apart into strided words, is the slower way here)
template <bool SAME_LAUNCH = false>
__device__ __forceinline__ void ema_and_clear(const Hyper& h, float* stat, float* sum, int64_t n) {
    constexpr int kDepth = 8;
    for (int64_t base = threadIdx.x; base < n; base += int64_t(kThreads) * kDepth) {
        float o[kDepth], v[kDepth];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const int64_t i = base + int64_t(u) * kThreads;
            o[u] = i < n ? stat[i] : 0.0f;
            v[u] = i < n ? ld_ws<SAME_LAUNCH>(sum + i) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const int64_t i = base + int64_t(u) * kThreads;
            if (i < n) { stat[i] = stat_ema(h, o[u], v[u]); sum[i] = 0.0f; }
        }
    }
}

// The last workgroup of a tensor's update pass makes R_t, C_t the state and clears the workspace;
// every other workgroup has read the old statistics and the sums before it took its ticket.
__device__ __forceinline__ void factor_publish(const Tensor4& a, const Hyper& h) {
    ema_and_clear(h, a.r, a.r_new, a.rows);
    ema_and_clear(h, a.c, a.c_new, a.cols);
    if (threadIdx.x == 0) *a.counter = 0u;
    if (int(threadIdx.x) < a.tot_slots) {
        a.counter[tot_new_word(threadIdx.x)] = 0u;
        a.counter[tot_old_word(threadIdx.x)] = 0u;
    }
}

// Deterministic sums (Tensor4::det): between the statistics pass and the update pass two small kernels turn the
// per-tile partial sums into what the float atomics would have left in the workspace, in a fixed order.
// Layout of the partial sums behind a.vq (rows_pad, cols_pad = rows, cols rounded up to 64):
//   float[strips2][rows_pad]  a row's sum over the columns of one strip
//   float[tiles][cols_pad]    a column's sum over the rows of one tile
//   float[2 * row_wgs]        per 256 rows: the sum of their new row sums, and of their old row statistics
__device__ __forceinline__ const float* det_rowpart(const Tensor4& a) { return reinterpret_cast<const float*>(a.vq); }
__device__ __forceinline__ const float* det_colpart(const Tensor4& a) {
    return det_rowpart(a) + int64_t(a.strips2) * ((a.rows + 63) / 64 * 64);
}
__device__ __forceinline__ float* det_totpart(const Tensor4& a) {
    const int64_t tiles = (a.rows + a.rw2 - 1) / a.rw2;
    return const_cast<float*>(det_colpart(a)) + tiles * ((a.cols + 63) / 64 * 64);
}
// sum over the workgroup, the same value in every thread, combined in a fixed order
__device__ __forceinline__ float wg_sum_fixed(float v, float* s_part) {
    v = wave_sum(v);
    __syncthreads();                                   // s_part may still be read from a previous call
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = v;
    __syncthreads();
    return (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
}

// Workgroup `w` of a tensor's reduce step: 256 rows (w < ceil(rows / 256)) or 64 columns.
__device__ __forceinline__ void factor_reduce_one(const Tensor4& a, int w, float* s_part) {
    const int64_t rows_pad = (a.rows + 63) / 64 * 64, cols_pad = (a.cols + 63) / 64 * 64;
    const int row_wgs = int((a.rows + kThreads - 1) / kThreads);
    if (w < row_wgs) {                                 // uniform over the workgroup
        const float* rowpart = det_rowpart(a);
        const int64_t i = int64_t(w) * kThreads + threadIdx.x;
        float acc = 0.0f, old = 0.0f;
        if (i < a.rows) {
            for (int s0 = 0; s0 < a.strips2; s0 += 8) {        // eight loads in flight, added in index order
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = s0 + u < a.strips2 ? rowpart[int64_t(s0 + u) * rows_pad + i] : 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u];
            }
            a.r_new[i] = acc;
            old = a.r[i];
        }
        const float t_new = wg_sum_fixed(acc, s_part), t_old = wg_sum_fixed(old, s_part);
        if (threadIdx.x == 0) {
            float* tp = det_totpart(a);
            tp[2 * w] = t_new;
            tp[2 * w + 1] = t_old;
        }
    } else {
        // 64 columns per workgroup; a tall tensor has hundreds of row tiles, so four threads share a column: thread
        // (q, c) adds tiles q, q + 4, ... in order, eight loads in flight, and the four sums are added in order of q
        const float* colpart = det_colpart(a);
        const int c = threadIdx.x & 63, q = threadIdx.x >> 6;
        const int64_t j = int64_t(w - row_wgs) * 64 + c;
        const int tiles = int((a.rows + a.rw2 - 1) / a.rw2);
        float acc = 0.0f;
        if (j < a.cols)
            for (int t0 = q; t0 < tiles; t0 += 32) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = t0 + 4 * u < tiles ? colpart[int64_t(t0 + 4 * u) * cols_pad + j] : 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u];
            }
        __shared__ float s_col[kThreads];
        s_col[threadIdx.x] = acc;
        __syncthreads();
        if (q == 0 && j < a.cols) a.c_new[j] = (s_col[c] + s_col[64 + c]) + (s_col[128 + c] + s_col[192 + c]);
    }
}
// One workgroup per tensor, after the reduce step: the two totals (sum of this step's row sums, sum of the old row
// statistics) into slot 0, from the per-256-rows sums dealt to the threads in a fixed pattern.
__device__ __forceinline__ void factor_totals_one(const Tensor4& a, float* s_part) {
    const int row_wgs = int((a.rows + kThreads - 1) / kThreads);
    const float* tp = det_totpart(a);
    float t_new = 0.0f, t_old = 0.0f;
    for (int k = threadIdx.x; k < row_wgs; k += kThreads) {
        t_new += tp[2 * k];
        t_old += tp[2 * k + 1];
    }
    t_new = wg_sum_fixed(t_new, s_part);
    t_old = wg_sum_fixed(t_old, s_part);
    if (threadIdx.x == 0) {
        float* tot = reinterpret_cast<float*>(a.counter);
        tot[tot_new_word(0)] = t_new;
        tot[tot_old_word(0)] = t_old;
    }
}

// General path of the factorized form (any rows x cols): lane t owns flat elements [8t, 8t+8), row and
// column tracked per element.  The statistics pass works like the general first pass: a.rw consecutive chunks of
// 2048 elements per workgroup, sums combined in LDS (float atomics) by column (tensors of at most 2048
// columns) and by row relative to the workgroup's first row, one global atomic per touched column and row at
// the end; wider tensors add straight to global memory.
template <bool BF16>
__device__ __forceinline__ void factor_stats_general_tile(const Tensor4& a, int wg, int n_wg, Lds& s) {
    float* col_l = s.col;                  // [kGenColsLds] (col and cold)
    float* row_l = s.blk_scale;            // [kGenRowsLds] (blk_scale and blk_vmax)
    const int n_chunks = a.rw;
    const int64_t e_first = int64_t(wg) * n_chunks * kGenChunkElems;
    const int64_t e_end = e_first + int64_t(n_chunks) * kGenChunkElems < a.P ? e_first + int64_t(n_chunks) * kGenChunkElems : a.P;
    const int64_t i0 = e_first / a.cols;
    const int64_t n_rows_wg = (e_end - 1) / a.cols - i0 + 1;
    const bool cols_in_lds = a.cols <= kGenColsLds;
    const bool rows_in_lds = n_rows_wg <= kGenRowsLds;
    if (cols_in_lds)
        for (int t = threadIdx.x; t < int(a.cols); t += kThreads) col_l[t] = 0.0f;
    if (rows_in_lds)
        for (int t = threadIdx.x; t < int(n_rows_wg); t += kThreads) row_l[t] = 0.0f;
    __syncthreads();
    auto add_col = [&](int64_t j, float v) {
        if (cols_in_lds) (void)__hip_atomic_fetch_add(col_l + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else atomic_add_f32(a.c_new + j, v);
    };
    auto add_row = [&](int64_t i, float v) {
        if (rows_in_lds) (void)__hip_atomic_fetch_add(row_l + (i - i0), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else atomic_add_f32(a.r_new + i, v);
    };
    float part = 0.0f, old = 0.0f;
    const int lane = threadIdx.x & 63;
    for (int c = 0; c < n_chunks; ++c) {
        const int64_t t = (int64_t(wg) * n_chunks + c) * kThreads + threadIdx.x;
        const LaneIo io = lane_io(a.P, a.cols, t);
        float g[8];
        if (io.nv == 8) {
            load_grad8<BF16>(a.g, io.base, g);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = e < io.nv ? load_grad1<BF16>(a.g, io.base + e) : 0.0f;
        }
        int64_t i = io.i, j = io.j, run_row = io.i;
        float run = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (e < io.nv) {
                const float sq = g[e] * g[e];
                if (i != run_row) { add_row(run_row, run); run_row = i; run = 0.0f; }
                run += sq;
                part += sq;
                add_col(j, sq);
                if (++j == a.cols) { j = 0; ++i; }
            }
        }
        // the lane's last row usually is its neighbours' too: add up over the wave first (rows are contiguous
        // runs of lanes, so lane k ends up with the sum over lanes k.. of its row), one atomic per row and wave
        long long rr = io.nv ? (long long)run_row : -1ll - lane;
        float rsum = run;
        for (int d = 1; d < 64; d <<= 1) {
            const float os = __shfl_down(rsum, d);
            const long long orow = __shfl_down(rr, d);
            if (lane + d < 64 && orow == rr) rsum += os;
        }
        const long long prev = __shfl_up(rr, 1);
        if (io.nv && (lane == 0 || prev != rr)) add_row(rr, rsum);
    }
    for (int64_t i = int64_t(wg) * kThreads + threadIdx.x; i < a.rows; i += int64_t(n_wg) * kThreads) old += a.r[i];
    part = wave_sum(part);
    old = wave_sum(old);
    __shared__ float s_tot[2 * kThreads / 64];
    if (lane == 0) { s_tot[threadIdx.x >> 6] = part; s_tot[4 + (threadIdx.x >> 6)] = old; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float* tot = reinterpret_cast<float*>(a.counter);
        atomic_add_f32(tot + tot_new_word(wg & (a.tot_slots - 1)), (s_tot[0] + s_tot[1]) + (s_tot[2] + s_tot[3]));
        atomic_add_f32(tot + tot_old_word(wg & (a.tot_slots - 1)), (s_tot[4] + s_tot[5]) + (s_tot[6] + s_tot[7]));
    }
    if (cols_in_lds)
        for (int t = threadIdx.x; t < int(a.cols); t += kThreads) {
            const float v = col_l[t];
            if (v != 0.0f) atomic_add_f32(a.c_new + t, v);
        }
    if (rows_in_lds)
        for (int t = threadIdx.x; t < int(n_rows_wg); t += kThreads) {
            const float v = row_l[t];
            if (v != 0.0f) atomic_add_f32(a.r_new + i0 + t, v);
        }
}

template <bool BF16, bool SAME_LAUNCH = false>
__device__ __forceinline__ void factor_update_general_tile(const Tensor4& a, const Hyper& h, int wg, Lds& s, int64_t only = -1) {
    const int64_t t = int64_t(wg) * kThreads + threadIdx.x;
    const int64_t block = t >> 4;                       // uniform over the 16 lanes of a block
    if (block * 128 >= a.P || (only >= 0 && block != only)) return;    // only: this block alone
    const LaneIo io = lane_io(a.P, a.cols, t);
    float w[8], g[8];
    if (io.nv == 8) {
        load8(a.p + io.base, w);
        load_grad8<BF16>(a.g, io.base, g);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            w[e] = e < io.nv ? a.p[io.base + e] : 0.0f;
            g[e] = e < io.nv ? load_grad1<BF16>(a.g, io.base + e) : 0.0f;
        }
    }
    const uint32_t mq = load_codes(a.mq, io);
    const float s_old = a.ms[block];
    const float inv_total = factor_inv_total<SAME_LAUNCH>(a, h);
    float mt[8], amax = 0.0f;
    int64_t i = io.i, j = io.j;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (e < io.nv) {
            const float2 tt = s.deq[(mq >> (8 * (e >> 1))) & 255u];
            const float m_prev = ((e & 1) ? tt.y : tt.x) * s_old;
            mt[e] = moment_m(h, m_prev, g[e]);
            const float rn = stat_ema(h, a.r[i], ld_ws<SAME_LAUNCH>(a.r_new + i)) * inv_total;
            const float vt = rn * stat_ema(h, a.c[j], ld_ws<SAME_LAUNCH>(a.c_new + j));
            w[e] = param_update(h, w[e], mt[e], vt);
            amax = fmaxf(amax, fabsf(mt[e]));
            if (++j == a.cols) { j = 0; ++i; }
        } else {
            mt[e] = 0.0f;
        }
    }
    const float s_new = row16_allmax(amax);
    uint32_t mq_new = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (e < io.nv) mq_new |= quant_m_code(s.search, mt[e], s_new) << (4 * e);
    if (io.nv == 8) {
        float4* pp = reinterpret_cast<float4*>(a.p + io.base);
        pp[0] = make_float4(w[0], w[1], w[2], w[3]);
        pp[1] = make_float4(w[4], w[5], w[6], w[7]);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < io.nv) a.p[io.base + e] = w[e];
    }
    if (io.nv) store_codes(a.mq, io, mq_new);
    if ((threadIdx.x & 15) == 0) a.ms[block] = s_new;
}

// =====================================================================================================
// Uncompressed fp32 states (tensors that are not quantized): Alg. 3 with identity compression.
// One workgroup handles kElemsPerWg32 consecutive elements.
// =====================================================================================================

template <bool BF16>
__device__ __forceinline__ void adamw32_tile(float* p, const void* g, float* m, float* v, int64_t n,
                                             const Hyper& h, int wg) {
    const int64_t base = int64_t(wg) * kElemsPerWg32;
#pragma unroll 4
    for (int k = 0; k < kElemsPerWg32 / kThreads; ++k) {
        const int64_t idx = base + int64_t(k) * kThreads + threadIdx.x;
        if (idx < n) {
            const float gi = load_grad1<BF16>(g, idx);
            const float mt = moment_m(h, m[idx], gi);
            const float vt = moment_v(h, v[idx], gi);
            m[idx] = mt;
            v[idx] = vt;
            p[idx] = param_update(h, p[idx], mt, vt);
        }
    }
}

// SGD with momentum on an uncompressed fp32 buffer (tensors that are not quantized)
template <bool BF16>
__device__ __forceinline__ void sgdm32_tile(float* p, const void* g, float* m, int64_t n, const Hyper& h, int wg) {
    const int64_t base = int64_t(wg) * kElemsPerWg32;
#pragma unroll 4
    for (int k = 0; k < kElemsPerWg32 / kThreads; ++k) {
        const int64_t idx = base + int64_t(k) * kThreads + threadIdx.x;
        if (idx < n) {
            const float mt = moment_sgdm(h, m[idx], load_grad1<BF16>(g, idx));
            m[idx] = mt;
            p[idx] = param_sgdm(h, p[idx], mt);
        }
    }
}

}  // namespace lpmm

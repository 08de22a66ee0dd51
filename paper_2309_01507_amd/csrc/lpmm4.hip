// lpmm4.so -- C ABI and launch logic of the 4-bit AdamW step (declared in include/lpmm4.h).
// Host side only: argument checks, launch geometry, work lists, bias corrections.  All arithmetic of the
// method runs in the kernels of kernels.hpp, ragged.hpp, launch.hpp, flow.hpp, convert.hpp and ablation.hpp.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <limits>
#include <memory>
#include <mutex>
#include <unordered_map>
#include <numeric>
#include <vector>

#include "../../include/lpmm4.h"
#include "flow.hpp"
#include "convert.hpp"
#include "ablation.hpp"

namespace {

using namespace lpmm;

constexpr int kMaxDevices = 16;
static_assert(kCounterWords * 4 <= 8192, "counter block");
constexpr size_t kCounterBytes = 8192;  // tail of the workspace: ticket counters of the second pass, one cache line apart

struct DeviceCtx {
    bool ready = false;
    float* ws = nullptr;        // workspace: floats [0, cap) for r', c'; then counters
    int64_t cap_floats = 0;
    unsigned int* counter = nullptr;
    int n_cu = 256;
    unsigned char* scratch = nullptr;   // this device's copy of `scratch` below (its address on this device)
};

// Device memory of the library's own for lpmm_adamw4_step_noalloc: the ticket counters of the second pass, then the row
// and column maxima of the updated second moment.  Every GPU that loads the library holds one copy until the
// process ends.  In host code this name is only a handle for hipGetSymbolAddress; the address of a device's
// copy is DeviceCtx::scratch, looked up once per device by lpmm_adamw4_init.
constexpr int64_t kScratchFloats = LPMM_NOALLOC_MAX_ROWS_PLUS_COLS + 128;     // rows and cols each padded to 64
static __device__ __align__(256) unsigned char scratch[kCounterBytes + kScratchFloats * 4];

DeviceCtx g_ctx[kMaxDevices];
std::mutex g_mu;
thread_local int g_last_hip = 0;

// per-kernel timing (lpmm_profile_begin / _end)
struct Profile {
    bool on = false;
    int64_t max_calls = 0, calls = 0;
    std::vector<hipEvent_t> ev;    // 3 per recorded call
};
Profile g_prof;

hipEvent_t prof_event(int64_t call, int which) {
    return g_prof.ev[size_t(call) * 3 + which];
}

// host copies of the tables (also serve the host-only entry points)
struct HostTables {
    float de[kCodes], lin[kCodes], thr[kCodes - 1];
    float byte_decode[512];
    SearchEntry search[kBucketsPadded];
    bool ok;
    HostTables() {
        build_de_signed(de);
        build_linear(lin);
        build_thresholds(de, thr);
        ok = build_search(thr, search);
        build_byte_decode(de, byte_decode);
    }
};
const HostTables& host_tables() { static const HostTables t; return t; }

int hip_fail(hipError_t e) { g_last_hip = int(e); return LPMM_EHIP; }
#define LPMM_HIP(call) do { hipError_t e_ = (call); if (e_ != hipSuccess) return hip_fail(e_); } while (0)

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
bool finite_nonneg(float x) { return std::isfinite(x) && x >= 0.0f; }

int env_int(const char* name, int dflt) {
    const char* s = std::getenv(name);
    return (s && *s) ? std::atoi(s) : dflt;
}

int check_shape(const int64_t* shape, int64_t* rows, int64_t* cols) {
    if (!shape) return LPMM_EINVAL;
    if (shape[0] < 1 || shape[1] < 1) return LPMM_EINVAL;
    if (shape[0] > (int64_t(1) << 31) || shape[1] > (int64_t(1) << 31)) return LPMM_EINVAL;
    if (shape[0] * shape[1] > (int64_t(1) << 40)) return LPMM_EINVAL;
    *rows = shape[0];
    *cols = shape[1];
    return LPMM_OK;
}

int make_hyper(float lr, float beta1, float beta2, float eps, float wd, int64_t step, Hyper* h) {
    if (step < 1) return LPMM_EINVAL;
    if (!finite_nonneg(lr) || !finite_nonneg(eps) || !finite_nonneg(wd)) return LPMM_EINVAL;
    if (!(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f)) return LPMM_EINVAL;
    h->beta1 = beta1;
    h->beta2 = beta2;
    h->omb1 = 1.0f - beta1;
    h->omb2 = 1.0f - beta2;
    h->eps = eps;
    const double bc1 = 1.0 - std::pow(double(beta1), double(step));
    const double bc2 = 1.0 - std::pow(double(beta2), double(step));
    h->step_size = float(double(lr) / bc1);
    h->inv_sqrt_bc2 = float(1.0 / std::sqrt(bc2));
    h->lr_wd = float(double(lr) * double(wd));
    return LPMM_OK;
}

int current_ctx(DeviceCtx** out) {
    int dev = 0;
    LPMM_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices || !g_ctx[dev].ready) return LPMM_ENOTINIT;
    *out = &g_ctx[dev];
    return LPMM_OK;
}

bool is_rank1(int kind) { return kind == kQuantFast || kind == kQuantRagged || kind == kQuantGeneral; }
int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
int pad8(int64_t n) { return int(round_up(n, kXcds)); }

// workgroups (of n, for `elems` elements) that make up kSkewElems elements, at least 1; less than an eighth of them all
int skew_of(int64_t n, int64_t elems) {
    const int64_t skew = int64_t(double(n) * double(kSkewElems) / double(std::max<int64_t>(elems, 1)) + 0.5);
    return int(std::max<int64_t>(1, skew) % std::max<int64_t>(1, round_up(n, kXcds) / kXcds));
}
// The skew of a launch on its own: none below 2^23 elements, whose eighths two or fewer such distances fill, and none where it
// would bring the eighths' distance (of their parameters) closer to a multiple of 8 MiB instead of farther from one (SGDM with
// bf16 gradients, us with and without: 2^25 elements, 16 MiB apart, 58.2 and 65.3; 2^24, 8 MiB, 29.1 and 30.0; 30000001, 14.3 MiB,
// 58.8 and 54.0; 60000001, 28.6 MiB, 103.9 and 101.4; factorized 30000 x 1000 103.5 and 93.9).
int launch_skew(int64_t n, int64_t elems) {
    const double mib = 1024.0 * 1024.0, distance = double(elems) * 4.0 / kXcds;
    auto off = [&](double d) { const double r = std::fmod(d, 8.0 * mib); return std::min(r, 8.0 * mib - r); };
    return elems >= int64_t(1) << 23 && off(distance + double(kSkewElems) * 4.0) > off(distance) ? skew_of(n, elems) : 0;
}
void set_skew(Tensor4* t) {
    t->skew = launch_skew(t->n_wg, t->P);
    t->skew2 = launch_skew(t->n_wg2, t->P);
}

// log2 of the smallest S in {1, 2, 4, 8} for which S rows of `row_bytes` bytes are a multiple of 32 KiB; 0 if
// there is none.  Rows in flight side by side then lie 32 KiB apart, which is what the memory system serves
// fastest (measured).  S must divide `per_group`, the rows of a tile that one group (or wave) takes: only
// then does row(k) = g*S + k%S + (k/S)*groups*S enumerate every row of the tile exactly once.
int row_spacing_log2(int64_t row_bytes, int64_t rows_per_tile, int groups, const char* env) {
    if (rows_per_tile % groups) return 0;
    const int64_t per_group = rows_per_tile / groups;
    auto fits = [&](int l) { return l >= 0 && l <= 3 && (per_group % (int64_t(1) << l)) == 0; };
    const int forced = env_int(env, -1);
    if (forced >= 0) return fits(forced) ? forced : 0;
    for (int l = 0; fits(l); ++l)
        if (((row_bytes << l) % 32768) == 0) return l;
    return 0;
}

// Geometry of the rank-1 step on the fast path.
// First pass (maxima): strips of 256 columns by rw2 rows.  Second pass (update): strips of gx (at most 8) column blocks by rw
// rows.  n_cu > 0: a tensor stepped on its own, whose tiles are cut until the update has two workgroups per CU and the first pass
// one (two of shorter tiles end with twice the column atomics: 2048 x 1024 bf16 15.8 us per step with two, 15.1 with one; 768 x
// 3072 and 1024 x 1024 the same); else `shrink` halvings of a plan's tiles.
void rank1_fast_geometry(Tensor4* a, int n_cu, int64_t rw_hint, int64_t rw2_hint, int grad_bytes, int shrink = 0, int widest = kFlatBlocks) {
    a->nb = int(a->cols / LPMM_BLOCK);
    const int64_t cap = std::max<int64_t>((int64_t(1) << 29) / a->cols, kGroups);     // lane offsets inside a tile stay below 2^31 bytes
    const int n_strips = (a->nb + widest - 1) / widest;
    int gx = (a->nb + n_strips - 1) / n_strips;
    const int gx_env = env_int("LPMM_GX", 0);
    if (gx_env > 0) gx = std::min(gx_env, kFlatBlocks);
    // rows of a group: a power of two
    int per_log2 = 0;
    // two of them; one where a large matrix is stepped on its own (32000 x 4096 fp32 400 us, with two 405; 11008 x 4096 bf16 111.5
    // and 113.8; 4096 x 4096 bf16 46.9 and 46.2); narrow matrices as many as give a group 8 blocks (bf16, with one row and with 8 /
    // gx: 1000000 x 128 895 and 710 us, 131072 x 384 179 and 176, 262144 x 512 373 and 362; in plans, with two: 8 of 131072 x 128 419 and
    // 334, 289 tensors of a transformer of width 256 111 and 96)
    const int64_t rw_one = std::max(n_cu > 0 && a->P >= int64_t(1) << 25 ? kGroups : 2 * kGroups, kGroups * kFlatBlocks / gx);
    const int64_t rw_want = env_int("LPMM_RW", 0) > 0 ? env_int("LPMM_RW", 0) : rw_hint > 0 ? rw_hint : rw_one;
    const bool fixed = env_int("LPMM_RW", 0) > 0;
    while (per_log2 < 3 && (kGroups << (per_log2 + 1)) <= rw_want) ++per_log2;
    // Rows between the groups: 32 KiB of parameters where a power of two of rows is exactly that long (rows of 128 to 8192
    // elements, a power of two), unless a super-tile of 8 times as many would leave much of itself empty; else next to each
    // other.
    int rs = 0;
    const int forced = env_int("LPMM_RS", -1);
    if (forced >= 0) rs = std::min(forced, 6);
    else if (a->cols <= 8192 && (a->cols & (a->cols - 1)) == 0) {
        while ((a->cols << rs) < 8192) ++rs;
        per_log2 = std::min(per_log2, rs);
        if (round_up(a->rows, int64_t(kGroups) << rs) > a->rows + a->rows / 16) rs = 0;
    }
    while (rs > 0 && (int64_t(kGroups) << rs) * a->cols >= (int64_t(1) << 29)) --rs;
    while (per_log2 > 0 && (kGroups << per_log2) >= 2 * a->rows) --per_log2;
    auto tiles = [&] { return int64_t((a->nb + gx - 1) / gx) * (((a->rows + (kGroups << std::max(rs, per_log2)) - 1) >> (3 + std::max(rs, per_log2))) << (std::max(rs, per_log2) - per_log2)); };
    auto cut = [&] {
        if (per_log2 > 0 && !fixed) --per_log2;
        else if (gx > 1 && gx_env <= 0) gx = (gx + 1) / 2;
        else return false;
        return true;
    };
    while (per_log2 > 0 && ((int64_t(kGroups) << per_log2) * a->cols) >= (int64_t(1) << 29)) --per_log2;
    // two workgroups per CU, three while a group has more than 8 blocks (3072 x 3072 bf16 576 tiles 35.3 us, 1152 32.8; 4096 x 2048
    // 512 27.8, 1024 26.5)
    if (n_cu > 0) { while (tiles() < ((gx << per_log2) > kFlatBlocks || widest < kFlatBlocks ? 3 : 2) * int64_t(n_cu) && cut()) {} }
    for (int k = 0; k < shrink && cut(); ++k) {}
    a->gx = gx;
    a->gy = kGroups;
    a->rw = kGroups << per_log2;
    a->rs = std::max(rs, per_log2);
    a->strips = (a->nb + gx - 1) / gx;
    a->n_wg2 = int(tiles());
    a->strips2 = (a->nb + 1) / 2;
    int64_t rw2 = env_int("LPMM_RW2", 0);
    const bool fixed2 = rw2 > 0;
    if (rw2 <= 0) rw2 = rw2_hint > 0 ? rw2_hint : 128;
    rw2 = std::clamp<int64_t>(rw2, 1, std::min<int64_t>({cap, kMaxRowSlots, a->rows}));
    while (n_cu > 0 && !fixed2 && rw2 > 2 * kGroups && a->strips2 * ((a->rows + rw2 - 1) / rw2) < int64_t(n_cu)) rw2 = round_up(rw2 / 2, kGroups);
    // Tall narrow ones take more rows: every tile ends with an atomic per column, and atomics on one address follow each other (at
    // 128 rows and at 512: 262144 x 128 fp32 211 and 196 us, 1000000 x 128 bf16 711 and 633; 262144 x 256 fp32 287 and, at 256, 283).
    if (n_cu > 0 && !fixed2)
        while (rw2 < kMaxRowSlots && rw2 * a->cols < 1 << 16 && a->strips2 * (a->rows / (2 * rw2)) >= 2 * int64_t(n_cu)) rw2 *= 2;
    a->rw2 = int(rw2);
    a->n_wg = int(a->strips2 * ((a->rows + rw2 - 1) / rw2));
    a->rs2 = row_spacing_log2(a->cols * grad_bytes, rw2, kGroups, "LPMM_RS2");
}

// Tiling of a tensor whose second moment is block-wise: super-tiles of 8 x 64 blocks, each shared by
// 64 / rounds workgroups (rounds: a power of two, blocks that a group takes in a row), plus one workgroup
// for a partial last block.  rounds_hint > 0 fixes the rounds.
void b128_geometry(Tensor4* a, int n_cu, int64_t rounds_hint) {
    a->nb = int(a->P / LPMM_BLOCK);
    const int64_t supers = (a->nb + kB128Super - 1) / kB128Super;
    int64_t want = env_int("LPMM_B128_ROUNDS", 0);
    if (want <= 0) want = rounds_hint;
    int64_t rounds = 16;
    if (want > 0) {
        rounds = 1;
        while (rounds * 2 <= want && rounds * 2 <= kB128MaxRounds) rounds *= 2;      // round down to a power of two
    } else {
        while (rounds > 1 && supers * (kB128Stride / rounds) < 2 * int64_t(n_cu)) rounds >>= 1;
    }
    a->rw = int(rounds);
    a->n_wg2 = int(supers * (kB128Stride / rounds));
    a->n_wg = a->n_wg2 + ((a->P % LPMM_BLOCK) ? 1 : 0);
    a->gx = 1; a->gy = kGroups; a->strips = 1; a->strips2 = 1; a->rw2 = 1;
}

bool fast_eligible(int64_t cols, const float* v_colmax) {
    return (cols % LPMM_BLOCK) == 0 && cols < (int64_t(1) << 24) && aligned(v_colmax, 16) &&     // 24-bit row offsets
           !env_int("LPMM_FORCE_GENERAL", 0);
}

// general path: the second pass takes one chunk of 2048 elements per workgroup, the first several consecutive ones (the
// more, the fewer atomics leave the workgroup; few enough that the tensor alone still fills the chip)
void general_geometry(Tensor4* a, int n_cu) {
    const int64_t chunks = (a->P + kGenChunkElems - 1) / kGenChunkElems;
    int64_t per_wg = env_int("LPMM_GEN_CHUNKS", 0);
    if (per_wg <= 0) per_wg = chunks / (4 * int64_t(n_cu));
    if (per_wg < 1) per_wg = 1;
    if (per_wg > kGenMaxChunks) per_wg = kGenMaxChunks;
    a->rw = int(per_wg);
    a->n_wg = int((chunks + per_wg - 1) / per_wg);
    a->n_wg2 = int(chunks);
}

// Matrices that miss the fast path but have at least one block per row take the ragged tiles (general / ragged, us per
// step: 4096 x 4000 bf16 419 / 60, 30000 x 1000 fp32 291 / 153, 2304 x 576 fp32 31 / 24, 300 x 200 fp32 14.4 / 13.5).
// Narrower ones stay on the general path: there a block touches several rows, and combining an element's row maximum
// is most of the work.
bool ragged_eligible(int64_t rows, int64_t cols) {
    return cols >= LPMM_BLOCK && cols < (int64_t(1) << 24) && rows * cols <= (int64_t(1) << 37) &&
           !env_int("LPMM_FORCE_GENERAL", 0);
}

// Tiling of the ragged path (see ragged.hpp): the first pass takes statistics of strips of 256 columns by rw2 rows, the second
// updates whole blocks.
// Update, cols <= 1024: tiles of 8 to 128 consecutive blocks.  Wider: strips of equal width, at most 1024 columns, by `tall`
// rows; the rows are halved down to one per group and then the strips down to 256 columns.  Both shrink while the tensor
// would give the chip fewer than two workgroups per CU (n_cu = 0: `shrink` halvings instead, for plans, of 32 rows).
// Low tiles end more evenly and touch fewer distant rows at a time, but a workgroup stages its columns' statistics for fewer of them.
// A tensor on its own takes 8 rows (update alone, bf16 gradients, us at 8 / 16 / 32: 1024 x 50257 111 / 114 / 122, 12288 x 4099 102 / 103 /
// 112, 3000 x 3001 23.4 / 27.2 / 27.1, 2000 x 3001 17.2 / 17.6 / 17.6; factorized 1024 x 50257 109 / 113 / 121, 4096 x 4099 37.2 / 36.0 / 42.2);
// a plan by phases 16 from 3 * 2^22 parameters on (transformers of width 1088, 65 M, 148 / 138 / 150; 704, 15 M, 46 / 42 / 45;
// 448, 12 M, 33.6 / 33.3 / 32.4; factorized 1472, 528 M, 1266 / 1276 / 1330 a step, 1088, 204 M, 501 / 506 / 558, 448 43.2 / 43.4 / 41.7);
// one launch, where other tensors' tiles fill every gap, 32 (width 1088, 204 M, 647 / 608 / 583 a step; 704, fp32, 93 M, 306 / 297 / 292).
// Statistics: 256 rows (plans: 128), halved down to 64 while there are fewer than 11/4 workgroups per CU (24178 x 808 bf16, 64 and 128
// rows, 1512 and 756 tiles: 63.3 and 60.8 us per step; 50257 x 1088 bf16, 64, 128 and 256, the last 985 tiles: 161.9, 160.7, 158.6; but
// 6025 x 6840 bf16, 64 and 256, 648 tiles: 123.3 and 125.9; 8678 x 776 bf16, 64 and 128, 272 tiles: 30.0 and 31.6), then down to 8 while
// there are fewer than two; a multiple of 8.  Every tile ends with an atomic per column, and atomics on one address follow each other
// at about 18 ns, so a tall narrow matrix takes more rows to a tile than the filling of the chip alone would ask for: rows / rw2 of them against a quarter of rw2 rows, about 0.3 us each, one
// after the other in a wave balance at rw2 = sqrt(rows / 4) (factorized form of 2000 x 190 with fp32 gradients: 16.5 us per
// step, 29.8 without this).
constexpr int64_t kRagTall = 32, kRagPhase = 16, kRagAlone = kGroups, kRagPhaseParams = int64_t(3) << 22;
void ragged_geometry(Tensor4* a, int n_cu, int64_t tall, int shrink = 0) {
    a->nb = int(a->P / LPMM_BLOCK);
    const int tail = (a->P % LPMM_BLOCK) ? 1 : 0;
    constexpr int64_t kWide = kFlatBlocks * LPMM_BLOCK;
    if (a->cols <= kWide) {
        a->strips = 1;
        a->sw = int(a->cols);
        int64_t rw = std::max<int64_t>(128 >> shrink, kGroups);
        while (rw > kGroups && (a->nb + rw - 1) / rw < 2 * int64_t(n_cu)) rw /= 2;
        a->rw = int(rw);
        a->n_wg2 = int((a->nb + rw - 1) / rw) + tail;
    } else {
        int64_t rw = tall, sw = kWide, tiles;
        while (rw > kGroups && rw * a->cols > (int64_t(1) << 28)) rw /= 2;        // byte offsets inside a tile stay below 2^30
        rw = std::max<int64_t>(std::min<int64_t>(rw, kRagTall >> shrink), kGroups);
        for (;;) {
            const int64_t want = (a->cols + sw - 1) / sw;
            a->sw = int(round_up((a->cols + want - 1) / want, LPMM_BLOCK));
            a->strips = int((a->cols + a->sw - 1) / a->sw);
            tiles = a->strips * ((a->rows + rw - 1) / rw);
            if (tiles >= 2 * int64_t(n_cu)) break;
            if (rw > kGroups) rw /= 2;
            else if (sw > 256) sw /= 2;
            else break;
        }
        a->rw = int(rw);
        a->n_wg2 = int(tiles) + tail;
    }
    a->strips2 = int((a->cols + 255) / 256);
    const int64_t rows2 = class_rows(*a);
    int64_t rw2 = n_cu ? kMaxRw2 : std::max<int64_t>(128 >> shrink, kGroups);
    // a tile reads its own rows and the one behind them, and kNowhere lies beyond all of them
    auto fits = [&](int64_t r) { return (r + 1) * a->cols * 4 <= int64_t(kNowhere); };
    while (rw2 > kGroups && !fits(rw2)) rw2 /= 2;
    while (n_cu && rw2 > kGroups && a->strips2 * ((rows2 + rw2 - 1) / rw2) < (rw2 > 64 ? 11 : 8) * int64_t(n_cu) / 4) rw2 /= 2;
    while (rw2 < 64 && rw2 * rw2 < a->rows / 4 && fits(2 * rw2)) rw2 *= 2;
    if (const int forced = env_int("LPMM_RW2", 0); forced > 0) rw2 = std::clamp(forced / kGroups * kGroups, kGroups, kMaxRw2);
    while (rw2 > kGroups && !fits(rw2)) rw2 -= kGroups;
    a->rw2 = int(rw2);
    a->rs2 = 0;
    a->n_wg = int(a->strips2 * ((rows2 + rw2 - 1) / rw2));
    if (a->P & 7) a->n_wg += int((a->P - tail_begin(*a) + kLastRowElems - 1) / kLastRowElems);
}

// first or second pass of the rank-1 step on one tensor
template <bool BF16>
void launch_pass(int pass, const Tensor4& t, const Hyper& h, hipStream_t s) {
    const int n = pass == 1 ? t.n_wg : t.n_wg2;
    const dim3 grid(t.kind == kQuantGeneral ? n : pad8(n)), block(kThreads);
    if (t.kind == kQuantFast) {
        if (pass == 1) hipLaunchKernelGGL(maxima_fast<BF16>, grid, block, 0, s, t, h);
        else hipLaunchKernelGGL(update_fast<BF16>, grid, block, 0, s, t, h);
    } else if (t.kind == kQuantRagged) {
        if (pass == 1) hipLaunchKernelGGL(maxima_ragged_kernel<BF16>, grid, block, 0, s, t, h);
        else hipLaunchKernelGGL(update_ragged_kernel<BF16>, grid, block, 0, s, t, h);
    } else {
        if (pass == 1) hipLaunchKernelGGL(pass1_general<BF16>, grid, block, 0, s, t, h);
        else hipLaunchKernelGGL(pass2_general<BF16>, grid, block, 0, s, t, h);
    }
}

// tiling of one rank-1 tensor stepped on its own
void rank1_geometry(Tensor4* t, int n_cu, int grad_bytes) {
    if (fast_eligible(t->cols, t->c)) {
        t->kind = kQuantFast;
        rank1_fast_geometry(t, n_cu, 0, 0, grad_bytes);
    } else if (ragged_eligible(t->rows, t->cols)) {
        t->kind = kQuantRagged;
        ragged_geometry(t, n_cu, kRagAlone);
    } else {
        t->kind = kQuantGeneral;
        general_geometry(t, n_cu);
    }
}

template <bool BF16>
int launch_step(const Tensor4& t, const Hyper& h, hipStream_t s) {
    const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
    const int64_t call = g_prof.calls;
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
    launch_pass<BF16>(1, t, h, s);
    LPMM_HIP(hipGetLastError());
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
    launch_pass<BF16>(2, t, h, s);
    LPMM_HIP(hipGetLastError());
    if (rec) {
        LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
        g_prof.calls = call + 1;
    }
    return LPMM_OK;
}

int fill(void* dst, int64_t n, uint8_t value, int64_t last_index, uint8_t last, hipStream_t s);

// Where a single-tensor step keeps its new maxima and ticket counters: the workspace given to lpmm_adamw4_init
// (the default), the library's own device array (lpmm_adamw4_step_noalloc), or a workspace of the caller's
// (lpmm_adamw4_step_ws).
struct WorkspaceChoice {
    bool use_scratch = false;
    void* own = nullptr;
    size_t own_bytes = 0;
};

int step_impl(bool bf16, void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
              uint8_t* v_codes, float* v_rowmax, float* v_colmax, const int64_t* shape, float lr,
              float beta1, float beta2, float eps, float wd, int64_t step, void* stream,
              const WorkspaceChoice& wc = WorkspaceChoice()) {
    int64_t rows, cols;
    int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if (!param || !grad || !m_codes || !m_blockscale || !v_codes || !v_rowmax || !v_colmax)
        return LPMM_EINVAL;
    if (!aligned(param, 16) || !aligned(grad, 16) || !aligned(m_codes, 4) || !aligned(v_codes, 4) ||
        !aligned(m_blockscale, 4) || !aligned(v_rowmax, 4) || !aligned(v_colmax, 4))
        return LPMM_EINVAL;
    Hyper h;
    rc = make_hyper(lr, beta1, beta2, eps, wd, step, &h);
    if (rc) return rc;
    DeviceCtx* ctx;
    rc = current_ctx(&ctx);
    if (rc) return rc;
    const int64_t rows_pad = round_up(rows, 64), cols_pad = round_up(cols, 64);
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* ws = ctx->ws;
    unsigned int* counter = ctx->counter;
    if (wc.own) {
        // same layout as the workspace of lpmm_adamw4_init: the floats, then the counters in the last 8 KiB
        if (!aligned(wc.own, 256) || wc.own_bytes < kCounterBytes + 256 * sizeof(float)) return LPMM_EINVAL;
        const int64_t cap = int64_t((wc.own_bytes - kCounterBytes) / sizeof(float)) / 64 * 64;
        if (rows_pad + cols_pad > cap) return LPMM_EWORKSPACE;
        ws = static_cast<float*>(wc.own);
        counter = reinterpret_cast<unsigned int*>(static_cast<char*>(wc.own) + size_t(cap) * sizeof(float));
    } else if (wc.use_scratch) {
        if (!ctx->scratch) return LPMM_ENOTINIT;
        if (rows_pad + cols_pad > kScratchFloats) return LPMM_EWORKSPACE;
        // The array keeps what the last call on this device left.  A completed step leaves zeros, a step that
        // was cut short may not have: clear the part this call uses (counters, then the two runs of maxima)
        // with a kernel, so that the call stays capturable.
        rc = fill(ctx->scratch, int64_t(kCounterBytes) + (rows_pad + cols_pad) * int64_t(sizeof(float)), 0, -1, 0, s);
        if (rc) return rc;
        counter = reinterpret_cast<unsigned int*>(ctx->scratch);
        ws = reinterpret_cast<float*>(ctx->scratch + kCounterBytes);
    } else if (rows_pad + cols_pad > ctx->cap_floats) {
        return LPMM_EWORKSPACE;
    }

    Tensor4 t{};
    t.p = static_cast<float*>(param);
    t.g = grad;
    t.mq = reinterpret_cast<uint32_t*>(m_codes);
    t.ms = m_blockscale;
    t.vq = reinterpret_cast<uint32_t*>(v_codes);
    t.r = v_rowmax;
    t.c = v_colmax;
    t.r_new = ws;
    t.c_new = ws + rows_pad;
    t.counter = counter;
    t.rows = rows;
    t.cols = cols;
    t.P = rows * cols;
    rank1_geometry(&t, ctx->n_cu, bf16 ? 2 : 4);
    set_skew(&t);
    return bf16 ? launch_step<true>(t, h, s) : launch_step<false>(t, h, s);
}

int b128_step_impl(bool bf16, void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                   uint8_t* v_codes, float* v_blockscale, int64_t numel, float lr, float beta1, float beta2,
                   float eps, float wd, int64_t step, void* stream) {
    if (numel < 1 || numel > (int64_t(1) << 37)) return LPMM_EINVAL;
    if (!param || !grad || !m_codes || !m_blockscale || !v_codes || !v_blockscale) return LPMM_EINVAL;
    if (!aligned(param, 16) || !aligned(grad, 16) || !aligned(m_codes, 4) || !aligned(v_codes, 4) ||
        !aligned(m_blockscale, 4) || !aligned(v_blockscale, 4))
        return LPMM_EINVAL;
    Hyper h;
    int rc = make_hyper(lr, beta1, beta2, eps, wd, step, &h);
    if (rc) return rc;
    DeviceCtx* ctx;
    rc = current_ctx(&ctx);      // the lookup tables live in device memory filled by init
    if (rc) return rc;
    Tensor4 t{};
    t.p = static_cast<float*>(param);
    t.g = grad;
    t.mq = reinterpret_cast<uint32_t*>(m_codes);
    t.ms = m_blockscale;
    t.vq = reinterpret_cast<uint32_t*>(v_codes);
    t.r = v_blockscale;
    t.rows = 1;
    t.cols = numel;
    t.P = numel;
    t.kind = kQuantBlockV;
    b128_geometry(&t, ctx->n_cu, 0);
    set_skew(&t);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
    const int64_t call = g_prof.calls;
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
    if (bf16) hipLaunchKernelGGL(b128_kernel<true>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t, h);
    else hipLaunchKernelGGL(b128_kernel<false>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t, h);
    LPMM_HIP(hipGetLastError());
    if (rec) {
        LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
        LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
        g_prof.calls = call + 1;
    }
    return LPMM_OK;
}

// Workgroups for `items` items at `per_thread` per thread.  Kernels that are not grid-stride loops must
// get the full count (the default cap is the largest grid HIP takes; 2^40 elements stay far below it).
int grid_for(int64_t items, int64_t per_thread, int max_blocks = 0x7FFFFFFF) {
    const int64_t threads = (items + per_thread - 1) / per_thread;
    int64_t blocks = (threads + kThreads - 1) / kThreads;
    if (blocks < 1) blocks = 1;
    if (blocks > max_blocks) blocks = max_blocks;
    return int(blocks);
}

int make_sgdm_hyper(float lr, float momentum, Hyper* h) {
    if (!finite_nonneg(lr) || !(momentum >= 0.0f && momentum < 1.0f)) return LPMM_EINVAL;
    *h = Hyper{};
    h->beta1 = momentum;
    h->step_size = lr;
    return LPMM_OK;
}

int sgdm4_step_impl(bool bf16, void* param, const void* grad, uint8_t* m_codes, float* m_blockscale, int64_t numel,
                    float lr, float momentum, void* stream) {
    if (numel < 1 || numel > (int64_t(1) << 37)) return LPMM_EINVAL;
    if (!param || !grad || !m_codes || !m_blockscale) return LPMM_EINVAL;
    if (!aligned(param, 16) || !aligned(grad, 16) || !aligned(m_codes, 4) || !aligned(m_blockscale, 4))
        return LPMM_EINVAL;
    Hyper h;
    int rc = make_sgdm_hyper(lr, momentum, &h);
    if (rc) return rc;
    DeviceCtx* ctx;
    rc = current_ctx(&ctx);      // the lookup tables live in device memory filled by init
    if (rc) return rc;
    Tensor4 t{};
    t.p = static_cast<float*>(param);
    t.g = grad;
    t.mq = reinterpret_cast<uint32_t*>(m_codes);
    t.ms = m_blockscale;
    t.rows = 1;
    t.cols = numel;
    t.P = numel;
    b128_geometry(&t, ctx->n_cu, 0);
    set_skew(&t);
    t.kind = kSgdmBlock;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
    const int64_t call = g_prof.calls;
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
    if (bf16) hipLaunchKernelGGL(sgdm4_kernel<true>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t, h);
    else hipLaunchKernelGGL(sgdm4_kernel<false>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t, h);
    LPMM_HIP(hipGetLastError());
    if (rec) {
        LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
        LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
        g_prof.calls = call + 1;
    }
    return LPMM_OK;
}

// shape of a tensor with p >= 2 dimensions as the matrix the kernels see, plus its inner dimensions
int nd_shape(const int64_t* dims, int ndim, int64_t* rows, int64_t* cols, int64_t* ext, InnerDims* dm) {
    if (!dims || ndim < 2 || ndim > 1 + kMaxInnerDims) return LPMM_EINVAL;
    int64_t c = 1, e = 0;
    InnerDims d{};
    d.n = ndim - 1;
    for (int r = 1; r < ndim; ++r) {
        if (dims[r] < 1 || dims[r] > (int64_t(1) << 31)) return LPMM_EINVAL;
        if (c > (int64_t(1) << 31) / dims[r]) return LPMM_EINVAL;
        c *= dims[r];
        d.d[r - 1] = dims[r];
        d.first[r - 1] = e;
        e += dims[r];
    }
    const int64_t shape[2] = {dims[0], c};
    const int rc = check_shape(shape, rows, cols);
    if (rc) return rc;
    *ext = e;
    if (dm) *dm = d;
    return LPMM_OK;
}

int nd_step_impl(bool bf16, void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                 uint8_t* v_codes, float* v_row, float* v_col, const int64_t* dims, int ndim, float lr,
                 float beta1, float beta2, float eps, float wd, int64_t step, void* stream) {
    int64_t rows, cols, ext;
    InnerDims dm;
    int rc = nd_shape(dims, ndim, &rows, &cols, &ext, &dm);
    if (rc) return rc;
    if (!param || !grad || !m_codes || !m_blockscale || !v_codes || !v_row || !v_col) return LPMM_EINVAL;
    if (!aligned(param, 16) || !aligned(grad, 16) || !aligned(m_codes, 4) || !aligned(v_codes, 4) ||
        !aligned(m_blockscale, 4) || !aligned(v_row, 4) || !aligned(v_col, 4))
        return LPMM_EINVAL;
    Hyper h;
    rc = make_hyper(lr, beta1, beta2, eps, wd, step, &h);
    if (rc) return rc;
    DeviceCtx* ctx;
    rc = current_ctx(&ctx);
    if (rc) return rc;
    const int64_t rows_pad = round_up(rows, 64);
    if (rows_pad + round_up(cols + ext, 64) > ctx->cap_floats) return LPMM_EWORKSPACE;
    Tensor4 t{};
    t.p = static_cast<float*>(param);
    t.g = grad;
    t.mq = reinterpret_cast<uint32_t*>(m_codes);
    t.ms = m_blockscale;
    t.vq = reinterpret_cast<uint32_t*>(v_codes);
    t.r = v_row;
    t.c = v_col;                          // [cols] column scales, then [ext] the inner dimensions' statistics
    t.r_new = ctx->ws;
    t.c_new = ctx->ws + rows_pad;         // [cols] column maxima of v_t, then [ext] the new statistics
    t.c_extra = int(ext);
    t.counter = ctx->counter;
    t.rows = rows;
    t.cols = cols;
    t.P = rows * cols;
    rank1_geometry(&t, ctx->n_cu, bf16 ? 2 : 4);
    set_skew(&t);
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto pass = [&](int p) -> int {
        if (bf16) launch_pass<true>(p, t, h, s); else launch_pass<false>(p, t, h, s);
        LPMM_HIP(hipGetLastError());
        return LPMM_OK;
    };
    rc = pass(1);
    if (rc) return rc;
    hipLaunchKernelGGL(nd_reduce_kernel, dim3(int(ext)), dim3(kThreads), 0, s, t.c_new, t.c_new + cols, cols, dm);
    LPMM_HIP(hipGetLastError());
    hipLaunchKernelGGL(nd_expand_kernel, dim3(grid_for(cols, 1)), dim3(kThreads), 0, s, t.c_new + cols, t.c_new, cols, dm);
    LPMM_HIP(hipGetLastError());
    return pass(2);
}

// Tiling of a tensor with a factorized second moment: the statistics pass, the step's first ("A") launch, in strips of 256
// columns, the update pass, the second ("B") one, in column blocks.
// rows per tile of the statistics pass when its sums are reduced in a fixed order: fixed, because the size of the
// partial-sum buffer (part of the plan's memory) follows from it
constexpr int64_t kDetStatRows = 128;

// floats of partial sums of a rows x cols tensor with deterministic sums
int64_t det_partial_floats(int64_t rows, int64_t cols) {
    const int64_t strips2 = (cols / LPMM_BLOCK + 1) / 2, tiles = (rows + kDetStatRows - 1) / kDetStatRows;
    const int64_t row_wgs = (rows + kThreads - 1) / kThreads;
    return strips2 * round_up(rows, 64) + tiles * round_up(cols, 64) + round_up(2 * row_wgs, 64);
}

// Tiles of the factorized form's update in plans, see factor_update_tile_down: gx column blocks share a workgroup, gy = 8 / gx groups walk
// interleaved rows of the same column blocks.
void factor_down_geometry(Tensor4* a, int64_t rw, int64_t cap) {
    int gx = env_int("LPMM_GX", 1);
    if (gx < 1 || gx > kGroups || (gx & (gx - 1))) gx = 1;
    while (gx > 1 && (a->nb % gx) != 0) gx >>= 1;
    a->gx = gx;
    a->gy = kGroups / gx;
    a->strips = a->nb / gx;
    if (const int forced = env_int("LPMM_RW", 0); forced > 0) rw = forced;
    if (rw > cap) rw = cap;
    if (rw * gx > kMaxRowSlots) rw = kMaxRowSlots / gx;    // per-row results of a tile are staged in LDS
    rw = round_up(rw, a->gy);
    if (rw > cap || rw * gx > kMaxRowSlots) rw -= a->gy;
    if (rw > a->rows) rw = round_up(a->rows, a->gy);
    if (rw < a->gy) rw = a->gy;
    a->rw = int(rw);
    a->n_wg2 = int(a->strips * ((a->rows + rw - 1) / rw));
    a->rs = row_spacing_log2(a->cols * 4, rw, a->gy, "LPMM_RS");      // the parameters' rows
}

// The update of a factorized tensor on its own, in the rank-1 form's tiles: strips of 1 to 8 column blocks by 1 to 8 rows of a group.
// Rows of a power of two up to 8192 elements, which are taken 32 KiB apart: strips of 8 blocks from 2^25 elements on, below of 4, cut as the
// rank-1 form's (us at 4 and 8, bf16: 4096 x 4096 33.6, 33.5; 12288 x 4096 90.5, 89.3); also 8 in multiples of 2^23 elements, where the
// eighths of the tensor that the XCDs work on lie at multiples of 4 MiB (us, down the rows of one block as in plans, at 4, at 8, bf16: 4096 x 2048
// 27.2, 27.8, 26.2; 16384 x 1024 53.4, 54.1, 51.5; 12288 x 2048 63.8, 68.3, 62.5; at others 8 is the slower: 6144 x 2048 33.7, 33.5, 35.1).
// Others from 2^24 elements on: strips of 8 blocks, below 2^25 elements of 4, or the next width down to 3 or up to 8 that wastes at most a
// sixteenth (fp32, a step: 20000 x 640 in strips of 3 + 2 54.4, of 5 51.0; 30000 x 1152 of 5 + 4 111.1, of 3 107.4).
// The rest get the tiling with the least ceil(tiles / CU) * (units of a group + 0.8 for a workgroup's start), where a CU has 3.5 tiles done
// no later than fewer: in strips of 3 to 5 blocks cut until there are just over 3 tiles per CU they wait for the CUs that have a fourth, or
// for a strip of one block left over (us, down the rows, in those strips, and so, bf16: 3125 x 640 17.7, 18.6, 17.5; 4464 x 896 20.8, 21.7,
// 20.8; 9516 x 1664 46.6, 49.4, 47.4; fp32: 3125 x 1280 21.1, 21.9, 20.9; over 300 shapes 25 by more than 1.5 % slower than down the rows, and 9).
void factor_alone_geometry(Tensor4* a, int n_cu, int grad_bytes) {
    const bool apart = a->cols <= 8192 && (a->cols & (a->cols - 1)) == 0;
    if (apart || a->P >= int64_t(1) << 24) {
        const int most = a->P >= int64_t(1) << 25 || (apart && a->P % (int64_t(1) << 23) == 0) ? kFlatBlocks : kFlatBlocks / 2;
        auto even = [&](int w) { return round_up(a->nb, w) - a->nb <= a->nb / 16; };
        int widest = most;
        while (widest >= 3 && !even(widest)) --widest;
        if (widest < 3) for (widest = most + 1; widest <= kFlatBlocks && !even(widest);) ++widest;
        if (apart || widest <= kFlatBlocks) return rank1_fast_geometry(a, n_cu, 0, 0, grad_bytes, 0, std::min(widest, kFlatBlocks));
    }
    int widest = 1, rows = kGroups;
    int64_t least = std::numeric_limits<int64_t>::max();
    for (int gx = 1; gx <= std::min(a->nb, kFlatBlocks); ++gx)
        for (int per = 1; per <= 8; per *= 2) {
            const int64_t tiles = ((a->nb + gx - 1) / gx) * ((a->rows + kGroups * per - 1) / (kGroups * per));
            const int64_t cost = std::max<int64_t>(2 * ((tiles + n_cu - 1) / n_cu), 7) * (5 * gx * per + 4);
            if (cost < least) { least = cost; widest = gx; rows = kGroups * per; }
        }
    rank1_fast_geometry(a, 0, rows, 0, grad_bytes, 0, widest);
}

// rw_hint: rows of a plan's update tiles, 0 for a tensor on its own.  Statistics: strips of 256 columns by rw2 rows, a wave per row.
void factor_geometry(Tensor4* a, int n_cu, int64_t rw_hint, int64_t rw2_hint, int grad_bytes, bool fast,
                     int tot_slots, int shrink = 0, int64_t tall = kRagTall) {
    a->tot_slots = tot_slots;
    a->kind = fast ? kFactorFast : kFactorGeneral;
    if (fast) {
        const int64_t cap = (int64_t(1) << 29) / a->cols;         // lane offsets inside a tile stay below 2^31 bytes
        a->nb = int(a->cols / LPMM_BLOCK);
        if (rw_hint > 0) factor_down_geometry(a, rw_hint, cap);
        else factor_alone_geometry(a, n_cu, grad_bytes);
        a->strips2 = (a->nb + 1) / 2;
        int64_t rw2 = env_int("LPMM_RW2", 0);
        if (rw2 <= 0) rw2 = rw2_hint;
        if (rw2 <= 0) {
            rw2 = 64;
            while (rw2 > kWaves && a->strips2 * ((a->rows + rw2 - 1) / rw2) < 2 * int64_t(n_cu)) rw2 >>= 1;
        }
        rw2 = a->det ? std::min<int64_t>(kDetStatRows, a->rows) : std::max<int64_t>(std::min<int64_t>({rw2, cap, kMaxRw2, a->rows}), 1);
        a->rw2 = int(rw2);
        a->n_wg = int(a->strips2 * ((a->rows + rw2 - 1) / rw2));
        a->rs2 = row_spacing_log2(a->cols * grad_bytes, rw2, kWaves, "LPMM_RS2");     // that pass only reads the gradient
    } else if (!a->det && ragged_eligible(a->rows, a->cols)) {
        ragged_geometry(a, rw_hint == 0 ? n_cu : 0, tall, shrink);
        a->kind = kFactorRagged;
    } else {
        general_geometry(a, n_cu);          // statistics pass: several chunks per workgroup; update pass: one
        a->kind = kFactorGeneral;
    }
}

int factor_step_impl(bool bf16, void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                     float* v_row, float* v_col, const int64_t* shape, float lr, float beta1, float beta2,
                     float eps, float wd, int64_t step, void* stream) {
    int64_t rows, cols;
    int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if (!param || !grad || !m_codes || !m_blockscale || !v_row || !v_col) return LPMM_EINVAL;
    if (!aligned(param, 16) || !aligned(grad, 16) || !aligned(m_codes, 4) || !aligned(m_blockscale, 4) ||
        !aligned(v_row, 4) || !aligned(v_col, 4))
        return LPMM_EINVAL;
    Hyper h;
    rc = make_hyper(lr, beta1, beta2, eps, wd, step, &h);
    if (rc) return rc;
    DeviceCtx* ctx;
    rc = current_ctx(&ctx);
    if (rc) return rc;
    const int64_t rows_pad = round_up(rows, 64), cols_pad = round_up(cols, 64);
    if (rows_pad + cols_pad > ctx->cap_floats) return LPMM_EWORKSPACE;
    Tensor4 t{};
    t.p = static_cast<float*>(param);
    t.g = grad;
    t.mq = reinterpret_cast<uint32_t*>(m_codes);
    t.ms = m_blockscale;
    t.r = v_row;
    t.c = v_col;
    t.r_new = ctx->ws;
    t.c_new = ctx->ws + rows_pad;
    t.counter = ctx->counter;
    t.rows = rows;
    t.cols = cols;
    t.P = rows * cols;
    const bool fast = fast_eligible(cols, v_col);
    factor_geometry(&t, ctx->n_cu, 0, 0, bf16 ? 2 : 4, fast, kMaxTotSlots, 0, kRagAlone);
    set_skew(&t);
    const bool ragged = t.kind == kFactorRagged;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
    const int64_t call = g_prof.calls;
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
#define LPMM_LAUNCH_FACTOR(B)                                                                                      \
    if (ragged) hipLaunchKernelGGL(factor_stats_ragged_kernel<B>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t);    \
    else if (fast) hipLaunchKernelGGL(factor_stats_fast<B>, dim3(pad8(t.n_wg)), dim3(kThreads), 0, s, t);               \
    else hipLaunchKernelGGL(factor_stats_general<B>, dim3(t.n_wg), dim3(kThreads), 0, s, t);                       \
    LPMM_HIP(hipGetLastError());                                                                                   \
    if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 1), s));                                                     \
    if (ragged) hipLaunchKernelGGL(factor_update_ragged_kernel<B>, dim3(pad8(t.n_wg2)), dim3(kThreads), 0, s, t, h); \
    else if (fast) hipLaunchKernelGGL(factor_update_fast<B>, dim3(pad8(t.n_wg2)), dim3(kThreads), 0, s, t, h);          \
    else hipLaunchKernelGGL(factor_update_general<B>, dim3(t.n_wg2), dim3(kThreads), 0, s, t, h);                  \
    LPMM_HIP(hipGetLastError());
    if (bf16) { LPMM_LAUNCH_FACTOR(true) } else { LPMM_LAUNCH_FACTOR(false) }
#undef LPMM_LAUNCH_FACTOR
    if (rec) {
        LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
        g_prof.calls = call + 1;
    }
    return LPMM_OK;
}

// ---- multi-tensor plans ---------------------------------------------------------------------------

struct PhaseLaunch {
    Phase ph;
    int grid;        // both kinds in one launch
    int grid_a;      // A work alone
    int grid_b;      // B work alone
    bool b_general;     // every B tensor of `ph` is on the general tiles (a lighter kernel variant runs)
    // the B tensors on the general tiles where they have a launch of their own, behind that of the others
    Phase gen;
    int grid_gen;
    bool plain_b;       // B work alone in the kernel without the ragged and the general tiles
    bool a_has_rank1;   // some A tensor takes the first pass of the rank-1 path (else the lighter kernel variant runs)
    // tensors with more than two dimensions among the B tensors: two small kernels run before their second pass
    NdPhase nd;
    bool has_nd;
    // tensors with deterministic sums among the B tensors (factorized plans): two small kernels before their update pass
    DetPhase det;
    bool has_det;
};

struct PlanHost {
    std::vector<char> staging;          // host image of the device tables (kept for the async copy)
    std::vector<PhaseLaunch> phases;
    bool bf16 = false;
    bool factor = false;                // the plan's 2-dimensional tensors keep a factorized second moment
    bool sgdm = false;                  // a plan of SGD-with-momentum tensors (lpmm_sgdm4_step_multi)
    bool serial = false;                // LPMM_MULTI_STREAMS=0: every pass a launch of its own on the caller's stream
    bool plain = false;                 // rows of whole blocks only: launches by phases in the kernels without ragged and general tiles
    bool flow = false;                  // the whole step is one launch (flow.hpp)
    bool flow_any = false;              // ... with ragged matrices or rows shorter than 128 elements
    FlowArgs flow_args{};
    int64_t params = 0;                 // parameters of all tensors of the plan
    Hyper* d_hyper = nullptr;           // device slot inside the plan for the hyper-parameters of a captured step
    int device = 0;
    // LPMM_MULTI_STREAMS=2: second stream for second passes (same priority as any other stream), with its ordering events
    hipStream_t side = nullptr;
    hipStream_t side_a = nullptr;       // =3: first passes of odd phases, so that consecutive launches of first passes overlap their tails
    hipEvent_t ev_join_a = nullptr;
    std::vector<hipEvent_t> ev_a;       // ev_a[j]: phase j's A work is complete
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    ~PlanHost() {
        for (hipEvent_t e : ev_a) (void)hipEventDestroy(e);
        if (ev_fork) (void)hipEventDestroy(ev_fork);
        if (ev_join) (void)hipEventDestroy(ev_join);
        if (ev_join_a) (void)hipEventDestroy(ev_join_a);
        if (side) (void)hipStreamDestroy(side);
        if (side_a) (void)hipStreamDestroy(side_a);
    }
};

// shared ownership: a step copies the pointer out under the lock and keeps the plan's host record (streams, events)
// alive until it has enqueued its work, even if another thread releases the plan meanwhile
std::unordered_map<void*, std::shared_ptr<PlanHost>> g_plans;

struct PlanLayout {
    size_t off_tensors, off_dims, off_hyper, off_items, off_counters, off_deferred, off_floats, total;
    int64_t n_nd;
    int64_t cap_items, cap_deferred;    // room for the work list and the deferred tiles of a one-launch step
};

bool desc_shape_ok(const lpmm_tensor_desc& d) {
    int64_t shape[2] = {d.rows, d.cols}, r, c;
    return check_shape(shape, &r, &c) == LPMM_OK && (d.kind == LPMM_KIND_4BIT || d.kind == LPMM_KIND_FP32 ||
                                                     d.kind == LPMM_KIND_4BIT_B128 || d.kind == LPMM_KIND_4BIT_FACTOR ||
                                                     d.kind == LPMM_KIND_SGDM_4BIT || d.kind == LPMM_KIND_SGDM_FP32 ||
                                                     d.kind == LPMM_KIND_4BIT_ND);
}

// inner dimensions of tensor i of a plan: inner_dims holds kMaxInnerDims sizes per tensor, inner_ndim their count
// (0 for tensors that are not LPMM_KIND_4BIT_ND).  Fills dm and ext (the number of statistics of those dimensions).
bool plan_inner_dims(const lpmm_tensor_desc& d, int64_t i, const int64_t* inner_dims, const int32_t* inner_ndim,
                     InnerDims* dm, int64_t* ext) {
    if (!inner_dims || !inner_ndim) return false;
    const int k = inner_ndim[i];
    if (k < 1 || k > kMaxInnerDims) return false;
    int64_t dims[1 + kMaxInnerDims];
    dims[0] = d.rows;
    for (int r = 0; r < k; ++r) dims[1 + r] = inner_dims[i * kMaxInnerDims + r];
    int64_t rows, cols;
    if (nd_shape(dims, 1 + k, &rows, &cols, ext, dm) != LPMM_OK) return false;
    return cols == d.cols;
}

// Tiles of one tensor of a plan that is stepped in one launch; `total`: parameters of the plan.  A function of the shapes
// alone, because the size of the plan's memory follows from it.
//
// Statistics tiles are 256 rows tall (8 x llama-like layers of 4096, bf16 gradients 4.24 ms, GPT-2-medium set 792 us, BERT-base
// 302; 128 rows: 4.28, 811, 305; 512: 4.56, 836, 333): every tile ends with an atomic per row and column.  Update tiles hold
// two rows per group (one row: 4.33 ms and 821 us; four: 4.62 ms, since rows of 4096 cannot be 32 KiB apart then).
// Sets of less than 2^25 parameters (they are here for the sake of their convolutions) take shorter tiles to have enough of
// them: a vision set of 7.4 million parameters takes 45, 38, 42 and 44 us with statistics tiles of 128, 32, 16 rows and of 64
// rows.
constexpr int64_t kFlowMinParams = int64_t(1) << 25;
// Parameters of second passes between the first pass of a tensor and its own second pass: what is in flight on the chip at a
// time, and a little more, so that a second pass finds its first one complete.  In one piece, 12, 16, 20 and 24 million:
// GPT-2-medium set 793, 790, 794 and 796 us, BERT-base 324, 303, 307 and 303, 8 llama layers 4.31, 4.24, 4.24 and 4.25 ms.
// Spread, 12, 16, 20 and 24: factorized GPT-2-medium 790, 711, 717 and 717, factorized BERT-base 313, 284, 276 and 275, 8
// factorized llama layers 3.94, 3.82, 3.82 and 3.84 ms, rank-1 with rows of 1472 1344, 1297, 1272 and 1273.  Factorized plans with
// rows shorter than 128 elements, 10, 14 and 20 million: adapters 64 x 4096 and 4096 x 64 181, 183 and 188 us, 30000 x 96 beside 1024
// x 4096 389, 369 and 380.
constexpr double kFlowLead = 16.0 * (1 << 20), kFlowLeadSpread = 20.0 * (1 << 20), kFlowLeadNarrow = 14.0 * (1 << 20);
// Unused dynamic LDS of the one launch: four workgroups on a CU instead of five (rank-1, plain rows: GPT-2-medium 799 us without,
// 790 with), five instead of six (factorized: 747 us at six, 711 at five, 730 at four).  More of them only move the point up to
// which the list has been handed out further ahead of the first passes that the second ones wait for.
constexpr unsigned kFlowLdsPad = 16000, kFlowLdsPadFactor = 8000;
// From here to kFlowMinParams the updates of tensors with more than two dimensions come after all others (see build_flow), and
// ragged tiles are twice as tall: vision sets, fp32, us before both / with the order alone / with both: 9.8 M parameters 48.1 /
// 51.0 / 49.1, 12.8 M 53.5 / 51.5 / 51.8, 16 M 71.7 / 67.6 / 64.3, 24 M 101.6 / 93.7 / 90.6, 31 M 125 / 118.6 / 113.1; 7.4 M
// 37.0 / 40.2.
constexpr int64_t kFlowNdLate = kFlowMinParams / 8 * 3;
void flow_geometry(Tensor4* t, int desc_kind, bool aligned_c, int64_t total, int grad_bytes) {
    constexpr int kCus = 256;
    const int shrink = total >= kFlowMinParams ? 0 : total >= kFlowMinParams / 4 ? 1 : 2;
    const int rw = 16, rw2 = shrink ? 32 : 256;
    if (desc_kind == LPMM_KIND_FP32) {
        t->kind = kFp32State;
        t->n_wg = t->n_wg2 = int((t->P + kElemsPerWg32 - 1) / kElemsPerWg32);
    } else if (desc_kind == LPMM_KIND_4BIT_B128) {
        t->kind = kQuantBlockV;
        b128_geometry(t, kCus, 8 >> shrink);
    } else if (desc_kind == LPMM_KIND_4BIT_FACTOR) {
        factor_geometry(t, kCus, 64 >> shrink, rw2, grad_bytes, (t->cols % LPMM_BLOCK) == 0 && aligned_c &&
                        fast_eligible(t->cols, nullptr), 1, shrink);
    } else if (aligned_c && fast_eligible(t->cols, nullptr)) {
        t->kind = kQuantFast;
        rank1_fast_geometry(t, 0, rw, rw2, grad_bytes, shrink ? 1 : 0);
    } else if (ragged_eligible(t->rows, t->cols)) {
        t->kind = kQuantRagged;
        ragged_geometry(t, 0, kRagTall, !shrink ? 0 : total >= kFlowNdLate ? 2 : 3);
    } else {
        t->kind = kQuantGeneral;
        general_geometry(t, kCus);
    }
}
bool flow_kind_second(int kind) { return is_rank1(kind) || kind == kFactorFast || kind == kFactorGeneral; }

// Whether a list of tensors is stepped in one launch.  It can be where some tensor has two passes, no sums are wanted in a
// fixed order, and the statistics of tensors with more than two dimensions are few enough for one workgroup.  It is where
// that is faster (us, phases / one launch; where two pairs are given, fp32 and bf16 gradients):
// - Sets of 2^25 parameters or more (transformers with an embedding: 35 M 116 / 110, 99 / 98; 66 M 220 / 189, 180 / 162;
//   131 M 408 / 363, 328 / 297; 498 M 1708 / 1418, 1356 / 1187; measured when the first pass still was the update).  Below, there is little in flight to hide a tensor's wait
//   between the passes behind (8.4 M 43 / 49, 39 / 47; 16.7 M 63 / 61, 55 / 56; 24 M 82 / 82, 72 / 75; factorized 29 M 88 /
//   89, 74 / 80).
// - Not sets of which one tensor is most, whose second pass finds little to run beside: rank-1 up to three quarters,
//   factorized up to a quarter.  Alone, one launch is the slower way (8192 x 4096 106 / 129, 91 / 109; 50257 x 1024 171 / 173,
//   144 / 149); beside other tensors it is by now the faster one on both sides of these lines (rank-1, 99 M, 0.75 of it in
//   one tensor 326 / 303, 259 / 243; 0.87 323 / 307, 259 / 251; factorized, 106 M, 0.28 296 / 277, 229 / 224), but the lines
//   were drawn when the waiting workgroups slowed the counting ones, and no call has been moved across them since.
// - Not sets of nothing but two to eight matrices of about one size, up to 2^25 parameters each: 2 of 4096 x 4096 105 / 128,
//   90 / 110; 4 of them 197 / 224, 164 / 187; 8 398 / 412, 313 / 341; 12 604 / 596, 482 / 493; 4 of 8192 x 8192 817 / 768,
//   654 / 623.  Launches by phases lose time to unequal tiles, and these have none.
// - Not sets of which the general tiles (rows shorter than 128) are most: in one kernel with the others they have fewer waves
//   in flight.  Rank-1 below half of the parameters (30000 x 96 beside 1024 x 4096, bf16 and fp32 gradients: 0.25 233
//   / 203, 297 / 218; 0.4 376 / 298, 470 / 327; 0.58 282 / 277, 336 / 275; 0.85 401 / 456, 436 / 470; all 352 / 460, 363 /
//   469), factorized up to half (adapters 64 x 4096 and 4096 x 64: 406 / 354, 394 / 337; all narrow 486 / 571, 478 / 572).
// - Sets with tensors of more than two dimensions, which by phases take four dependent launches, also below 2^25 parameters
//   (a vision set of 7.4 M 61 / 41, 56 / 38; 8 of 128 x 128 x 3 x 3 34 / 24; 2048 x 4096 and one of 64 x 64 x 3 x 3 46 /
//   42), unless it is one large tensor alone (1024 x 1024 x 3 x 3 67 / 73; 640 x 640 x 3 x 3 44 / 44).  From 2^25 on the
//   lines above hold for them, too, where such tensors are few (two of 4096 x 4096 and one of 64 x 64 x 3 x 3 117 / 124,
//   102 / 110; with one of 512 x 512 x 3 x 3, a fifteenth of the parameters, 130 / 128, 113 / 113; with four 162 / 146, 137
//   / 127).
bool flow_possible(const lpmm_tensor_desc* descs, int64_t n, const int64_t* inner_dims, const int32_t* inner_ndim) {
    if (env_int("LPMM_FLOW", 1) == 0 || std::getenv("LPMM_MULTI_STREAMS") || std::getenv("LPMM_PHASE_MPARAMS")) return false;
    bool factor = false;
    int64_t total = 0, largest = 0, n_second = 0, general = 0, nd = 0;
    for (int64_t i = 0; i < n; ++i) {
        const lpmm_tensor_desc& d = descs[i];
        const int64_t P = d.rows * d.cols;
        if (d.kind == LPMM_KIND_SGDM_4BIT || d.kind == LPMM_KIND_SGDM_FP32 || (d.flags & LPMM_FLAG_DETERMINISTIC)) return false;
        if (P > (int64_t(1) << 37)) return false;
        // ragged factorized tensors: their update in the same kernel takes 125 registers in place of 74, three or four
        // waves on a SIMD in place of six
        if (d.kind == LPMM_KIND_4BIT_FACTOR && !fast_eligible(d.cols, nullptr) && ragged_eligible(d.rows, d.cols)) return false;
        if (d.kind == LPMM_KIND_4BIT_ND) {
            InnerDims dm;
            int64_t ext;
            if (!plan_inner_dims(d, i, inner_dims, inner_ndim, &dm, &ext)) return false;
            if (d.cols > kFlowNdCols || ext > kFlowNdStats) return false;
            nd += P;
        }
        total += P;
        largest = std::max(largest, P);
        if (d.kind == LPMM_KIND_4BIT || d.kind == LPMM_KIND_4BIT_ND || d.kind == LPMM_KIND_4BIT_FACTOR) {
            ++n_second;
            factor = factor || d.kind == LPMM_KIND_4BIT_FACTOR;
            if (!fast_eligible(d.cols, nullptr) && !ragged_eligible(d.rows, d.cols)) general += P;
        }
    }
    if (n_second == 0) return false;
    const int64_t least = env_int("LPMM_FLOW_MIN", int(kFlowMinParams));
    if (least == 0) return true;
    if (factor ? general > total / 2 : general >= total / 2) return false;
    if (nd > 0 && (total < least || nd >= total / 32)) return n_second > 1 || total <= (int64_t(1) << 22);
    if (total < least || largest > (factor ? total / 4 : total / 4 * 3)) return false;
    int64_t n_large = 0, large = 0;                  // tensors of about the largest one's size
    for (int64_t i = 0; i < n; ++i) {
        const int64_t P = descs[i].rows * descs[i].cols;
        if (P >= largest / 2) { ++n_large; large += P; }
    }
    return factor || n_large > 8 || large < total / 16 * 15 || largest > (int64_t(1) << 25);
}

// one_launch: with room for a work list, if the plan is one for a single launch
bool plan_layout(const lpmm_tensor_desc* descs, int64_t n, const int64_t* inner_dims, const int32_t* inner_ndim,
                 PlanLayout* L, bool one_launch = true) {
    if (!descs || n < 1 || n > (1 << 20)) return false;
    int64_t floats = 0, n_nd = 0;
    bool rank1 = false, factor = false;
    for (int64_t i = 0; i < n; ++i) {
        if (!desc_shape_ok(descs[i])) return false;
        if (descs[i].kind == LPMM_KIND_4BIT || descs[i].kind == LPMM_KIND_4BIT_FACTOR)
            floats += round_up(descs[i].rows, 64) + round_up(descs[i].cols, 64);
        if (descs[i].kind == LPMM_KIND_4BIT_FACTOR && (descs[i].flags & LPMM_FLAG_DETERMINISTIC))
            floats += det_partial_floats(descs[i].rows, descs[i].cols);
        if (descs[i].kind == LPMM_KIND_4BIT_ND) {
            InnerDims dm;
            int64_t ext;
            if (!plan_inner_dims(descs[i], i, inner_dims, inner_ndim, &dm, &ext)) return false;
            floats += round_up(descs[i].rows, 64) + round_up(descs[i].cols + ext, 64);
            ++n_nd;
        }
        if (descs[i].kind == LPMM_KIND_4BIT || descs[i].kind == LPMM_KIND_4BIT_ND) rank1 = true;
        if (descs[i].kind == LPMM_KIND_4BIT_FACTOR) factor = true;
    }
    L->n_nd = n_nd;
    int64_t n_sgdm = 0;
    for (int64_t i = 0; i < n; ++i)
        if (descs[i].kind == LPMM_KIND_SGDM_4BIT || descs[i].kind == LPMM_KIND_SGDM_FP32) ++n_sgdm;
    if (rank1 && factor) return false;       // two different optimizers: one plan holds one of them
    if (n_sgdm != 0 && n_sgdm != n) return false;
    L->cap_items = L->cap_deferred = 0;
    if (one_launch && flow_possible(descs, n, inner_dims, inner_ndim)) {
        int64_t total = 0;
        for (int64_t i = 0; i < n; ++i) total += descs[i].rows * descs[i].cols;
        for (int64_t i = 0; i < n; ++i) {
            Tensor4 t{};
            t.rows = descs[i].rows; t.cols = descs[i].cols; t.P = t.rows * t.cols;
            flow_geometry(&t, descs[i].kind, true, total, 4);
            L->cap_items += t.n_wg + 16;                          // lists are padded to multiples of 8
            if (flow_kind_second(t.kind)) {
                L->cap_items += t.n_wg2 + 16;
                L->cap_deferred += t.n_wg2;
            }
        }
        if (L->cap_items > (int64_t(1) << 28)) L->cap_items = L->cap_deferred = 0;
    }
    size_t off = 0;
    L->off_tensors = off;   off += size_t(round_up(n * int64_t(sizeof(Tensor4)), 256));
    L->off_dims = off;      off += size_t(round_up(n_nd * int64_t(sizeof(InnerDims)), 256));
    L->off_hyper = off;     off += 256;                       // hyper-parameters of a captured step
    L->off_items = off;     off += size_t(round_up(L->cap_items * int64_t(sizeof(FlowItem)), 256));
    L->off_counters = off;  off += size_t(n) * kCounterWords * sizeof(unsigned int);
    L->off_deferred = off;  off += size_t(round_up(L->cap_deferred * int64_t(sizeof(int)), 256));
    L->off_floats = off;    off += size_t(floats) * sizeof(float);
    L->total = size_t(round_up(int64_t(off), 256));
    return true;
}

// The work list of a plan that is stepped in one launch, and the tensors' tiles for it; leaves the plan to the
// launches by groups if the list does not fit (column maxima that turned out misaligned give more tiles).
//
// The second passes follow each other; the first pass of a tensor is put kFlowLead parameters of second passes in front of its own
// one.  It reads little (the gradient and, rank-1, the second moment's codes), nothing else of the step stays in the memory-side
// cache (parameters pass it by: non-temporal), and so the second pass reads what the first one read from there.  In place of that
// the first passes were the updates before, with the codes' second pass 2^23 parameters behind: 7B-shaped set 16.5 ms, now 14.9;
// GPT-2-medium 843 us, now 790; with all first passes ahead of all second ones 949.
// The first pass of a tensor on the plain tiles goes in one piece, others spread over the length of the tensor (spread / in one
// piece: factorized GPT-2-medium 711 / 738 us; rank-1 with rows of 1472 1272 / 1297; but rank-1 with rows of 4096 4.29 / 4.24
// ms).  Tensors with more than two dimensions come first, the widest ones ahead: one workgroup turns their maxima into
// statistics between the passes, and that takes longest where there are many columns.  Then the largest ones: what is left at
// the end is the second pass of the smallest.  In sets of kFlowNdLate to kFlowMinParams parameters, whose first passes all
// together are short beside that one workgroup, the others' updates run meanwhile and those of such tensors follow at the end.
//
// Workgroups are laid out eight at a time: ids are dealt to the 8 XCDs in turn, and the eight of a row take their tiles from eight
// equal contiguous parts of the pass (skewed as in logical_wg), so that neighbouring tiles, which share cache lines, stay on one
// XCD.
void build_flow(const lpmm_tensor_desc* descs, int64_t n, const PlanLayout& L, char* dplan, int gbytes, PlanHost* host,
                Tensor4* tens) {
    int64_t total = 0, n_def = 0;
    for (int64_t i = 0; i < n; ++i) total += tens[i].P;
    std::vector<Tensor4> flow(tens, tens + n);
    for (int64_t i = 0; i < n; ++i) {
        Tensor4& t = flow[i];
        flow_geometry(&t, descs[i].kind, aligned(descs[i].v_colmax, 16), total, gbytes);
        if (t.kind == kFactorRagged) return;
        if (flow_kind_second(t.kind)) {
            t.deferred = int(n_def);
            n_def += t.n_wg2;
        }
    }
    if (n_def > L.cap_deferred) return;
    struct Row { FlowItem it[kXcds]; };
    // tiles of one pass in rows of 8; a pass of fewer than 8 workgroups shares the row of the ones before it
    struct Open { std::vector<Row>* rows = nullptr; int fill = 0; };
    auto add = [](std::vector<Row>& rows, int what, int n_wg, int64_t elems, Open* open) {
        if (n_wg < kXcds) {
            for (int w = 0; w < n_wg; ++w) {
                if (open->fill == 0) {
                    rows.push_back(Row{{{-1, 0}, {-1, 0}, {-1, 0}, {-1, 0}, {-1, 0}, {-1, 0}, {-1, 0}, {-1, 0}}});
                    open->rows = &rows;
                }
                open->rows->back().it[open->fill] = FlowItem{what, w};
                open->fill = (open->fill + 1) % kXcds;
            }
            return;
        }
        open->fill = 0;
        const int part = (n_wg + kXcds - 1) / kXcds, skew = skew_of(n_wg, elems);
        for (int k = 0; k < part; ++k) {
            Row r{};
            for (int x = 0; x < kXcds; ++x) {
                const int w = x * part + (k + x * skew) % part;            // as in logical_wg
                r.it[x] = w < n_wg ? FlowItem{what, w} : FlowItem{-1, 0};
            }
            rows.push_back(r);
        }
    };
    std::vector<int64_t> order(static_cast<size_t>(n));
    std::iota(order.begin(), order.end(), int64_t(0));
    std::stable_sort(order.begin(), order.end(), [&](int64_t x, int64_t y) {
        const bool nx = descs[x].kind == LPMM_KIND_4BIT_ND, ny = descs[y].kind == LPMM_KIND_4BIT_ND;
        return nx != ny ? nx : nx ? flow[x].cols > flow[y].cols : flow[x].P > flow[y].P;
    });
    struct Passes { std::vector<Row> first, second; };
    std::vector<Passes> passes(order.size());
    Open open1, open2;
    for (size_t k = 0; k < order.size(); ++k) {
        const Tensor4& t = flow[order[k]];
        const int id = int(order[k]);
        if (flow_kind_second(t.kind)) {
            add(passes[k].first, id, t.n_wg, t.P, &open1);
            add(passes[k].second, id | kFlowSecond, t.n_wg2, t.P, &open2);
        } else {
            add(passes[k].second, id, t.n_wg, t.P, &open2);
        }
    }
    struct Timed { double time; Row row; };
    std::vector<Timed> first, second;
    auto is_nd = [&](size_t k) { return descs[order[k]].kind == LPMM_KIND_4BIT_ND; };
    const bool late = total >= kFlowNdLate && total < kFlowMinParams;
    std::vector<size_t> updates(order.size());              // the tensors in the order of their second passes
    std::iota(updates.begin(), updates.end(), size_t(0));
    if (late) std::stable_partition(updates.begin(), updates.end(), [&](size_t k) { return !is_nd(k); });
    const bool narrow_factor = std::any_of(flow.begin(), flow.end(), [](const Tensor4& t) { return t.kind == kFactorGeneral; });
    double begin = 0.0;
    for (const size_t k : updates) {
        const Tensor4& t = flow[order[k]];
        const double length = double(t.P), n1 = double(passes[k].first.size()), n2 = double(passes[k].second.size());
        const double spread = t.kind == kQuantFast ? 0.0 : length, lead = spread == 0.0 ? kFlowLead : narrow_factor ? kFlowLeadNarrow : kFlowLeadSpread;
        for (const Row& r : passes[k].first) {
            const double at = begin - lead - spread * (1.0 - double(&r - passes[k].first.data()) / n1);
            first.push_back(Timed{late && is_nd(k) ? std::numeric_limits<double>::lowest() : at, r});    // ahead of everything
        }
        for (const Row& r : passes[k].second) second.push_back(Timed{begin + length * double(&r - passes[k].second.data()) / n2, r});
        begin += length;
    }
    std::stable_sort(first.begin(), first.end(), [](const Timed& x, const Timed& y) { return x.time < y.time; });
    std::vector<Row> rows;
    size_t a = 0, b = 0;
    while (a < first.size() || b < second.size()) {
        const bool take_first = b == second.size() || (a < first.size() && first[a].time <= second[b].time);
        rows.push_back(take_first ? first[a++].row : second[b++].row);
    }
    const int64_t n_items = int64_t(rows.size()) * kXcds;
    if (n_items > L.cap_items) return;
    FlowItem* items = reinterpret_cast<FlowItem*>(host->staging.data() + L.off_items);
    for (const Row& r : rows)
        for (int x = 0; x < kXcds; ++x) *items++ = r.it[x];
    std::copy(flow.begin(), flow.end(), tens);
    host->flow = true;
    for (const Tensor4& t : flow) host->flow_any = host->flow_any || t.kind == kQuantRagged || t.kind == kQuantGeneral || t.kind == kFactorGeneral;
    host->flow_args.tensors = reinterpret_cast<const Tensor4Table*>(dplan + L.off_tensors);
    host->flow_args.items = reinterpret_cast<const FlowItem*>(dplan + L.off_items);
    host->flow_args.dims = reinterpret_cast<const InnerDims*>(dplan + L.off_dims);
    host->flow_args.deferred = reinterpret_cast<int*>(dplan + L.off_deferred);
    host->flow_args.n_items = int(n_items);
    host->flow_args.spin_limit = env_int("LPMM_FLOW_SPIN", 20000);
}

int fill(void* dst, int64_t n, uint8_t value, int64_t last_index, uint8_t last, hipStream_t s) {
    if (n <= 0) return LPMM_OK;
    hipLaunchKernelGGL(fill_bytes_kernel, dim3(grid_for(n, 16, 4096)), dim3(kThreads), 0, s,
                       static_cast<uint8_t*>(dst), n, value, last_index, last);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

int rank_grid(int64_t elems, int units) { return grid_for(elems, units * kCvtUnitElems / kThreads); }

// Row and column maxima of q.x_in into q.sa / q.sb.  Tiles of 64 rows, halved down to 16 while the tensor would give the chip fewer
// than two workgroups per CU (11008 x 4096: 16, 32 and 64 rows 35.5 us, 128, the last of whose workgroups run alone, 45; 4096 x 4096 at
// 32, 64 and 128 14.4, 13.8, 19; 200 x 16000 at 16, 32 and 64 5.8, 5.6, 6.4).  Tall ones take more: atomics on one column's maximum
// follow each other (3000 x 1001 at 16, 32 and 64 8.2, 6.3, 6.5 us; 16384 x 80 at 64, 128 and 256 7.8, 6.5, 7.6).
// So do those on one row's maximum, one per strip at about 12 ns, and a matrix of some hundred rows or fewer has nothing to do meanwhile:
// workgroups take runs of strips, about 1 us each, so that the two balance at the root of the strips (rows of up to 82000 elements take
// single ones).  With all rows in one tile the columns' maxima are complete, and stored.  (With codes, us: strips of 1024 columns with atomics for
// both, of 256, and so: 1 x 1000003 22.5, 55, 22.7; 1 x 10000000 151, 483, 100; 4 x 4000000 84, 216, 69; 8 x 4000000 105, 235, 92; 16 x
// 1000000 57, 72, 42; 20 x 100000 14.5, 14.6, 12.0; 70 x 500000 67, 83, 65; 128 x 500000 107, 119, 101; 1024 x 100000 158, 158, 156.)
int launch_maxima(const QuantArgs& q, int n_cu, hipStream_t s) {
    hipLaunchKernelGGL(clear_two_kernel, dim3(grid_for(q.rows + q.cols, 4, 1024)), dim3(kThreads), 0, s, q.sa, q.rows, q.sb,
                       q.cols);
    LPMM_HIP(hipGetLastError());
    int tx = 4;
    while (tx < 32 && tx * kMaxCols < q.cols) tx *= 2;
    const int64_t strip = tx * kMaxCols;
    MaxTiling t;
    t.strips = int((q.cols + strip - 1) / strip);
    auto tiles = [&](int64_t per) { return t.strips * ((q.rows + per - 1) / per); };
    int64_t per = 64;
    while (per > 16 && tiles(per) < 2 * int64_t(n_cu)) per /= 2;
    while (per < kMaxTileRows && per * per < q.rows / 3) per *= 2;
    t.rows_per_wg = int(per);
    t.run = std::max(1, int(std::sqrt(double(t.strips)) / 9.0));
    t.groups = (t.strips + t.run - 1) / t.run;
    t.whole = q.rows <= per;
    const dim3 grid(unsigned(t.groups * ((q.rows + per - 1) / per))), block(kThreads);
    const bool single = q.cols < kMaxCols || (tx <= 8 && q.cols % 4 != 0);
    if (single && tx == 4) hipLaunchKernelGGL((quant_v_max_kernel<4, true>), grid, block, 0, s, q, t);
    else if (single) hipLaunchKernelGGL((quant_v_max_kernel<8, true>), grid, block, 0, s, q, t);
    else if (tx == 4) hipLaunchKernelGGL((quant_v_max_kernel<4, false>), grid, block, 0, s, q, t);
    else if (tx == 8) hipLaunchKernelGGL((quant_v_max_kernel<8, false>), grid, block, 0, s, q, t);
    else if (tx == 16) hipLaunchKernelGGL((quant_v_max_kernel<16, false>), grid, block, 0, s, q, t);
    else hipLaunchKernelGGL((quant_v_max_kernel<32, false>), grid, block, 0, s, q, t);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

}  // namespace

extern "C" {

const char* lpmm_strerror(int code) {
    switch (code) {
        case LPMM_OK: return "ok";
        case LPMM_EINVAL: return "invalid argument (null or misaligned pointer, bad shape, step < 1, or bad hyper-parameter)";
        case LPMM_ENOTINIT: return "lpmm_adamw4_init has not been called for the current device";
        case LPMM_EHIP: return "a HIP call failed (see lpmm_last_hip_error)";
        case LPMM_EWORKSPACE: return "workspace too small for this tensor (rows + cols)";
        default: return "unknown lpmm error code";
    }
}

int lpmm_last_hip_error(void) { return g_last_hip; }

int lpmm_table(int which, float* out) {
    if (!out || (which != 0 && which != 1)) return LPMM_EINVAL;
    const HostTables& t = host_tables();
    for (int i = 0; i < kCodes; ++i) out[i] = which == 0 ? t.de[i] : t.lin[i];
    return LPMM_OK;
}

int lpmm_host_nearest_codes(int which, const float* n, int64_t count, uint8_t* out) {
    if (!n || !out || count < 0 || (which != 0 && which != 1)) return LPMM_EINVAL;
    const HostTables& t = host_tables();
    if (!t.ok) return LPMM_EINVAL;
    for (int64_t i = 0; i < count; ++i) {
        if (which == 0) {
            out[i] = uint8_t(search_code(t.search, n[i]));
        } else {
            const float f = std::ceil(std::fmaf(16.0f, n[i], -1.5f));
            out[i] = uint8_t(std::fmin(std::fmax(f, 0.0f), 15.0f));
        }
    }
    return LPMM_OK;
}

size_t lpmm_adamw4_workspace_bytes(int64_t max_rows_plus_cols) {
    if (max_rows_plus_cols < 2) max_rows_plus_cols = 2;
    // rows and cols are each rounded up to 64 floats inside the workspace
    return size_t(round_up(max_rows_plus_cols, 64) + 128) * sizeof(float) + kCounterBytes;
}

int lpmm_adamw4_init(int device, void* workspace, size_t workspace_bytes, void* stream) {
    if (device < 0 || device >= kMaxDevices) return LPMM_EINVAL;
    if (!workspace || !aligned(workspace, 256) || workspace_bytes < kCounterBytes + 256 * sizeof(float))
        return LPMM_EINVAL;
    const HostTables& t = host_tables();
    if (!t.ok) return LPMM_EINVAL;
    std::lock_guard<std::mutex> lock(g_mu);
    int prev = 0;
    LPMM_HIP(hipGetDevice(&prev));
    LPMM_HIP(hipSetDevice(device));
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyToSymbolAsync(HIP_SYMBOL(d_byte_decode), t.byte_decode, sizeof(t.byte_decode), 0,
                                          hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyToSymbolAsync(HIP_SYMBOL(d_search), t.search, sizeof(t.search), 0,
                                   hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemsetAsync(workspace, 0, workspace_bytes, s);
    int n_cu = 256;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device);
    // where this device keeps its copy of the library's own scratch array (`device` is current here)
    unsigned char* scratch_ptr = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(reinterpret_cast<void**>(&scratch_ptr), HIP_SYMBOL(scratch));
    (void)hipSetDevice(prev);
    if (e != hipSuccess) return hip_fail(e);
    DeviceCtx& c = g_ctx[device];
    c.scratch = scratch_ptr;
    c.ws = static_cast<float*>(workspace);
    c.cap_floats = int64_t((workspace_bytes - kCounterBytes) / sizeof(float)) / 64 * 64;
    c.counter = reinterpret_cast<unsigned int*>(static_cast<char*>(workspace) + size_t(c.cap_floats) * sizeof(float));
    c.n_cu = n_cu > 0 ? n_cu : 256;
    c.ready = true;
    return LPMM_OK;
}

int lpmm_adamw4_state_sizes(const int64_t shape[2], size_t sizes[5]) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if (!sizes) return LPMM_EINVAL;
    const int64_t P = rows * cols;
    sizes[0] = size_t((P + 1) / 2);
    sizes[1] = size_t((P + LPMM_BLOCK - 1) / LPMM_BLOCK) * sizeof(float);
    sizes[2] = size_t((P + 1) / 2);
    sizes[3] = size_t(rows) * sizeof(float);
    sizes[4] = size_t(cols) * sizeof(float);
    return LPMM_OK;
}

int lpmm_adamw4_state_zero(uint8_t* m_codes, float* m_blockscale, uint8_t* v_codes, float* v_rowmax,
                           float* v_colmax, const int64_t shape[2], void* stream) {
    size_t sz[5];
    const int rc = lpmm_adamw4_state_sizes(shape, sz);
    if (rc) return rc;
    if (!m_codes || !m_blockscale || !v_codes || !v_rowmax || !v_colmax) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t P = shape[0] * shape[1];
    // code 7 is the rank of 0.0 in the DE map; an odd tail leaves its unused high nibble 0
    int r = fill(m_codes, int64_t(sz[0]), 0x77, (P & 1) ? int64_t(sz[0]) - 1 : -1, 0x07, s);
    if (!r) r = fill(m_blockscale, int64_t(sz[1]), 0, -1, 0, s);
    if (!r) r = fill(v_codes, int64_t(sz[2]), 0, -1, 0, s);
    if (!r) r = fill(v_rowmax, int64_t(sz[3]), 0, -1, 0, s);
    if (!r) r = fill(v_colmax, int64_t(sz[4]), 0, -1, 0, s);
    return r;
}

int lpmm_adamw4_step(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                     uint8_t* v_codes, float* v_rowmax, float* v_colmax, const int64_t shape[2],
                     float lr, float beta1, float beta2, float eps, float weight_decay, int64_t step,
                     void* stream) {
    return step_impl(false, param, grad, m_codes, m_blockscale, v_codes, v_rowmax, v_colmax, shape, lr,
                     beta1, beta2, eps, weight_decay, step, stream);
}

int lpmm_adamw4_step_bf16g(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                           uint8_t* v_codes, float* v_rowmax, float* v_colmax, const int64_t shape[2],
                           float lr, float beta1, float beta2, float eps, float weight_decay,
                           int64_t step, void* stream) {
    return step_impl(true, param, grad, m_codes, m_blockscale, v_codes, v_rowmax, v_colmax, shape, lr,
                     beta1, beta2, eps, weight_decay, step, stream);
}

int lpmm_adamw4_step_noalloc(void* param, const void* grad, int grad_dtype, uint8_t* m_codes, float* m_blockscale,
                             uint8_t* v_codes, float* v_rowmax, float* v_colmax, const int64_t shape[2],
                             float lr, float beta1, float beta2, float eps, float weight_decay, int64_t step,
                             void* stream) {
    if (grad_dtype != LPMM_GRAD_F32 && grad_dtype != LPMM_GRAD_BF16) return LPMM_EINVAL;
    return step_impl(grad_dtype == LPMM_GRAD_BF16, param, grad, m_codes, m_blockscale, v_codes, v_rowmax, v_colmax,
                     shape, lr, beta1, beta2, eps, weight_decay, step, stream, WorkspaceChoice{true, nullptr, 0});
}

int lpmm_adamw4_step_ws(void* param, const void* grad, int grad_dtype, uint8_t* m_codes, float* m_blockscale,
                        uint8_t* v_codes, float* v_rowmax, float* v_colmax, const int64_t shape[2], float lr,
                        float beta1, float beta2, float eps, float weight_decay, int64_t step, void* workspace,
                        size_t workspace_bytes, void* stream) {
    if (grad_dtype != LPMM_GRAD_F32 && grad_dtype != LPMM_GRAD_BF16) return LPMM_EINVAL;
    if (!workspace) return LPMM_EINVAL;
    return step_impl(grad_dtype == LPMM_GRAD_BF16, param, grad, m_codes, m_blockscale, v_codes, v_rowmax, v_colmax,
                     shape, lr, beta1, beta2, eps, weight_decay, step, stream,
                     WorkspaceChoice{false, workspace, workspace_bytes});
}

int lpmm_adamw4_b128_state_sizes(int64_t numel, size_t sizes[4]) {
    if (numel < 1 || numel > (int64_t(1) << 37) || !sizes) return LPMM_EINVAL;
    sizes[0] = sizes[2] = size_t((numel + 1) / 2);
    sizes[1] = sizes[3] = size_t((numel + LPMM_BLOCK - 1) / LPMM_BLOCK) * sizeof(float);
    return LPMM_OK;
}

int lpmm_adamw4_b128_state_zero(uint8_t* m_codes, float* m_blockscale, uint8_t* v_codes, float* v_blockscale,
                                int64_t numel, void* stream) {
    size_t sz[4];
    const int rc = lpmm_adamw4_b128_state_sizes(numel, sz);
    if (rc) return rc;
    if (!m_codes || !m_blockscale || !v_codes || !v_blockscale) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int r = fill(m_codes, int64_t(sz[0]), 0x77, (numel & 1) ? int64_t(sz[0]) - 1 : -1, 0x07, s);
    if (!r) r = fill(m_blockscale, int64_t(sz[1]), 0, -1, 0, s);
    if (!r) r = fill(v_codes, int64_t(sz[2]), 0, -1, 0, s);
    if (!r) r = fill(v_blockscale, int64_t(sz[3]), 0, -1, 0, s);
    return r;
}

int lpmm_adamw4_b128_step(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                          uint8_t* v_codes, float* v_blockscale, int64_t numel, float lr, float beta1,
                          float beta2, float eps, float weight_decay, int64_t step, void* stream) {
    return b128_step_impl(false, param, grad, m_codes, m_blockscale, v_codes, v_blockscale, numel, lr, beta1,
                          beta2, eps, weight_decay, step, stream);
}

int lpmm_adamw4_b128_step_bf16g(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                                uint8_t* v_codes, float* v_blockscale, int64_t numel, float lr, float beta1,
                                float beta2, float eps, float weight_decay, int64_t step, void* stream) {
    return b128_step_impl(true, param, grad, m_codes, m_blockscale, v_codes, v_blockscale, numel, lr, beta1,
                          beta2, eps, weight_decay, step, stream);
}

int lpmm_adamw4_factor_state_sizes(const int64_t shape[2], size_t sizes[4]) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if (!sizes) return LPMM_EINVAL;
    const int64_t P = rows * cols;
    sizes[0] = size_t((P + 1) / 2);
    sizes[1] = size_t((P + LPMM_BLOCK - 1) / LPMM_BLOCK) * sizeof(float);
    sizes[2] = size_t(rows) * sizeof(float);
    sizes[3] = size_t(cols) * sizeof(float);
    return LPMM_OK;
}

int lpmm_adamw4_factor_state_zero(uint8_t* m_codes, float* m_blockscale, float* v_row, float* v_col,
                                  const int64_t shape[2], void* stream) {
    size_t sz[4];
    const int rc = lpmm_adamw4_factor_state_sizes(shape, sz);
    if (rc) return rc;
    if (!m_codes || !m_blockscale || !v_row || !v_col) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t P = shape[0] * shape[1];
    int r = fill(m_codes, int64_t(sz[0]), 0x77, (P & 1) ? int64_t(sz[0]) - 1 : -1, 0x07, s);
    if (!r) r = fill(m_blockscale, int64_t(sz[1]), 0, -1, 0, s);
    if (!r) r = fill(v_row, int64_t(sz[2]), 0, -1, 0, s);
    if (!r) r = fill(v_col, int64_t(sz[3]), 0, -1, 0, s);
    return r;
}

int lpmm_adamw4_factor_step(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale, float* v_row,
                            float* v_col, const int64_t shape[2], float lr, float beta1, float beta2, float eps,
                            float weight_decay, int64_t step, void* stream) {
    return factor_step_impl(false, param, grad, m_codes, m_blockscale, v_row, v_col, shape, lr, beta1, beta2,
                            eps, weight_decay, step, stream);
}

int lpmm_adamw4_factor_step_bf16g(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                                  float* v_row, float* v_col, const int64_t shape[2], float lr, float beta1,
                                  float beta2, float eps, float weight_decay, int64_t step, void* stream) {
    return factor_step_impl(true, param, grad, m_codes, m_blockscale, v_row, v_col, shape, lr, beta1, beta2,
                            eps, weight_decay, step, stream);
}

int lpmm_adamw4_nd_state_sizes(const int64_t* dims, int ndim, size_t sizes[5]) {
    int64_t rows, cols, ext;
    const int rc = nd_shape(dims, ndim, &rows, &cols, &ext, nullptr);
    if (rc) return rc;
    if (!sizes) return LPMM_EINVAL;
    const int64_t P = rows * cols;
    sizes[0] = size_t((P + 1) / 2);
    sizes[1] = size_t((P + LPMM_BLOCK - 1) / LPMM_BLOCK) * sizeof(float);
    sizes[2] = size_t((P + 1) / 2);
    sizes[3] = size_t(rows) * sizeof(float);
    sizes[4] = size_t(cols + ext) * sizeof(float);
    return LPMM_OK;
}

int lpmm_adamw4_nd_state_zero(uint8_t* m_codes, float* m_blockscale, uint8_t* v_codes, float* v_row, float* v_col,
                              const int64_t* dims, int ndim, void* stream) {
    size_t sz[5];
    const int rc = lpmm_adamw4_nd_state_sizes(dims, ndim, sz);
    if (rc) return rc;
    if (!m_codes || !m_blockscale || !v_codes || !v_row || !v_col) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int64_t P = 1;
    for (int r = 0; r < ndim; ++r) P *= dims[r];
    int r = fill(m_codes, int64_t(sz[0]), 0x77, (P & 1) ? int64_t(sz[0]) - 1 : -1, 0x07, s);
    if (!r) r = fill(m_blockscale, int64_t(sz[1]), 0, -1, 0, s);
    if (!r) r = fill(v_codes, int64_t(sz[2]), 0, -1, 0, s);
    if (!r) r = fill(v_row, int64_t(sz[3]), 0, -1, 0, s);
    if (!r) r = fill(v_col, int64_t(sz[4]), 0, -1, 0, s);
    return r;
}

int lpmm_adamw4_nd_step(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale, uint8_t* v_codes,
                        float* v_row, float* v_col, const int64_t* dims, int ndim, float lr, float beta1,
                        float beta2, float eps, float weight_decay, int64_t step, void* stream) {
    return nd_step_impl(false, param, grad, m_codes, m_blockscale, v_codes, v_row, v_col, dims, ndim, lr, beta1,
                        beta2, eps, weight_decay, step, stream);
}

int lpmm_adamw4_nd_step_bf16g(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale,
                              uint8_t* v_codes, float* v_row, float* v_col, const int64_t* dims, int ndim,
                              float lr, float beta1, float beta2, float eps, float weight_decay, int64_t step,
                              void* stream) {
    return nd_step_impl(true, param, grad, m_codes, m_blockscale, v_codes, v_row, v_col, dims, ndim, lr, beta1,
                        beta2, eps, weight_decay, step, stream);
}

int lpmm_sgdm4_state_sizes(int64_t numel, size_t sizes[2]) {
    if (numel < 1 || numel > (int64_t(1) << 37) || !sizes) return LPMM_EINVAL;
    sizes[0] = size_t((numel + 1) / 2);
    sizes[1] = size_t((numel + LPMM_BLOCK - 1) / LPMM_BLOCK) * sizeof(float);
    return LPMM_OK;
}

int lpmm_sgdm4_state_zero(uint8_t* m_codes, float* m_blockscale, int64_t numel, void* stream) {
    size_t sz[2];
    const int rc = lpmm_sgdm4_state_sizes(numel, sz);
    if (rc) return rc;
    if (!m_codes || !m_blockscale) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int r = fill(m_codes, int64_t(sz[0]), 0x77, (numel & 1) ? int64_t(sz[0]) - 1 : -1, 0x07, s);
    if (!r) r = fill(m_blockscale, int64_t(sz[1]), 0, -1, 0, s);
    return r;
}

int lpmm_sgdm4_step(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale, int64_t numel, float lr,
                    float momentum, void* stream) {
    return sgdm4_step_impl(false, param, grad, m_codes, m_blockscale, numel, lr, momentum, stream);
}

int lpmm_sgdm4_step_bf16g(void* param, const void* grad, uint8_t* m_codes, float* m_blockscale, int64_t numel,
                          float lr, float momentum, void* stream) {
    return sgdm4_step_impl(true, param, grad, m_codes, m_blockscale, numel, lr, momentum, stream);
}

int lpmm_sgdm32_step(void* param, const void* grad, float* m, int64_t numel, int grad_dtype, float lr,
                     float momentum, void* stream) {
    if (!param || !grad || !m || numel < 1) return LPMM_EINVAL;
    if (grad_dtype != LPMM_GRAD_F32 && grad_dtype != LPMM_GRAD_BF16) return LPMM_EINVAL;
    if (!aligned(param, 4) || !aligned(m, 4) || !aligned(grad, grad_dtype == LPMM_GRAD_F32 ? 4 : 2)) return LPMM_EINVAL;
    Hyper h;
    const int rc = make_sgdm_hyper(lr, momentum, &h);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int grid = int((numel + kElemsPerWg32 - 1) / kElemsPerWg32);
    if (grad_dtype == LPMM_GRAD_BF16)
        hipLaunchKernelGGL(sgdm32_kernel<true>, dim3(grid), dim3(kThreads), 0, s, static_cast<float*>(param), grad, m, numel, h);
    else
        hipLaunchKernelGGL(sgdm32_kernel<false>, dim3(grid), dim3(kThreads), 0, s, static_cast<float*>(param), grad, m, numel, h);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

int lpmm_adamw32_step(void* param, const void* grad, float* m, float* v, int64_t numel, int grad_dtype,
                      float lr, float beta1, float beta2, float eps, float weight_decay, int64_t step,
                      void* stream) {
    if (!param || !grad || !m || !v || numel < 1) return LPMM_EINVAL;
    if (grad_dtype != LPMM_GRAD_F32 && grad_dtype != LPMM_GRAD_BF16) return LPMM_EINVAL;
    if (!aligned(param, 4) || !aligned(m, 4) || !aligned(v, 4) ||
        !aligned(grad, grad_dtype == LPMM_GRAD_F32 ? 4 : 2))
        return LPMM_EINVAL;
    Hyper h;
    const int rc = make_hyper(lr, beta1, beta2, eps, weight_decay, step, &h);
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int grid = int((numel + kElemsPerWg32 - 1) / kElemsPerWg32);
    if (grad_dtype == LPMM_GRAD_BF16)
        hipLaunchKernelGGL(adamw32_kernel<true>, dim3(grid), dim3(kThreads), 0, s,
                           static_cast<float*>(param), grad, m, v, numel, h);
    else
        hipLaunchKernelGGL(adamw32_kernel<false>, dim3(grid), dim3(kThreads), 0, s,
                           static_cast<float*>(param), grad, m, v, numel, h);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

int lpmm_dequant_state(int which, const uint8_t* codes, const float* scale_a, const float* scale_b,
                       const int64_t shape[2], float* out, void* stream) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if ((which != 0 && which != 1 && which != 2) || !codes || !scale_a || !out || (which == 1 && !scale_b))
        return LPMM_EINVAL;
    if (!aligned(codes, 4) || !aligned(out, 4)) return LPMM_EINVAL;
    DeviceCtx* ctx;
    const int rc2 = current_ctx(&ctx);   // the DE table lives in device memory filled by init
    if (rc2) return rc2;
    QuantArgs q{};
    q.q_in = reinterpret_cast<const uint32_t*>(codes);
    q.x_out = out;
    q.sa = const_cast<float*>(scale_a);
    q.sb = const_cast<float*>(scale_b);
    q.rows = rows; q.cols = cols; q.P = rows * cols;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int grid = grid_for(q.P, kCvtElems / kThreads);
    if (which == 0) hipLaunchKernelGGL(dequant_m_kernel, dim3(grid), dim3(kThreads), 0, s, q);
    else if (which == 1 && q.P <= kRankShortElems) hipLaunchKernelGGL(dequant_v_kernel<2>, dim3(rank_grid(q.P, 2)), dim3(kThreads), 0, s, q);
    else if (which == 1) hipLaunchKernelGGL(dequant_v_kernel<4>, dim3(rank_grid(q.P, 4)), dim3(kThreads), 0, s, q);
    else hipLaunchKernelGGL(dequant_vb_kernel, dim3(grid), dim3(kThreads), 0, s, q);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

int lpmm_quant_state(int which, const float* in, const int64_t shape[2], uint8_t* codes, float* scale_a,
                     float* scale_b, void* stream) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    if ((which != 0 && which != 1 && which != 2) || !codes || !scale_a || !in || (which == 1 && !scale_b))
        return LPMM_EINVAL;
    if (!aligned(codes, 4) || !aligned(in, 4)) return LPMM_EINVAL;
    DeviceCtx* ctx;
    const int rc2 = current_ctx(&ctx);
    if (rc2) return rc2;
    QuantArgs q{};
    q.x_in = in;
    q.q_out = reinterpret_cast<uint32_t*>(codes);
    q.sa = scale_a;
    q.sb = scale_b;
    q.rows = rows; q.cols = cols; q.P = rows * cols;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int grid = grid_for(q.P, kCvtElems / kThreads);
    if (which == 0) {
        hipLaunchKernelGGL(quant_m_kernel, dim3(grid), dim3(kThreads), 0, s, q);
        LPMM_HIP(hipGetLastError());
    } else if (which == 2) {
        hipLaunchKernelGGL(quant_vb_kernel, dim3(grid), dim3(kThreads), 0, s, q);
        LPMM_HIP(hipGetLastError());
    } else {
        const int r = launch_maxima(q, ctx->n_cu, s);
        if (r) return r;
        if (q.P <= kRankShortElems) hipLaunchKernelGGL(quant_v_code_kernel<2>, dim3(rank_grid(q.P, 2)), dim3(kThreads), 0, s, q);
        else hipLaunchKernelGGL(quant_v_code_kernel<4>, dim3(rank_grid(q.P, 4)), dim3(kThreads), 0, s, q);
        LPMM_HIP(hipGetLastError());
    }
    return LPMM_OK;
}

}  // extern "C"

namespace {

// the map of an ablation quantizer with what its kernels search it by
struct AblationMap {
    AblEntries entries;
    AblSearch<false> nearest;
    AblSearch<true> stochastic;
};
// false for a combination that does not exist
bool build_ablation_map(int map, int is_signed, AblationMap* m) {
    float T[kCodes], thr[kCodes];
    int n = kCodes;
    if (map == LPMM_MAP_DE) {
        if (is_signed) build_de_signed(T); else build_de_unsigned(T);
    } else if (map == LPMM_MAP_DE0 && !is_signed) {
        float U[kCodes];
        build_de_unsigned(U);                 // U[0] is the zero that DE-0 drops
        n = kCodes - 1;
        for (int i = 0; i < n; ++i) T[i] = U[i + 1];
    } else if (map == LPMM_MAP_LINEAR && !is_signed) {
        build_linear(T);
    } else {
        return false;
    }
    *m = AblationMap{};
    std::copy(T, T + n, m->entries.T);
    build_thresholds_n(T, n, thr);
    const float* zero = std::find(T, T + n, 0.0f);
    auto fill_search = [&](AblMap* s, const float* v, int count) {
        for (int i = 0; i < kCodes; ++i) s->v[i] = i < count ? v[i] : std::numeric_limits<float>::infinity();
        std::fill(s->bucket, s->bucket + kCodes, kBuckets);
        s->n = n;
        s->zero4 = 0x1111u * (zero < T + n ? uint32_t(zero - T) : 0u);       // maps without a zero have nothing below their first entry
        s->least = is_signed ? -1.0f : 0.0f;
        return one_per_bucket(v, count, s->bucket);
    };
    bool ok = fill_search(&m->stochastic, T, n) && fill_search(&m->nearest, thr, n - 1);
    for (int i = 0; i < kCodes; ++i) {
        const int k = std::clamp(i, 1, n - 1);              // the gap between entries k - 1 and k
        float inv = float(0x1p24 / (double(T[k]) - double(T[k - 1])));
        while ((T[k] - T[k - 1]) * inv < 0x1p24f) inv = std::nextafterf(inv, std::numeric_limits<float>::infinity());
        m->stochastic.inv[i] = inv;
        // what the kernels' margins rest on
        ok = ok && std::max(std::fabs(double(T[k])), std::fabs(double(T[k - 1]))) <= 17.9 * (double(T[k]) - double(T[k - 1]));
    }
    return ok;
}
// null for a combination that does not exist
const AblationMap* ablation_map(int map, int is_signed) {
    struct Maps {
        AblationMap m[3][2];
        bool ok[3][2];
        Maps() {
            for (int k = 0; k < 3; ++k)
                for (int s = 0; s < 2; ++s) ok[k][s] = build_ablation_map(k, s, &m[k][s]);
        }
    };
    static const Maps maps;
    const int s = is_signed ? 1 : 0;
    return map >= 0 && map <= 2 && maps.ok[map][s] ? &maps.m[map][s] : nullptr;
}

bool ablation_valid(int norm, int is_signed) {
    return (norm == LPMM_NORM_B128 || norm == LPMM_NORM_B2048 || (norm == LPMM_NORM_RANK1 && !is_signed));
}

}  // namespace

extern "C" {

int lpmm_ablation_table(int map, int is_signed, float out[16]) {
    const AblationMap* m = ablation_map(map, is_signed);
    if (!out || !m) return LPMM_EINVAL;
    std::copy(m->entries.T, m->entries.T + kCodes, out);
    return m->nearest.n;
}

int lpmm_quant_ablation(int norm, int map, int is_signed, int rounding, uint64_t seed, const float* in,
                        const int64_t shape[2], uint8_t* codes, float* scale_a, float* scale_b, void* stream) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    const AblationMap* m = ablation_map(map, is_signed);
    if (!ablation_valid(norm, is_signed) || !m) return LPMM_EINVAL;
    if (rounding != LPMM_ROUND_NEAREST && rounding != LPMM_ROUND_STOCHASTIC) return LPMM_EINVAL;
    if (!in || !codes || !scale_a || (norm == LPMM_NORM_RANK1 && !scale_b)) return LPMM_EINVAL;
    if (!aligned(in, 4) || !aligned(codes, 4) || !aligned(scale_a, 4)) return LPMM_EINVAL;
    AblArgs a{};
    a.x_in = in;
    a.q_out = reinterpret_cast<uint32_t*>(codes);
    a.sa = scale_a;
    a.sb = scale_b;
    a.rows = rows; a.cols = cols; a.P = rows * cols;
    a.stochastic = rounding == LPMM_ROUND_STOCHASTIC;
    a.seed = seed;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int grid = grid_for(a.P, kCvtElems / kThreads);
    if (norm == LPMM_NORM_RANK1) {
        QuantArgs q{};
        q.x_in = in; q.sa = scale_a; q.sb = scale_b;
        q.rows = rows; q.cols = cols; q.P = a.P;
        const int r = launch_maxima(q, 256, s);       // this call needs no init, hence no device context
        if (r) return r;
    }
#define LPMM_ABL_BLOCK(SR, UNITS, M)                                                                                      \
    if (norm == LPMM_NORM_B128) hipLaunchKernelGGL((abl_quant_block_kernel<128, SR, UNITS>), dim3(blocks), dim3(kThreads), 0, s, a, M); \
    else hipLaunchKernelGGL((abl_quant_block_kernel<2048, SR, UNITS>), dim3(blocks), dim3(kThreads), 0, s, a, M);
    const bool shorter = a.stochastic && a.P <= kAblShortElems;
    const int blocks = shorter ? grid_for(a.P, 2 * kCvtUnitElems / kThreads) : grid;
    if (norm == LPMM_NORM_RANK1) {
#define LPMM_RANK1(SR, M)                                                                                                                  \
    if (a.P <= kAblShortElems) hipLaunchKernelGGL((abl_quant_rank1_kernel<SR, 2>), dim3(rank_grid(a.P, 2)), dim3(kThreads), 0, s, a, M); \
    else hipLaunchKernelGGL((abl_quant_rank1_kernel<SR, kCvtUnits>), dim3(grid), dim3(kThreads), 0, s, a, M);
        if (a.stochastic) { LPMM_RANK1(true, m->stochastic) } else { LPMM_RANK1(false, m->nearest) }
#undef LPMM_RANK1
    } else if (shorter) { LPMM_ABL_BLOCK(true, 2, m->stochastic) }
    else if (a.stochastic) { LPMM_ABL_BLOCK(true, kCvtUnits, m->stochastic) }
    else { LPMM_ABL_BLOCK(false, kCvtUnits, m->nearest) }
#undef LPMM_ABL_BLOCK
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

int lpmm_dequant_ablation(int norm, int map, int is_signed, const uint8_t* codes, const float* scale_a,
                          const float* scale_b, const int64_t shape[2], float* out, void* stream) {
    int64_t rows, cols;
    const int rc = check_shape(shape, &rows, &cols);
    if (rc) return rc;
    const AblationMap* m = ablation_map(map, is_signed);
    if (!ablation_valid(norm, is_signed) || !m) return LPMM_EINVAL;
    if (!codes || !scale_a || !out || (norm == LPMM_NORM_RANK1 && !scale_b)) return LPMM_EINVAL;
    if (!aligned(codes, 4) || !aligned(out, 4) || !aligned(scale_a, 4)) return LPMM_EINVAL;
    AblArgs a{};
    a.q_in = reinterpret_cast<const uint32_t*>(codes);
    a.x_out = out;
    a.sa = const_cast<float*>(scale_a);
    a.sb = const_cast<float*>(scale_b);
    a.rows = rows; a.cols = cols; a.P = rows * cols;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(abl_dequant_kernel, dim3(grid_for(a.P, kCvtElems / kThreads)), dim3(kThreads), 0, s, a, m->entries, norm);
    LPMM_HIP(hipGetLastError());
    return LPMM_OK;
}

size_t lpmm_adamw4_plan_bytes(const lpmm_tensor_desc* descs, int64_t n) {
    return lpmm_adamw4_plan_bytes_nd(descs, n, nullptr, nullptr);
}

size_t lpmm_adamw4_plan_bytes_nd(const lpmm_tensor_desc* descs, int64_t n, const int64_t* inner_dims,
                                 const int32_t* inner_ndim) {
    PlanLayout L;
    return plan_layout(descs, n, inner_dims, inner_ndim, &L) ? L.total : 0;
}

int lpmm_adamw4_plan_build(const lpmm_tensor_desc* descs, int64_t n, int grad_dtype, void* plan,
                           size_t plan_bytes, void* stream) {
    return lpmm_adamw4_plan_build_nd(descs, n, nullptr, nullptr, grad_dtype, plan, plan_bytes, stream);
}

int lpmm_adamw4_plan_build_nd(const lpmm_tensor_desc* descs, int64_t n, const int64_t* inner_dims,
                              const int32_t* inner_ndim, int grad_dtype, void* plan, size_t plan_bytes,
                              void* stream) {
    PlanLayout L;
    if (!plan_layout(descs, n, inner_dims, inner_ndim, &L)) return LPMM_EINVAL;
    // memory sized without a work list (under other settings of the environment): launches by phases
    if (plan_bytes < L.total) (void)plan_layout(descs, n, inner_dims, inner_ndim, &L, false);
    if (!plan || !aligned(plan, 256) || plan_bytes < L.total) return LPMM_EINVAL;
    if (grad_dtype != LPMM_GRAD_F32 && grad_dtype != LPMM_GRAD_BF16) return LPMM_EINVAL;
    DeviceCtx* ctx;
    int rc = current_ctx(&ctx);          // the lookup tables are uploaded by lpmm_adamw4_init
    if (rc) return rc;
    int dev = 0;
    LPMM_HIP(hipGetDevice(&dev));

    auto host = std::make_shared<PlanHost>();
    host->bf16 = grad_dtype == LPMM_GRAD_BF16;
    host->device = dev;
    host->staging.assign(L.off_counters, 0);
    Tensor4* tens = reinterpret_cast<Tensor4*>(host->staging.data() + L.off_tensors);
    InnerDims* h_dims = reinterpret_cast<InnerDims*>(host->staging.data() + L.off_dims);
    int64_t n_nd = 0;
    char* dplan = static_cast<char*>(plan);
    const Tensor4* d_tens = reinterpret_cast<const Tensor4*>(dplan + L.off_tensors);
    float* d_floats = reinterpret_cast<float*>(dplan + L.off_floats);
    const InnerDims* d_dims = reinterpret_cast<const InnerDims*>(dplan + L.off_dims);
    host->d_hyper = reinterpret_cast<Hyper*>(dplan + L.off_hyper);
    unsigned int* d_counters = reinterpret_cast<unsigned int*>(dplan + L.off_counters);

    int64_t all_params = 0;
    for (int64_t i = 0; i < n; ++i) all_params += descs[i].rows * descs[i].cols;
    const int64_t tall = all_params >= kRagPhaseParams ? kRagPhase : kRagTall;      // ragged_geometry
    const int64_t rw_hint = env_int("LPMM_MULTI_RW", -1);      // -1: the plan defaults (see the geometries)
    const int64_t rw2_hint = env_int("LPMM_MULTI_RW2", 128);
    // parameters per group of consecutive tensors: large groups win (fewer kernel tails)
    int64_t group_params = int64_t(env_int("LPMM_PHASE_MPARAMS", 2048)) << 20;
    if (n > kMaxSeg && env_int("LPMM_PHASE_MPARAMS", 0) <= 0) {
        // More tensors than one group's tables hold: cut by parameters, into about equal parts, instead of filling
        // every group up to the table size (292 tensors of 354 M parameters: 190 M + 164 M parameters measured 0.895
        // ms per step, the first 192 tensors + the rest, 254 M + 100 M, 0.905).  The tenth on top keeps the greedy fill
        // below from leaving a small group over.
        const int64_t k = (n + kMaxSeg - 1) / kMaxSeg;
        group_params = std::min(group_params, all_params / k + all_params / (10 * k) + 1);
    }
    // Tiling of one quantized tensor of the plan.  shrink = 0 gives the plan's default tiles (sized for sets that
    // fill the chip many times over); each further level halves the rows (blocks) a workgroup takes, for groups of
    // tensors that are too small to give every CU a couple of workgroups (see below).
    const int gbytes = grad_dtype == LPMM_GRAD_BF16 ? 2 : 4;
    auto set_geometry = [&](Tensor4& t, const lpmm_tensor_desc& d, int shrink) {
        const int64_t rw_s = std::max<int64_t>((rw_hint <= 0 ? 64 : rw_hint) >> shrink, 8);
        const int64_t rw2_s = std::max<int64_t>(rw2_hint >> shrink, 4);
        const int64_t rounds_s = std::max<int64_t>(int64_t(env_int("LPMM_MULTI_B128_ROUNDS", 8)) >> shrink, 1);
        if (d.kind == LPMM_KIND_SGDM_4BIT) {
            b128_geometry(&t, ctx->n_cu, rounds_s);
            t.kind = kSgdmBlock;
        } else if (d.kind == LPMM_KIND_4BIT_B128) {
            b128_geometry(&t, ctx->n_cu, rounds_s);
        } else if (d.kind == LPMM_KIND_4BIT_FACTOR) {
            factor_geometry(&t, ctx->n_cu, rw_s, rw2_s, gbytes, fast_eligible(d.cols, d.v_colmax), 1, shrink, tall);
        } else if (t.kind == kQuantFast) {
            rank1_fast_geometry(&t, 0, rw_hint > 0 ? rw_hint : 0, std::max<int64_t>(rw2_hint >> shrink, kGroups), gbytes, shrink);
        } else if (t.kind == kQuantRagged) {
            ragged_geometry(&t, 0, tall, shrink);
        }
    };
    int64_t fofs = 0;
    for (int64_t i = 0; i < n; ++i) {
        const lpmm_tensor_desc& d = descs[i];
        const size_t galign = grad_dtype == LPMM_GRAD_F32 ? 4 : 2;
        Tensor4 t{};
        t.rows = d.rows; t.cols = d.cols; t.P = d.rows * d.cols;
        if (d.flags & ~(LPMM_FLAG_NO_DECAY | LPMM_FLAG_DETERMINISTIC)) return LPMM_EINVAL;
        if ((d.flags & LPMM_FLAG_DETERMINISTIC) &&
            (d.kind != LPMM_KIND_4BIT_FACTOR || !fast_eligible(d.cols, d.v_colmax))) return LPMM_EINVAL;
        t.no_decay = (d.flags & LPMM_FLAG_NO_DECAY) ? 1 : 0;
        t.p = static_cast<float*>(d.param);
        t.g = d.grad;
        t.mq = static_cast<uint32_t*>(d.m_state);
        t.vq = static_cast<uint32_t*>(d.v_state);
        if (!d.param || !d.grad || !d.m_state) return LPMM_EINVAL;
        const bool is_sgdm = d.kind == LPMM_KIND_SGDM_4BIT || d.kind == LPMM_KIND_SGDM_FP32;
        if (!d.v_state && d.kind != LPMM_KIND_4BIT_FACTOR && !is_sgdm) return LPMM_EINVAL;
        if (d.kind == LPMM_KIND_SGDM_FP32) {
            if (!aligned(d.param, 4) || !aligned(d.m_state, 4) || !aligned(d.grad, galign)) return LPMM_EINVAL;
            t.vq = nullptr;
            t.kind = kSgdmFp32;
            t.n_wg = t.n_wg2 = int((t.P + kElemsPerWg32 - 1) / kElemsPerWg32);
            host->sgdm = true;
        } else if (d.kind == LPMM_KIND_SGDM_4BIT) {
            if (!d.m_blockscale) return LPMM_EINVAL;
            if (!aligned(d.param, 16) || !aligned(d.grad, 16) || !aligned(d.m_state, 4) || !aligned(d.m_blockscale, 4))
                return LPMM_EINVAL;
            t.vq = nullptr;
            t.ms = d.m_blockscale;
            set_geometry(t, d, 0);
            host->sgdm = true;
        } else if (d.kind == LPMM_KIND_4BIT_FACTOR) {
            if (!d.m_blockscale || !d.v_rowmax || !d.v_colmax) return LPMM_EINVAL;
            if (!aligned(d.param, 16) || !aligned(d.grad, 16) || !aligned(d.m_state, 4) ||
                !aligned(d.m_blockscale, 4) || !aligned(d.v_rowmax, 4) || !aligned(d.v_colmax, 4))
                return LPMM_EINVAL;
            t.vq = nullptr;
            t.ms = d.m_blockscale;
            t.r = d.v_rowmax;                      // row statistics
            t.c = d.v_colmax;                      // column statistics
            t.r_new = d_floats + fofs;
            fofs += round_up(d.rows, 64);
            t.c_new = d_floats + fofs;
            fofs += round_up(d.cols, 64);
            t.counter = d_counters + i * kCounterWords;
            if (d.flags & LPMM_FLAG_DETERMINISTIC) {
                t.det = 1;
                t.vq = reinterpret_cast<uint32_t*>(d_floats + fofs);      // the partial sums
                fofs += det_partial_floats(d.rows, d.cols);
            }
            set_geometry(t, d, 0);
            host->factor = true;
        } else if (d.kind == LPMM_KIND_FP32) {
            if (!aligned(d.param, 4) || !aligned(d.m_state, 4) || !aligned(d.v_state, 4) || !aligned(d.grad, galign))
                return LPMM_EINVAL;
            t.kind = kFp32State;
            t.n_wg = t.n_wg2 = int((t.P + kElemsPerWg32 - 1) / kElemsPerWg32);
        } else if (d.kind == LPMM_KIND_4BIT_B128) {
            if (!d.m_blockscale || !d.v_rowmax) return LPMM_EINVAL;
            if (!aligned(d.param, 16) || !aligned(d.grad, 16) || !aligned(d.m_state, 4) || !aligned(d.v_state, 4) ||
                !aligned(d.m_blockscale, 4) || !aligned(d.v_rowmax, 4))
                return LPMM_EINVAL;
            t.ms = d.m_blockscale;
            t.r = d.v_rowmax;                      // block scales of the second moment
            t.kind = kQuantBlockV;
            set_geometry(t, d, 0);
        } else {
            if (!d.m_blockscale || !d.v_rowmax || !d.v_colmax) return LPMM_EINVAL;
            if (!aligned(d.param, 16) || !aligned(d.grad, 16) || !aligned(d.m_state, 4) || !aligned(d.v_state, 4) ||
                !aligned(d.m_blockscale, 4) || !aligned(d.v_rowmax, 4) || !aligned(d.v_colmax, 4))
                return LPMM_EINVAL;
            t.ms = d.m_blockscale;
            t.r = d.v_rowmax;
            t.c = d.v_colmax;
            t.nd_index = -1;
            int64_t ext = 0;
            if (d.kind == LPMM_KIND_4BIT_ND) {
                // more than two dimensions: v_colmax holds the column scales and, behind them, the statistics of
                // the inner dimensions; the workspace mirrors that layout (see lpmm_adamw4_nd_step)
                InnerDims dm;
                if (!plan_inner_dims(d, i, inner_dims, inner_ndim, &dm, &ext)) return LPMM_EINVAL;
                h_dims[n_nd] = dm;
                t.nd_index = int(n_nd++);
                t.c_extra = int(ext);
            }
            t.r_new = d_floats + fofs;
            fofs += round_up(d.rows, 64);
            t.c_new = d_floats + fofs;
            fofs += round_up(d.cols + ext, 64);
            t.counter = d_counters + i * kCounterWords;
            if (fast_eligible(d.cols, d.v_colmax)) {
                t.kind = kQuantFast;
                set_geometry(t, d, 0);
            } else if (ragged_eligible(d.rows, d.cols)) {
                t.kind = kQuantRagged;
                set_geometry(t, d, 0);
            } else {
                t.kind = kQuantGeneral;
                general_geometry(&t, ctx->n_cu);
            }
        }
        tens[i] = t;
        host->params += t.P;
    }

    if (L.cap_items > 0) build_flow(descs, n, L, dplan, gbytes, host.get(), tens);

    // groups of consecutive tensors; phase j = A work of group j + B work of group j-1
    std::vector<std::pair<int64_t, int64_t>> groups;      // [first, last)
    for (int64_t i = 0; i < n;) {
        int64_t j = i, acc = 0;
        while (j < n && j - i < kMaxSeg && (j == i || acc + tens[j].P <= group_params)) acc += tens[j++].P;
        groups.emplace_back(i, j);
        i = j;
    }
    // A group whose tensors are small would put few, long workgroups on the chip (one 1024 x 1024 matrix: 128 for
    // its first pass, 32 for its second, on 256 CUs): halve its tiles until each of its launches has two
    // workgroups per CU (measured on that matrix: 23.5 -> 13.8 us per step).
    if (host->flow) groups.clear();
    for (const auto& gr : groups) {
        for (int shrink = 1; shrink <= 3; ++shrink) {
            int64_t n_a = 0, n_b = 0;
            bool two_pass = false;
            for (int64_t i = gr.first; i < gr.second; ++i) {
                n_a += tens[i].n_wg;
                const bool has_b = is_rank1(tens[i].kind) ||
                                   tens[i].kind == kFactorFast || tens[i].kind == kFactorGeneral ||
                                   tens[i].kind == kFactorRagged;
                if (has_b) { n_b += tens[i].n_wg2; two_pass = true; }
            }
            if (n_a >= 2 * int64_t(ctx->n_cu) && (!two_pass || n_b >= 2 * int64_t(ctx->n_cu))) break;
            for (int64_t i = gr.first; i < gr.second; ++i) set_geometry(tens[i], descs[i], shrink);
        }
    }
    // Rank-1 plans of several groups run second passes on a stream of their own beside the next group's first pass: what takes
    // launches by phases is mostly many small tensors, whose launches leave the chip half empty (one after the other / on two
    // streams, bf16 gradients: 300 of 200 x 300 108 / 103 us, 224 adapters of 8 x 4096 and 4096 x 8 139 / 119, 256 of 64 x 4096 and 4096 x
    // 64 326 / 314).  A group's passes follow each other in any case.  Factorized plans take their launches one after the other: a
    // statistics pass and an update each run at the memory system's rate alone, and side by side they only get in each other's way
    // (7B-shaped set: 14.71 ms per step against 14.84, 354 M set 0.841 against 0.854).
    auto narrow_kind = [](int kind) { return kind == kQuantGeneral || kind == kFactorGeneral; };
    const int stream_mode = env_int("LPMM_MULTI_STREAMS", host->factor || host->sgdm ? 0 : 2);
    for (size_t j = 0; j <= groups.size() && !host->flow; ++j) {
        PhaseLaunch pl{};
        int64_t elems_a = 0, elems_b = 0, elems_gen = 0;
        int64_t narrow_a = 0, narrow_b = 0;     // of elems_a and elems_b, those on the general tiles of either form
        pl.ph.tensors = reinterpret_cast<const Tensor4Table*>(d_tens);
        if (j < groups.size())
            for (int64_t i = groups[j].first; i < groups[j].second; ++i) {
                pl.ph.seg_a[pl.ph.n_seg_a++] = Segment{pl.ph.n_a, int(i)};
                if (is_rank1(tens[i].kind)) pl.a_has_rank1 = true;
                pl.ph.n_a += tens[i].n_wg;
                elems_a += tens[i].P;
                narrow_a += narrow_kind(tens[i].kind) ? tens[i].P : 0;
            }
        // The second pass of the general tiles gathers, and what it needs is many waves: 62 registers and no LDS, where the others'
        // update takes 85 and 24 KB.  Beside others it gets a launch of its own where that saves more than the launch and its tail
        // cost, from 2^23 parameters on and where it is two thirds of the group (seven of 30000 x 96 and two of 1024 x 4096, fp32: together
        // 242 us, apart 197; three and one 126 and 110; twelve and six, 0.58, 407 and 412; half, 64 x 4096 and 4096 x 64, 149 and 159; 5.8 M
        // and 2 M parameters 87 and 91).
        bool split = false;
        if (j >= 1 && (stream_mode == 0 || stream_mode >= 2)) {
            int64_t narrow = 0, others = 0;
            for (int64_t i = groups[j - 1].first; i < groups[j - 1].second; ++i)
                (tens[i].kind == kQuantGeneral ? narrow : others) += is_rank1(tens[i].kind) ? tens[i].P : 0;
            split = narrow >= int64_t(1) << 23 && others > 0 && narrow >= 2 * others;
        }
        if (j >= 1)
            for (int64_t i = groups[j - 1].first; i < groups[j - 1].second; ++i) {
                if (tens[i].kind == kFp32State || tens[i].kind == kQuantBlockV || tens[i].kind == kSgdmBlock ||
                    tens[i].kind == kSgdmFp32)
                    continue;
                const bool apart = split && tens[i].kind == kQuantGeneral;
                Phase& to = apart ? pl.gen : pl.ph;
                if (!apart) pl.b_general = (pl.ph.n_b == 0 || pl.b_general) && tens[i].kind == kQuantGeneral;
                to.seg_b[to.n_seg_b++] = Segment{to.n_b, int(i)};
                to.n_b += tens[i].n_wg2;
                (apart ? elems_gen : elems_b) += tens[i].P;
                narrow_b += !apart && narrow_kind(tens[i].kind) ? tens[i].P : 0;
                if (tens[i].det) {
                    pl.has_det = true;
                    pl.det.seg_r[pl.det.n_seg++] = Segment{pl.det.n_r, int(i)};
                    pl.det.n_r += int((tens[i].rows + kThreads - 1) / kThreads + (tens[i].cols + 63) / 64);
                }
                if (tens[i].nd_index >= 0 && is_rank1(tens[i].kind)) {
                    pl.has_nd = true;
                    pl.nd.seg_r[pl.nd.n_seg] = Segment{pl.nd.n_r, int(i)};
                    pl.nd.seg_e[pl.nd.n_seg] = Segment{pl.nd.n_e, int(i)};
                    ++pl.nd.n_seg;
                    pl.nd.n_r += tens[i].c_extra;                                       // one workgroup per statistic
                    pl.nd.n_e += int((tens[i].cols + kThreads - 1) / kThreads);
                }
            }
        pl.nd.tensors = pl.ph.tensors;
        pl.nd.dims = d_dims;
        pl.det.tensors = pl.ph.tensors;
        if (pl.ph.n_a + pl.ph.n_b == 0) continue;
        // A workgroup of the general tiles' second pass takes 2048 elements, of the other tiles' up to 16384: where the list has the
        // narrow tensors in one place, eighths of the launch would give one XCD most of the others' work, and it is dealt in runs (three
        // of 30000 x 96 before three of 1024 x 4096, fp32 and bf16 gradients: 190 and 158 us in eighths, 138 and 116 in runs; 64 x 4096
        // and 4096 x 64 in turn, 268 M parameters, even as they are: 1251 and 1251, in runs 1287 and 1280).  First passes keep the
        // eighths: in runs all XCDs raise the same tensor's column maxima at a time (157 and 146 in place of 138 and 116).
        bool dealt = false;
        if (narrow_b > 0 && !host->factor) {
            double part[kXcds] = {};
            const double eighth = double(std::max(pad8(pl.ph.n_b), kXcds)) / kXcds;
            for (int k = 0; k < pl.ph.n_seg_b; ++k) {
                const Tensor4& t = tens[pl.ph.seg_b[k].tensor];
                const double begin = pl.ph.seg_b[k].wg_begin, end = begin + t.n_wg2;
                for (int x = 0; x < kXcds; ++x)
                    part[x] += double(t.P) * std::max(0.0, std::min(end, (x + 1) * eighth) - std::max(begin, x * eighth)) / (end - begin);
            }
            dealt = *std::max_element(part, part + kXcds) > 1.25 * double(elems_b) / kXcds;
        }
        // No skew where the general tiles are most of a launch (30000 x 96 as 0.85 of the parameters, factorized, fp32 gradients, 625 us
        // with it, 611 without; as 0.4, rank-1, 138 and 143).
        auto skew = [](int n, int64_t elems, int64_t narrow) { return narrow > elems / 4 * 3 ? 0 : launch_skew(n, elems); };
        pl.ph.skew_a = skew(pl.ph.n_a, elems_a, narrow_a);
        pl.ph.skew_b = dealt ? kDealt : skew(pl.ph.n_b, elems_b, narrow_b);
        if (int64_t(pl.ph.n_a) + pl.ph.n_b > (int64_t(1) << 30)) return LPMM_EINVAL;
        pl.grid_a = pad8(pl.ph.n_a);
        pl.grid_b = dealt ? int(round_up(pl.ph.n_b, kXcds * kDealRun)) : pad8(pl.ph.n_b);
        pl.grid = pl.ph.n_a == 0 ? pl.grid_b : pad8(int64_t(pl.ph.n_a) + pl.ph.n_b);
        pl.gen.tensors = pl.ph.tensors;
        pl.gen.skew_b = skew(pl.gen.n_b, elems_gen, elems_gen);
        pl.grid_gen = pad8(pl.gen.n_b);
        host->phases.push_back(pl);
    }
    host->serial = stream_mode == 0 && !host->sgdm;
    host->plain = std::all_of(tens, tens + n, [&](const Tensor4& t) { return t.kind != kQuantRagged && t.kind != kFactorRagged && !narrow_kind(t.kind); });
    // The factorized update is six waves on a SIMD with the ragged tile in the kernel and eight without.  Where a launch is long that is
    // more streams over the memory than it serves well, so the lighter kernel is for launches below 2^25 parameters (with the ragged tile
    // and without, us, bf16 gradients: 4 of 1024 x 1024 20.9 and 19.4, 12 layers of width 256 34.4 and 33.4, 16 of 1024 x 1024 44.2 and
    // 43.4, 24 62.5 and 61.8, 8192 x 4096 89.7 and 89.9; 2 layers of width 1024 with 50257 x 1024 beside them 190.1 and 194.6, 12 such
    // layers 454 and 461).
    for (PhaseLaunch& pl : host->phases) {
        int64_t elems = 0;
        for (int k = 0; k < pl.ph.n_seg_b; ++k) elems += tens[pl.ph.seg_b[k].tensor].P;
        pl.plain_b = host->plain && (!host->factor || elems < int64_t(1) << 25);
    }
    bool any_b = false;
    for (const PhaseLaunch& pl : host->phases) any_b = any_b || pl.ph.n_b > 0;
    if (stream_mode >= 2 && groups.size() > 1 && !host->sgdm && any_b && !host->flow) {
        LPMM_HIP(hipStreamCreateWithFlags(&host->side, hipStreamNonBlocking));
        LPMM_HIP(hipEventCreateWithFlags(&host->ev_fork, hipEventDisableTiming));
        LPMM_HIP(hipEventCreateWithFlags(&host->ev_join, hipEventDisableTiming));
        if (stream_mode >= 3) {
            LPMM_HIP(hipStreamCreateWithFlags(&host->side_a, hipStreamNonBlocking));
            LPMM_HIP(hipEventCreateWithFlags(&host->ev_join_a, hipEventDisableTiming));
        }
        host->ev_a.resize(host->phases.size());
        for (hipEvent_t& e : host->ev_a) LPMM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    }

    hipStream_t s = static_cast<hipStream_t>(stream);
    LPMM_HIP(hipMemsetAsync(dplan + L.off_counters, 0, L.total - L.off_counters, s));
    LPMM_HIP(hipMemcpyAsync(dplan, host->staging.data(), L.off_counters, hipMemcpyHostToDevice, s));
    std::lock_guard<std::mutex> lock(g_mu);
    g_plans[plan] = std::move(host);
    return LPMM_OK;
}

}  // extern "C"

namespace {

// One-pass kernels (block-wise AdamW, SGDM) of plans of 2^30 parameters or more run with four workgroups per CU
// instead of the seven or eight that their registers allow, by way of unused dynamic LDS: 1 % less time per step on
// the 7B-shaped set (more resident waves only lengthen every wave's queueing), 2-3 % more on the 354 M set, whose
// launches are short, hence the size condition.  LPMM_P3_LDS_PAD overrides the number of bytes.
unsigned one_pass_lds_pad(const PlanHost& host) {
    return unsigned(std::clamp(env_int("LPMM_P3_LDS_PAD", host.params >= (int64_t(1) << 30) ? 14336 : 0), 0, 45056));
}

// lr_dev / step_dev non-null: the capturable form, hyper-parameters prepared on the device
int adamw4_step_multi_impl(void* plan, float lr, const float* lr_dev, float beta1, float beta2, float eps,
                           float weight_decay, int64_t step, const int64_t* step_dev, void* stream) {
#define LPMM_CHECK(call) do { const int rc_ = (call); if (rc_) return rc_; } while (0)
    // column maxima -> new statistics -> new column scales, for the group's tensors with more than two dimensions
    auto launch_nd = [](const PhaseLaunch& pl, hipStream_t on) -> int {
        hipLaunchKernelGGL(nd_plan_reduce, dim3(pl.nd.n_r), dim3(kThreads), 0, on, pl.nd);
        LPMM_HIP(hipGetLastError());
        hipLaunchKernelGGL(nd_plan_expand, dim3(pl.nd.n_e), dim3(kThreads), 0, on, pl.nd);
        LPMM_HIP(hipGetLastError());
        return LPMM_OK;
    };
    // per-tile partial sums -> row / column sums and totals, for the group's tensors with deterministic sums
    auto launch_det = [](const PhaseLaunch& pl, hipStream_t on) -> int {
        hipLaunchKernelGGL(factor_plan_reduce, dim3(pl.det.n_r), dim3(kThreads), 0, on, pl.det);
        LPMM_HIP(hipGetLastError());
        hipLaunchKernelGGL(factor_plan_totals, dim3(pl.det.n_seg), dim3(kThreads), 0, on, pl.det);
        LPMM_HIP(hipGetLastError());
        return LPMM_OK;
    };
    const bool capturable = lr_dev != nullptr;
    HyperArg h{};
    const int rc = make_hyper(capturable ? 0.0f : lr, beta1, beta2, eps, weight_decay, capturable ? 1 : step, &h.h);
    if (rc) return rc;
    if (capturable && !step_dev) return LPMM_EINVAL;
    std::shared_ptr<const PlanHost> host;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        auto it = g_plans.find(plan);
        if (it == g_plans.end()) return LPMM_EINVAL;
        host = it->second;
    }
    int dev = 0;
    LPMM_HIP(hipGetDevice(&dev));
    if (dev != host->device || host->sgdm) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool bf16 = host->bf16;
    if (capturable) {
        hipLaunchKernelGGL(hyper_prepare_kernel, dim3(1), dim3(64), 0, s, lr_dev, step_dev, beta1, beta2, eps,
                           weight_decay, host->d_hyper);
        LPMM_HIP(hipGetLastError());
        h.dev = host->d_hyper;
    }
    if (host->flow) {
        const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
        const int64_t call = g_prof.calls;
        if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
        const dim3 grid(unsigned(host->flow_args.n_items)), block(kThreads);
#define LPMM_FLOW_CASE(F)                                                                                   \
        if (bf16) hipLaunchKernelGGL((flow_kernel<true, F>), grid, block, host->flow_any ? 0 : host->factor ? kFlowLdsPadFactor : kFlowLdsPad, s, host->flow_args, h);        \
        else hipLaunchKernelGGL((flow_kernel<false, F>), grid, block, host->flow_any ? 0 : host->factor ? kFlowLdsPadFactor : kFlowLdsPad, s, host->flow_args, h);
        if (host->factor) { LPMM_FLOW_CASE(kFlowFactor) }
        else if (host->flow_any) { LPMM_FLOW_CASE(kFlowRank1Any) }
        else { LPMM_FLOW_CASE(kFlowRank1) }
#undef LPMM_FLOW_CASE
        LPMM_HIP(hipGetLastError());
        if (rec) {
            LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
            LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
            g_prof.calls = call + 1;
        }
        return LPMM_OK;
    }
    const unsigned pad3 = one_pass_lds_pad(*host);
    // roles: 0 = A and B work in one launch, 1 = A only, 2 = B only, 3 = A only without rank-1 tensors
    // B work: behind it, where they are apart, the tensors on the general tiles
    auto launch = [&](int roles, int grid, hipStream_t on, const PhaseLaunch& pl) -> int {
#define LPMM_PHASE_LAUNCH(K, R, PLAIN)                                                                      \
        if (bf16) hipLaunchKernelGGL((K<true, R, PLAIN>), dim3(grid), dim3(kThreads), (R == 3 ? pad3 : 0), on, pl.ph, h);     \
        else hipLaunchKernelGGL((K<false, R, PLAIN>), dim3(grid), dim3(kThreads), (R == 3 ? pad3 : 0), on, pl.ph, h);
#define LPMM_PHASE_CASE(K, R) { LPMM_PHASE_LAUNCH(K, R, false) }
#define LPMM_PHASE_PASS(K, R) { if (R == 2 ? pl.plain_b : host->plain) { LPMM_PHASE_LAUNCH(K, R, true) } else { LPMM_PHASE_LAUNCH(K, R, false) } }
        if (host->factor) {
            if (roles == 0) LPMM_PHASE_CASE(factor_phase_kernel, 0)
            else if (roles == 2) LPMM_PHASE_PASS(factor_phase_kernel, 2)
            else LPMM_PHASE_PASS(factor_phase_kernel, 1)
        } else {
            if (roles == 0) LPMM_PHASE_CASE(phase_kernel, 0)
            else if (roles == 1) LPMM_PHASE_PASS(phase_kernel, 1)
            else if (roles == 2 && pl.b_general) LPMM_PHASE_CASE(phase_kernel, 4)
            else if (roles == 2) LPMM_PHASE_PASS(phase_kernel, 2)
            else LPMM_PHASE_CASE(phase_kernel, 3)
        }
#undef LPMM_PHASE_CASE
#undef LPMM_PHASE_PASS
#undef LPMM_PHASE_LAUNCH
        LPMM_HIP(hipGetLastError());
        if (roles == 2 && pl.grid_gen > 0) {
            if (bf16) hipLaunchKernelGGL((phase_kernel<true, 4>), dim3(pl.grid_gen), dim3(kThreads), 0, on, pl.gen, h);
            else hipLaunchKernelGGL((phase_kernel<false, 4>), dim3(pl.grid_gen), dim3(kThreads), 0, on, pl.gen, h);
            LPMM_HIP(hipGetLastError());
        }
        return LPMM_OK;
    };
    bool two_pass = false;
    for (const PhaseLaunch& pl : host->phases) two_pass = two_pass || pl.ph.n_b > 0;
    if (host->side || host->serial) {
        // A work of phase j on the caller's stream, B work (second pass of the tensors whose first pass
        // ran in phase j-1) on the side stream behind an event; the caller's stream rejoins at the end.
        // Serial plans take the same launches one after the other on the caller's stream, without events.
        const bool two = host->side != nullptr;
        hipStream_t s2 = two ? host->side : s;
        // The side stream's first work waits for the event behind the first A launch, which also puts it behind
        // everything that was on the caller's stream before this call (and into a capture of that stream): no fork
        // event is needed for it.  A second stream for first passes starts with work of its own and does need one.
        if (host->side_a) {
            LPMM_HIP(hipEventRecord(host->ev_fork, s));
            LPMM_HIP(hipStreamWaitEvent(host->side_a, host->ev_fork, 0));
        }
        // The last phase holds B work only, with no first pass left to run beside: it goes on the caller's stream,
        // straight behind the A work it depends on, and spares the step one hand-over between the streams (a
        // dependent launch on another stream starts 10-15 us later than one on the same stream).
        const size_t n_ph = host->phases.size();
        const bool tail_on_s = two && !host->side_a && n_ph >= 2 && host->phases[n_ph - 1].ph.n_a == 0;
        for (size_t j = 0; j < n_ph; ++j) {
            const PhaseLaunch& pl = host->phases[j];
            const bool tail = tail_on_s && j + 1 == n_ph;
            if (tail) {
                LPMM_HIP(hipEventRecord(host->ev_join, s2));      // everything the side stream was given
                s2 = s;
            }
            if (pl.ph.n_b > 0) {
                if (two && !tail) LPMM_HIP(hipStreamWaitEvent(s2, host->ev_a[j - 1], 0));
                // the heavy kernel of a plan with two passes is its B work (the update pass): that one is timed
                const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
                const int64_t call = g_prof.calls;
                if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s2));
                if (pl.has_nd) LPMM_CHECK(launch_nd(pl, s2));
                if (pl.has_det) LPMM_CHECK(launch_det(pl, s2));
                LPMM_CHECK(launch(2, pl.grid_b, s2, pl));
                if (rec) {
                    LPMM_HIP(hipEventRecord(prof_event(call, 1), s2));
                    LPMM_HIP(hipEventRecord(prof_event(call, 2), s2));
                    g_prof.calls = call + 1;
                }
            }
            hipStream_t sa = (host->side_a && (j & 1)) ? host->side_a : s;
            if (pl.ph.n_a > 0) {
                const bool rec = !two_pass && g_prof.on && g_prof.calls < g_prof.max_calls;
                const int64_t call = g_prof.calls;
                if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), sa));
                LPMM_CHECK(launch(pl.a_has_rank1 ? 1 : 3, pl.grid_a, sa, pl));
                if (rec) {
                    LPMM_HIP(hipEventRecord(prof_event(call, 1), sa));
                    LPMM_HIP(hipEventRecord(prof_event(call, 2), sa));
                    g_prof.calls = call + 1;
                }
            }
            // an event only where the next phase has B work that waits for it on the side stream (nobody waits
            // for the A work of the last group when its B work follows it on the same stream)
            const bool waited_for = j + 1 < n_ph && host->phases[j + 1].ph.n_b > 0 && !(tail_on_s && j + 2 >= n_ph);
            if (two && waited_for) LPMM_HIP(hipEventRecord(host->ev_a[j], sa));
        }
        if (!two) return LPMM_OK;
        if (!tail_on_s) LPMM_HIP(hipEventRecord(host->ev_join, s2));
        LPMM_HIP(hipStreamWaitEvent(s, host->ev_join, 0));
        if (host->side_a) {
            LPMM_HIP(hipEventRecord(host->ev_join_a, host->side_a));
            LPMM_HIP(hipStreamWaitEvent(s, host->ev_join_a, 0));
        }
        return LPMM_OK;
    }
    for (const PhaseLaunch& pl : host->phases) {
        // as on the other route, only launches that carry the update are timed
        const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls && (two_pass ? pl.ph.n_b > 0 : pl.ph.n_a > 0);
        const int64_t call = g_prof.calls;
        if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
        // a launch that holds only one kind of work takes that kind's (lighter) kernel
        if (pl.has_nd) LPMM_CHECK(launch_nd(pl, s));      // the A work of these tensors ran in the previous launch
        if (pl.has_det) LPMM_CHECK(launch_det(pl, s));
        const int roles = pl.ph.n_b == 0 ? (pl.a_has_rank1 ? 1 : 3) : (pl.ph.n_a == 0 ? 2 : 0);
        LPMM_CHECK(launch(roles, pl.grid, s, pl));
        if (rec) {
            LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
            LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
            g_prof.calls = call + 1;
        }
    }
    return LPMM_OK;
}

int sgdm4_step_multi_impl(void* plan, float lr, const float* lr_dev, float momentum, void* stream) {
    HyperArg h{};
    const int rc = make_sgdm_hyper(lr_dev ? 0.0f : lr, momentum, &h.h);
    if (rc) return rc;
    std::shared_ptr<const PlanHost> host;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        auto it = g_plans.find(plan);
        if (it == g_plans.end()) return LPMM_EINVAL;
        host = it->second;
    }
    int dev = 0;
    LPMM_HIP(hipGetDevice(&dev));
    if (dev != host->device || !host->sgdm) return LPMM_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (lr_dev) {
        hipLaunchKernelGGL(sgdm_hyper_prepare_kernel, dim3(1), dim3(64), 0, s, lr_dev, momentum, host->d_hyper);
        LPMM_HIP(hipGetLastError());
        h.dev = host->d_hyper;
    }
    for (const PhaseLaunch& pl : host->phases) {
        if (pl.ph.n_a == 0) continue;
        const bool rec = g_prof.on && g_prof.calls < g_prof.max_calls;
        const int64_t call = g_prof.calls;
        if (rec) LPMM_HIP(hipEventRecord(prof_event(call, 0), s));
        const unsigned pads = one_pass_lds_pad(*host);
        if (host->bf16) hipLaunchKernelGGL(sgdm_phase_kernel<true>, dim3(pl.grid_a), dim3(kThreads), pads, s, pl.ph, h);
        else hipLaunchKernelGGL(sgdm_phase_kernel<false>, dim3(pl.grid_a), dim3(kThreads), pads, s, pl.ph, h);
        LPMM_HIP(hipGetLastError());
        if (rec) {
            LPMM_HIP(hipEventRecord(prof_event(call, 1), s));
            LPMM_HIP(hipEventRecord(prof_event(call, 2), s));
            g_prof.calls = call + 1;
        }
    }
    return LPMM_OK;
}

}  // namespace

extern "C" {

int lpmm_adamw4_step_multi(void* plan, float lr, float beta1, float beta2, float eps, float weight_decay,
                           int64_t step, void* stream) {
    return adamw4_step_multi_impl(plan, lr, nullptr, beta1, beta2, eps, weight_decay, step, nullptr, stream);
}

int lpmm_adamw4_step_multi_capturable(void* plan, const float* lr, const int64_t* step, float beta1, float beta2,
                                      float eps, float weight_decay, void* stream) {
    if (!lr || !step) return LPMM_EINVAL;
    return adamw4_step_multi_impl(plan, 0.0f, lr, beta1, beta2, eps, weight_decay, 1, step, stream);
}

int lpmm_sgdm4_step_multi(void* plan, float lr, float momentum, void* stream) {
    return sgdm4_step_multi_impl(plan, lr, nullptr, momentum, stream);
}

int lpmm_sgdm4_step_multi_capturable(void* plan, const float* lr, float momentum, void* stream) {
    if (!lr) return LPMM_EINVAL;
    return sgdm4_step_multi_impl(plan, 0.0f, lr, momentum, stream);
}

int lpmm_adamw4_plan_release(void* plan) {
    std::lock_guard<std::mutex> lock(g_mu);
    return g_plans.erase(plan) ? LPMM_OK : LPMM_EINVAL;
}

int lpmm_adamw4_plan_launches(const void* plan) {
    std::lock_guard<std::mutex> lock(g_mu);
    auto it = g_plans.find(const_cast<void*>(plan));
    if (it == g_plans.end()) return LPMM_EINVAL;
    const PlanHost& host = *it->second;
    if (host.flow) return 1;
    int n = 0;
    for (const PhaseLaunch& pl : host.phases) {
        const int between = (pl.has_nd ? 2 : 0) + (pl.has_det ? 2 : 0) + (pl.grid_gen > 0 ? 1 : 0);
        if (host.sgdm) n += pl.ph.n_a > 0;
        else if (host.side || host.serial) n += (pl.ph.n_a > 0) + (pl.ph.n_b > 0) + between;
        else n += 1 + between;
    }
    return n;
}

int lpmm_profile_begin(int64_t max_calls) {
    if (max_calls < 1 || max_calls > (int64_t(1) << 20)) return LPMM_EINVAL;
    while (int64_t(g_prof.ev.size()) < 3 * max_calls) {
        hipEvent_t e;
        LPMM_HIP(hipEventCreate(&e));
        g_prof.ev.push_back(e);
    }
    g_prof.max_calls = max_calls;
    g_prof.calls = 0;
    g_prof.on = true;
    return LPMM_OK;
}

int lpmm_profile_end(double ms[2], int64_t* n_calls) {
    if (!ms || !n_calls) return LPMM_EINVAL;
    g_prof.on = false;
    ms[0] = ms[1] = 0.0;
    *n_calls = g_prof.calls;
    for (int64_t c = 0; c < g_prof.calls; ++c) {
        LPMM_HIP(hipEventSynchronize(prof_event(c, 2)));
        float a = 0.0f, b = 0.0f;
        LPMM_HIP(hipEventElapsedTime(&a, prof_event(c, 0), prof_event(c, 1)));
        LPMM_HIP(hipEventElapsedTime(&b, prof_event(c, 1), prof_event(c, 2)));
        ms[0] += a;
        ms[1] += b;
    }
    g_prof.calls = 0;
    return LPMM_OK;
}

}  // extern "C"

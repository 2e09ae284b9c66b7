// Host side of the C ABI: argument validation, plan storage layout, kernel selection and launch.
// Every check that can be made without the GPU is made before the first HIP call.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <mutex>
#include <new>
#include <thread>

#include "../../include/lora_mi355x.h"
#include "kernels.h"

using namespace lora;

static_assert(LORA_ERR_BAD_ADAPTER_ID == kErrBadAdapterId, "status codes out of sync");
static_assert(LORA_ERR_LENGTH_MISMATCH == kErrLengthMismatch, "status codes out of sync");
static_assert(LORA_ERR_ADAPTER_NOT_RESIDENT == kErrNotResident, "status codes out of sync");
static_assert(LORA_ERR_RANK_TOO_LARGE == kErrRankTooLarge, "status codes out of sync");
static_assert(LORA_ERR_SHAPE == kErrShape, "status codes out of sync");
static_assert(LORA_MAX_MULTI == kMaxGemmSets, "projection limit out of sync");
static_assert(LORA_MAX_RANK == kMaxRank, "rank limit out of sync");

// Scratch of lora_linear_static(): the layer's workspace for callers that cannot bring or allocate one.  One copy
// per GPU, at its own address (looked up once per context, on that context's device), held until the process ends.
static __device__ __align__(256) unsigned char scratch[LORA_STATIC_SCRATCH_BYTES];

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    (void)hipGetLastError();  // clear the sticky error so that the caller's next HIP call is not blamed
    return LORA_ERR_HIP;
}
#define LORA_HIP(call)                           \
    do {                                         \
        hipError_t e_ = (call);                  \
        if (e_ != hipSuccess) return hip_fail(e_); \
    } while (0)

enum ProfKind { kProfPlanSegments = 0, kProfPlanFill = 1, kProfShrink = 2, kProfGemm = 3, kProfExpand = 4, kProfKinds = 5 };
static_assert(kProfKinds == LORA_PROFILE_KINDS, "profile kinds out of sync");

constexpr int kRingSlots = 4;
constexpr size_t kRingSlotInts = 2 * (size_t)LORA_MAX_REQUESTS + LORA_MAX_ADAPTERS;
constexpr int kTableSlots = 16;  // plan tables in flight (a batch of a few hundred requests: ~10 KB, and a plan lasts as long as its layers)

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Scratch of the plan tables' counting sort, one entry per adapter slot and one for "no adapter"; made with the context, so
// that lora_plan() allocates nothing.  Only the entries of the slots in use are ever touched.
struct KeyScratch {
    int32_t rows[LORA_MAX_ADAPTERS + 1], seg[LORA_MAX_ADAPTERS + 1];
    uint64_t used[(LORA_MAX_ADAPTERS + 63) / 64];
};

}  // namespace

struct lora_ctx {
    int device = 0;
    int num_cu = 256;
    unsigned char *static_scratch = nullptr;  // this device's copy of `scratch`
    // pinned staging ring for lora_plan's small host arrays
    int32_t *ring = nullptr;
    hipEvent_t ring_event[kRingSlots] = {};
    bool ring_used[kRingSlots] = {};
    int ring_next = 0;
    // pinned tables that plan_apply_kernel reads in place, and the words in which it reports having read them
    int32_t *tables = nullptr;
    uint32_t *table_done = nullptr;
    uint32_t table_ticket[kTableSlots] = {};  // what the slot's word reads when its table is free
    uint32_t last_ticket = 0;
    int table_next = 0;
    KeyScratch *keys = nullptr;
    std::mutex ring_mutex;  // guards everything above
    // tuning overrides (-1 = heuristic)
    int opt_gemm_variant = -1;
    int opt_decode_waves = -1;
    int opt_decode_max_rows = -1;
    int opt_plan_fused_rows = -1;
    int opt_shrink_rank_block = -1;
    int opt_plan_variant = -1;
    int opt_expand_split = -1;
    int opt_gemm_split_k = -1;
    // profiling mode: event pairs recorded tightly around each kernel
    bool prof_on = false;
    int prof_cap = 0;
    int prof_used[kProfKinds] = {};
    hipEvent_t *prof_start[kProfKinds] = {};
    hipEvent_t *prof_stop[kProfKinds] = {};
};

namespace {

// Sets the context's device for the duration of a call and restores the caller's.
struct DeviceGuard {
    int prev = -1;
    bool changed = false;
    hipError_t err = hipSuccess;
    explicit DeviceGuard(int dev) {
        err = hipGetDevice(&prev);
        if (err == hipSuccess && prev != dev) {
            err = hipSetDevice(dev);
            changed = err == hipSuccess;
        }
    }
    ~DeviceGuard() {
        if (changed) (void)hipSetDevice(prev);
    }
};

// Next event pair of a kernel kind while profiling (null otherwise, or when the pairs ran out).
bool next_timer(lora_ctx *ctx, int kind, KernelTimer *out) {
    if (!ctx->prof_on || ctx->prof_used[kind] >= ctx->prof_cap) return false;
    const int i = ctx->prof_used[kind]++;
    out->start = ctx->prof_start[kind][i];
    out->stop = ctx->prof_stop[kind][i];
    return true;
}

void free_profiler(lora_ctx *ctx) {
    for (int k = 0; k < kProfKinds; ++k) {
        for (int i = 0; i < ctx->prof_cap; ++i) {
            if (ctx->prof_start[k] && ctx->prof_start[k][i]) (void)hipEventDestroy(ctx->prof_start[k][i]);
            if (ctx->prof_stop[k] && ctx->prof_stop[k][i]) (void)hipEventDestroy(ctx->prof_stop[k][i]);
        }
        delete[] ctx->prof_start[k];
        delete[] ctx->prof_stop[k];
        ctx->prof_start[k] = ctx->prof_stop[k] = nullptr;
        ctx->prof_used[k] = 0;
    }
    ctx->prof_cap = 0;
    ctx->prof_on = false;
}

// ---- plan storage layout ------------------------------------------------------------------------
struct PlanLayout {
    size_t staged, tok_off, req_dst, hist, cursor, key_seg, perm, row_seg, row_adapter, row_ext, seg_adapter, seg_indptr, seg_rank, seg_ext,
        seg_unit, unit_rec, ext_rec, scalars, total_bytes;
    int32_t seg_cap, ext_cap;
};

bool plan_sizes_ok(int32_t n_req, int64_t T, int32_t n_adapters, int32_t r_max) {
    return n_req >= 0 && n_req <= LORA_MAX_REQUESTS && n_adapters >= 0 && n_adapters <= LORA_MAX_ADAPTERS && T >= 0 &&
           T <= (int64_t)INT32_MAX - 65536 && r_max >= 0 && r_max <= LORA_MAX_RANK && (r_max & 7) == 0;
}

PlanLayout plan_layout(int32_t n_req, int64_t T, int32_t n_adapters, int32_t r_max) {
    PlanLayout L;
    size_t off = 0;  // in int32 units; every section starts on a 256-byte boundary
    auto take = [&](size_t n) {
        size_t o = off;
        off = align_up(off + n, 64);
        return o;
    };
    const size_t R = (size_t)n_req, A = (size_t)n_adapters;
    L.seg_cap = n_adapters + 1;
    const size_t used_max = R < A ? R : A;
    L.ext_cap = (int32_t)(used_max * (size_t)(r_max / 8));
    L.staged = take(2 * R + A);
    L.tok_off = take(R + 1);
    L.req_dst = take(R);
    L.hist = take(A + 1);
    L.cursor = take(A + 1);
    L.key_seg = take(A + 1);
    L.perm = take((size_t)T);
    L.row_seg = take((size_t)T);
    L.row_adapter = take((size_t)T);
    L.row_ext = take((size_t)T);
    L.seg_adapter = take((size_t)L.seg_cap);
    L.seg_indptr = take((size_t)L.seg_cap + 1);
    L.seg_rank = take((size_t)L.seg_cap);
    L.seg_ext = take((size_t)L.seg_cap + 1);
    L.seg_unit = take((size_t)L.seg_cap + 1);
    // (room for either unit size, and for the shrink grid, padded to eight units, to read the records of its padding)
    L.unit_rec = take(((size_t)T / kShrinkRowsSmall + (size_t)L.seg_cap + 8) * 4);
    L.ext_rec = take((size_t)L.ext_cap * 4);
    L.scalars = take(8);
    L.total_bytes = off * sizeof(int32_t);
    return L;
}

int validate_batch(const int32_t *req_adapter, const int32_t *req_ntok, int32_t n_req, const int32_t *adapter_rank,
                   int32_t n_adapters, int32_t r_max, int64_t T_expected, int32_t *n_seg_out, int64_t *ext_total_out) {
    if (!plan_sizes_ok(n_req, T_expected, n_adapters, r_max)) return LORA_ERR_INVALID_ARG;
    if (n_req > 0 && (!req_adapter || !req_ntok)) return LORA_ERR_INVALID_ARG;
    if (n_adapters > 0 && !adapter_rank) return LORA_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n_req; ++i)
        if (req_adapter[i] < -1 || req_adapter[i] >= n_adapters) return LORA_ERR_BAD_ADAPTER_ID;
    int64_t sum = 0;
    for (int32_t i = 0; i < n_req; ++i) {
        if (req_ntok[i] < 0) return LORA_ERR_LENGTH_MISMATCH;
        sum += req_ntok[i];
    }
    if (sum != T_expected) return LORA_ERR_LENGTH_MISMATCH;
    // used adapters: O(R) marks in a bitmap on the stack-free heap (n_adapters <= 65536 -> 8 KiB)
    const size_t words = ((size_t)n_adapters + 1 + 63) / 64;
    uint64_t *used = new (std::nothrow) uint64_t[words ? words : 1]();
    if (!used) return LORA_ERR_INVALID_ARG;
    bool any_none = false;
    for (int32_t i = 0; i < n_req; ++i) {
        if (req_ntok[i] == 0) continue;
        if (req_adapter[i] < 0)
            any_none = true;
        else
            used[req_adapter[i] >> 6] |= 1ull << (req_adapter[i] & 63);
    }
    int rc = LORA_OK;
    int32_t n_seg = any_none ? 1 : 0;
    int64_t ext = 0;
    for (size_t w = 0; w < words && rc == LORA_OK; ++w)
        for (uint64_t m = used[w]; m != 0 && rc == LORA_OK; m &= m - 1) {
            const int32_t r = adapter_rank[w * 64 + (size_t)__builtin_ctzll(m)];
            if (r <= 0)
                rc = LORA_ERR_ADAPTER_NOT_RESIDENT;
            else if (r & 7)
                rc = LORA_ERR_SHAPE;
            else if (r > r_max)
                rc = LORA_ERR_RANK_TOO_LARGE;
            ++n_seg;
            ext += r;
        }
    delete[] used;
    if (rc != LORA_OK) return rc;
    if (n_seg_out) *n_seg_out = n_seg;
    if (ext_total_out) *ext_total_out = ext;
    return LORA_OK;
}

PlanBuildArgs plan_args(const lora_ctx *ctx, const int32_t *req_adapter_dev, const int32_t *req_ntok_dev, const int32_t *rank_dev,
                        int32_t n_req, int32_t n_adapters, int32_t r_max, int64_t T, const PlanLayout &L, int32_t *base) {
    PlanBuildArgs a;
    a.req_adapter = req_adapter_dev;
    a.req_ntok = req_ntok_dev;
    a.rank = rank_dev;
    a.n_req = n_req;
    a.n_adapters = n_adapters;
    a.r_max = r_max;
    a.T = (int32_t)T;
    a.seg_cap = L.seg_cap;
    a.ext_cap = L.ext_cap;
    // Work units of 16 rows while that keeps their number within one workgroup per CU (decode batches, small mixed
    // batches: the long segments then spread over the chip instead of holding a few CUs four times as long), of 64
    // rows otherwise (a unit of 64 rows reads its adapter once for four times the rows).
    const int64_t seg_bound = std::min<int64_t>(std::min<int64_t>(n_req, n_adapters), T);
    const bool small_units = T / kShrinkRowsSmall + seg_bound <= (int64_t)ctx->num_cu;
    a.unit_rows = small_units ? kShrinkRowsSmall : kShrinkRows;
    a.unit_shift = small_units ? 4 : 6;
    a.tok_off = base + L.tok_off;
    a.req_dst = base + L.req_dst;
    a.hist = base + L.hist;
    a.cursor = base + L.cursor;
    a.key_seg = base + L.key_seg;
    a.perm = base + L.perm;
    a.row_seg = base + L.row_seg;
    a.row_adapter = base + L.row_adapter;
    a.row_ext = base + L.row_ext;
    a.seg_adapter = base + L.seg_adapter;
    a.seg_indptr = base + L.seg_indptr;
    a.seg_rank = base + L.seg_rank;
    a.seg_ext = base + L.seg_ext;
    a.seg_unit = base + L.seg_unit;
    a.unit_rec = base + L.unit_rec;
    a.ext_rec = base + L.ext_rec;
    a.scalars = base + L.scalars;
    return a;
}

void fill_plan(const PlanBuildArgs &a, lora_plan_t *out) {
    out->T = a.T;
    out->n_req = a.n_req;
    out->n_adapters = a.n_adapters;
    out->r_max = a.r_max;
    out->seg_cap = a.seg_cap;
    out->ext_cap = a.ext_cap;
    out->magic = kPlanMagic;
    out->unit_rows = a.unit_rows;
    out->perm = a.perm;
    out->row_seg = a.row_seg;
    out->row_adapter = a.row_adapter;
    out->row_ext = a.row_ext;
    out->seg_adapter = a.seg_adapter;
    out->seg_indptr = a.seg_indptr;
    out->seg_rank = a.seg_rank;
    out->seg_ext = a.seg_ext;
    out->seg_unit = a.seg_unit;
    out->unit_rec = a.unit_rec;
    out->ext_rec = a.ext_rec;
    out->tok_off = a.tok_off;
    out->scalars = a.scalars;
}

int build_plan(lora_ctx *ctx, const PlanBuildArgs &a, hipStream_t stream, lora_plan_t *out) {
    // One workgroup builds the whole plan (per-row arrays included) up to 4096 rows, up to 8192 for batches of at
    // most 64 requests (the one-lane-per-request kernel leaves its workgroup more time for the rows); beyond that
    // the per-row arrays are filled by a second, grid-wide kernel.
    const int fused_rows = ctx->opt_plan_fused_rows >= 0 ? ctx->opt_plan_fused_rows : (a.n_req <= 64 ? 8192 : 4096);
    const bool fuse = a.T <= fused_rows && a.ext_cap <= 8192;
    KernelTimer timers[2];
    const bool timed = next_timer(ctx, kProfPlanSegments, &timers[0]) && (fuse || next_timer(ctx, kProfPlanFill, &timers[1]));
    LORA_HIP(launch_plan_build(a, fuse, ctx->opt_plan_variant > 0 ? ctx->opt_plan_variant : 0, stream, timed ? timers : nullptr));

    fill_plan(a, out);
    return LORA_OK;
}

// Request- and segment-level quantities of a validated batch, in the order of PlanTable: a counting sort by adapter that looks
// only at the slots in use, as the validation does (64 requests, 65536 slots: 45 us of
// host time with a pass over every slot in each of the two walks).
void build_table(const int32_t *req_adapter, const int32_t *req_ntok, const int32_t *adapter_rank, int32_t n_adapters, const PlanBuildArgs &a,
                 KeyScratch *keys, int32_t *out, PlanTable *t) {
    const int R = a.n_req;
    int32_t *rows = keys->rows, *seg = keys->seg;
    const int words = (n_adapters + 63) / 64;
    memset(keys->used, 0, sizeof(uint64_t) * (size_t)words);
    rows[n_adapters] = 0;  // (key n_adapters: requests without an adapter)
    for (int i = 0; i < R; ++i) {
        const int k = req_adapter[i], n = req_ntok[i];
        if (n == 0) continue;
        if (k < 0) {
            rows[n_adapters] += n;
            continue;
        }
        const uint64_t bit = 1ull << (k & 63);
        if (!(keys->used[k >> 6] & bit)) rows[k] = 0;
        keys->used[k >> 6] |= bit;
        rows[k] += n;
    }
    int32_t *sad = out + t->sad(), *sip = out + t->sip(), *srk = out + t->srk(), *sex = out + t->sex(), *sun = out + t->sun();
    int s = 0, slot = 0, ext = 0, units = 0;
    auto segment = [&](int k, int adapter, int rank, int n_units) {
        sad[s] = adapter;
        sip[s] = slot;
        srk[s] = rank;
        sex[s] = ext;
        sun[s] = units;
        seg[k] = s;
        ext += rank;
        units += n_units;
        const int n = rows[k];
        rows[k] = slot;  // from here on: the key's running slot
        slot += n;
        ++s;
    };
    for (int w = 0; w < words; ++w)
        for (uint64_t m = keys->used[w]; m != 0; m &= m - 1) {
            const int k = w * 64 + __builtin_ctzll(m);
            segment(k, k, adapter_rank[k], (rows[k] + a.unit_rows - 1) >> a.unit_shift);
        }
    if (rows[n_adapters] > 0) segment(n_adapters, -1, 0, 0);
    sip[s] = slot;
    sex[s] = ext;
    sun[s] = units;
    int32_t *tok = out + t->tok(), *dst = out + t->dst(), *rseg = out + t->rseg();
    int row = 0;
    for (int i = 0; i < R; ++i) {
        const int k = req_adapter[i] < 0 ? n_adapters : req_adapter[i];
        const int n = req_ntok[i];
        tok[i] = row;
        row += n;
        dst[i] = n > 0 ? rows[k] : 0;
        rseg[i] = n > 0 ? seg[k] : 0;  // (a request without rows has no segment; nothing looks its entries up)
        if (n > 0) rows[k] += n;
    }
    tok[R] = row;
    t->ext_total = ext;
    t->n_units = units;
}

// Most time lora_plan() waits for a table: several times what the layers of most plans take on the GPU, so that a host that
// runs ahead of it finds one.  Past that the upload takes over, whose events the runtime can report errors on.
constexpr auto kTableWait = std::chrono::milliseconds(20);

bool table_free(const lora_ctx *ctx, int i) { return __atomic_load_n(ctx->table_done + i, __ATOMIC_ACQUIRE) == ctx->table_ticket[i]; }

// A slot whose last table has been read, the next one in turn if possible; -1 if there is none within the time above.
int take_table(const lora_ctx *ctx) {
    const auto t0 = std::chrono::steady_clock::now();
    for (;;) {
        for (int k = 0; k < kTableSlots; ++k) {
            const int i = (ctx->table_next + k) % kTableSlots;
            if (table_free(ctx, i)) return i;
        }
        const auto waited = std::chrono::steady_clock::now() - t0;
        if (waited >= kTableWait) return -1;
        if (waited < std::chrono::milliseconds(1))
            std::this_thread::yield();
        else
            std::this_thread::sleep_for(std::chrono::microseconds(50));
    }
}

int check_plan_buf(const void *plan_buf, size_t plan_buf_bytes, const PlanLayout &L, lora_plan_t *out) {
    if (!out) return LORA_ERR_INVALID_ARG;
    if (!plan_buf) return LORA_ERR_INVALID_ARG;
    if (((uintptr_t)plan_buf & 255u) != 0) return LORA_ERR_ALIGNMENT;
    if (plan_buf_bytes < L.total_bytes) return LORA_ERR_WORKSPACE_TOO_SMALL;
    return LORA_OK;
}

// ---- kernel selection ---------------------------------------------------------------------------------
// Blocks of exactly as many 16-row pieces as the batch has: padding costs partial tiles written and read, MFMAs and LDS.
int decode_tblk(int64_t T) { return T <= 16 ? 1 : (int)((T + 15) / 16); }

struct GemmChoice {
    int variant;
    int tblk;   // decode path only: 16-row blocks of the batch
    int waves;  // decode path only: waves (16-row weight blocks) per workgroup of the streaming kernel
};

// Geometry of the decode path's launches and workspace: blocks of 16 weight rows (extension rows first, by an upper
// bound of how many ranks the batch can use), slices of 512 along K.
struct DecodeGeom {
    int tblk, nbw, nbe_cap, ks;
    size_t p_bytes;
};
DecodeGeom decode_geom(int64_t T, int32_t K, int32_t N, int64_t ext_rows_bound) {
    DecodeGeom g;
    g.tblk = decode_tblk(T);
    g.nbw = (N + 15) / 16;
    g.nbe_cap = (int)((ext_rows_bound + 15) / 16);
    g.ks = (K / 8 + 63) / 64;
    g.p_bytes = (size_t)(g.nbe_cap + g.nbw) * (size_t)g.ks * (size_t)g.tblk * 1024;
    return g;
}

// A decode-sized batch takes the decode path unless the tiled GEMM is clearly cheaper: towards 128 rows and wide
// outputs the partial tiles of the K slices (T x N x 4 bytes per slice, written and read) outgrow the weights.
// Both sides are fits to measured layer times in microseconds (bf16, with adapters): the decode path moves its bytes
// at ~3.6 TB/s behind ~8 us of fixed cost; the tiled path (64x64 tiles, shrink and expand launches ~15 us) is bound
// by its chain of K stages or by the weights at ~3 TB/s.  The fit is older than the kernels for odd numbers of blocks and
// counts rows by pairs of blocks, as those it was made on did; today it errs towards tiles by up to 6 us at a few sizes:
// 4096 -> 11008: decode up to 96 rows (45 vs 52 us), tiled from 97 (52 vs 47; 54.6 vs 55.6 at 128); 5120 -> 13824: tiled from 65
// rows (63 vs 57; 64 vs 60 at 72, even at 80, 74 vs 86 at 128); 4096 -> 4096 and 11008 -> 4096: decode throughout (23 vs 37 us,
// 53 vs 84 us at 128 rows).
bool decode_path_cheaper(int64_t T, int32_t K, int32_t N) {
    const double w_mb = 2.0e-6 * (double)K * (double)N;
    const int tblk = T <= 32 ? decode_tblk(T) : 2 * (int)((T + 31) / 32);  // (the fit's own measure of the rows)
    const double p_mb = 1.024e-3 * (double)((N + 15) / 16) * (double)((K / 8 + 63) / 64) * (double)tblk;
    const double t_decode = 8.0 + (w_mb + 2.0 * p_mb) / 3.6;
    const double t_tiled = 15.0 + std::max(29.0 * (double)K / 4096.0, w_mb / 3.0 + 6.0);
    return t_decode <= 1.08 * t_tiled;
}

// (ns / n_sets: the output widths of the projections one tiled launch covers; the decode path is chosen per projection,
// with n_sets == 1, and covers several projections with its own launches)
GemmChoice choose_gemm_sets(const lora_ctx *ctx, int64_t T, int32_t K, const int32_t *ns, int n_sets, int32_t dtype) {
    GemmChoice c{kGemmTile128x128, 0, kDecodeMinWaves};
    const int max_rows = ctx && ctx->opt_decode_max_rows >= 0 ? ctx->opt_decode_max_rows : kDecodeMaxRows;
    int forced = ctx ? ctx->opt_gemm_variant : -1;
    const bool fits = dtype == LORA_DTYPE_BF16 && T <= kDecodeMaxRows && n_sets == 1;
    if (forced == kGemmDecode && !fits) forced = -1;
    const bool decode = forced == kGemmDecode || (forced < 0 && fits && T <= max_rows && decode_path_cheaper(T, K, ns[0]));
    if (decode) {
        c.variant = kGemmDecode;
        c.tblk = decode_tblk(T);
        // (waves per workgroup of the streaming kernel: chosen at launch, when the plan's bound of extension rows is known)
        return c;
    }
    if (forced >= 0 && forced != kGemmDecode) {
        c.variant = forced;
        return c;
    }
    const int cus = ctx ? ctx->num_cu : 256;
    // (192x128: 1500 rows on 4096 -> 4096 in fp32 481 -> 368 us per layer, in bf16 65 -> 62; 1300 rows on 5120 -> 13824 221 -> 205)
    // Time model: rounds of one tile per CU, a tile costing its area over its MFMA efficiency.  The efficiencies are those of the
    // kernel that staged its tiles through registers (us per round at K = 4096: 256x256 104, 256x224 100, 256x192 88, 256x128 64, 128x192
    // 51, 128x128 34), and choices that were measured against each other rest on them.  They are not what a round takes now -- bf16,
    // K = 4096: 256x256 97.9, 256x224 87.4, 256x192 75.7, 256x128 55.1, 128x192 43.7, 192x128 43.6, 128x128 32.6, 64x64 20.3, area per time
    // relative to 256x256 0.98, 0.97, 0.89, 0.84, 0.84, 0.75, 0.30; K = 1024: 0.98, 0.97, 0.85, 0.78, 0.79, 0.71, 0.33; K = 11008: 0.99,
    // 0.97, 0.90, 0.86, 0.86, 0.78, 0.31; fp32: 1.00 to 0.97, 64x64 0.91 -- and the model knows no start and end of a tile.
    // Of 128x128 against 256x192, the pair where that cost most, 24 shapes in which the two are close by this table, 128x128 over
    // 256x192: K = 2048 0.88 to 0.97; 3072 0.96 to 1.00, and 1.13 to 1.23 with N = 22016; 3584 0.96 to 1.01, 1.13 to 1.26; 4096 0.97 to 1.03,
    // 1.07 to 1.19; 5120 1.02 to 1.31; 8192 1.01 to 1.22; 11008 1.15 to 1.36.  So from K = 4096 on 128x128 counts 0.72 instead of 0.77, which
    // takes 256x192 there.  At 0.68 it would also give way to 128x192, which loses (556 rows 4096 -> 22016: 125 us and 133).
    const double eff128 = dtype == LORA_DTYPE_BF16 && K >= 4096 ? 0.72 : 0.77;
    struct Cand {
        int variant, bm, bn;
        double eff;
    };
    const Cand cands[] = {{kGemmTile256x256w4, 256, 256, 1.00},
                          {kGemmTile256x128, 256, 128, 0.81},
                          {kGemmTile256x224, 256, 224, 0.905},
                          {kGemmTile256x192, 256, 192, 0.89},
                          {kGemmTile128x192, 128, 192, 0.77},
                          {kGemmTile192x128, 192, 128, 0.77},
                          {kGemmTile128x128, 128, 128, eff128},
                          {kGemmTile64x64, 64, 64, 0.45}};
    double best = 0.0;
    bool have = false;
    for (const Cand &cd : cands) {
        int64_t tiles_n = 0;
        for (int i = 0; i < n_sets; ++i) tiles_n += (ns[i] + cd.bn - 1) / cd.bn;
        const int64_t tiles = ((T + cd.bm - 1) / cd.bm) * tiles_n;
        const int64_t rounds = (tiles + cus - 1) / cus;
        const double cost = (double)rounds * cd.bm * cd.bn / cd.eff;
        if (!have || cost < best) {
            best = cost;
            have = true;
            c.variant = cd.variant;
        }
    }
    return c;
}

GemmChoice choose_gemm(const lora_ctx *ctx, int64_t T, int32_t K, int32_t N, int32_t dtype) {
    return choose_gemm_sets(ctx, T, K, &N, 1, dtype);
}

struct WorkspaceLayout {
    size_t v_off, p_off, p_bytes, total;          // total: what every call needs
    size_t d_off, d_bytes, ldd, total_preferred;  // fp32 adapter term of the separate expand kernel (optional)
    size_t sk_off, sk_bytes;                      // partial outputs of a GEMM split along K (optional, inside total_preferred)
};

// Batches whose tiles alone would leave most CUs idle: the tiled GEMM is split along K as well, its fp32 partial
// outputs summed by a second launch.  Depends on the shape alone (the workspace is sized from it).
struct SplitK {
    int s, k_chunk, variant;
};
// (room: bytes for the partial outputs.  A workspace kept for another shape may have room for some: fewer stretches still beat
// none when K is long -- 13824 -> 5120, 160 rows: 64 us per layer with six, 66 with five, 73 with three, 109 unsplit; 11008 -> 4096, 300
// rows: 77 with two, 99 unsplit -- and lose below 8192 -- 4096 -> 4096, 256 rows: 37-39 with three and two, 32 unsplit)
SplitK choose_split_k(int64_t T, int32_t K, int32_t N, int32_t dtype, size_t room = SIZE_MAX) {
    SplitK r{1, 0, kGemmTile128x128};
    if (T <= kDecodeMaxRows) return r;  // (the decode path, or a batch too small to matter)
    const int stage = dtype == LORA_DTYPE_BF16 ? 64 : 32;
    const size_t one = (size_t)T * align_up((size_t)N, 8) * sizeof(float);  // bytes of one partial output
    int64_t s = 0;
    if (T <= 1024 && dtype == LORA_DTYPE_BF16) {
        // Mid-sized batches.  As many stretches of K as fit one round of at most one workgroup per CU, on 128x128 or on
        // 192x128 tiles: with one and a half workgroups per CU (the earlier rule) half the CUs worked twice as long as the
        // rest (11008 -> 4096, 384 rows: 4 x 96 workgroups of 128x128 88 us per layer, 2 x 96 of them 86, 4 x 64 of 192x128
        // 75; 160 rows: 61 -> 52 with 8 x 32 of 192x128; 13824 -> 5120, 450 rows: 145 unsplit, 110 with 2 x 120 of 192x128).
        // The choice between the two is a fit to such layer times: a stage of K costs 0.36 us on 128x128 and 0.45 on
        // 192x128 tiles, the partial outputs are written and read at ~5 TB/s.  Short contraction axes take 192x128 tiles
        // up to 384 rows only (4096 -> 4096: 700 rows 52 -> 55 us, 450 rows even; 4096 -> 11008: 160 rows 60 -> 55), and
        // below 4096 none (2048 -> 6000, 333 rows: 38 -> 41).
        double best = 0.0;
        for (int v = 0; v < 2; ++v) {
            const int bm = v ? 192 : 128;
            if (v && (K < 4096 || (K < 8192 && T > 384))) continue;
            const int64_t tiles = ((T + bm - 1) / bm) * (((int64_t)N + 127) / 128);
            if (tiles > 96 && K < 4096) continue;
            int64_t sv = std::min<int64_t>(std::min<int64_t>(256 / tiles, 8), K / (16 * stage));  // (256: the part's CUs)
            if (K >= 8192) sv = std::min<int64_t>(sv, (int64_t)std::min<size_t>(room / one, 8));
            if (sv < 2) continue;
            const double cost = (v ? 0.45 : 0.36) * (double)((K / stage + sv - 1) / sv) + (double)sv * (double)T * (double)N * 1.6e-6;
            if (s < 2 || cost < best) {
                best = cost;
                s = sv;
                r.variant = v ? kGemmTile192x128 : kGemmTile128x128;
            }
        }
    } else if (T <= 1024) {
        // The same in fp32, on 128x128 tiles, while the tiles alone leave most of the chip idle.
        const int64_t tiles = ((T + 127) / 128) * (((int64_t)N + 127) / 128);
        if (tiles > 128 || (tiles > 96 && K < 8192)) return r;
        s = (384 + tiles - 1) / tiles;  // about one and a half workgroups per CU (two of them fit one)
    } else {
        // A long contraction axis into few columns (a down projection at a thousand-odd rows): 256x256 tiles, as many
        // stretches of K as make one round of workgroups.  Measured per layer, 11008 -> 4096: 1100 rows 169 -> 154 us,
        // 1216 rows 171 -> 157; with two stretches (1536 and 2048 rows: 192 -> 190, 198 -> 218) and at 8192 -> 4096 (three
        // stretches, 1216 rows: 130 -> 130) the partial outputs cost what the idle CUs did, or more.
        const int64_t tiles = ((T + 255) / 256) * (((int64_t)N + 255) / 256);
        if (tiles > 85 || K < 10240) return r;
        s = 256 / tiles;  // (the part's 256 CUs: the workspace size must not depend on the context)
        r.variant = kGemmTile256x256w4;
    }
    s = std::min<int64_t>(s, 8);
    s = std::min<int64_t>(s, K / (16 * stage));  // at least 16 stages per split
    if (s < 2) return SplitK{1, 0, kGemmTile128x128};
    r.k_chunk = (int)(((K + s - 1) / s + stage - 1) / stage * stage);
    r.s = (K + r.k_chunk - 1) / r.k_chunk;
    if (r.s < 2 || (size_t)r.s * one > room) r = SplitK{1, 0, kGemmTile128x128};
    return r;
}

WorkspaceLayout workspace_layout(int64_t T, int32_t K, int32_t N, int32_t r_max, int32_t dtype) {
    WorkspaceLayout w;
    const size_t es = dtype == LORA_DTYPE_BF16 ? 2 : 4;
    w.v_off = 0;
    size_t off = align_up((size_t)T * (size_t)r_max * es, 256);
    // decode-sized bf16 batches: the partial tiles of the K slices (any batch of T rows uses at most T * r_max ranks)
    w.p_off = off;
    w.p_bytes = (dtype == LORA_DTYPE_BF16 && T > 0 && T <= kDecodeMaxRows) ? decode_geom(T, K, N, T * (int64_t)r_max).p_bytes : 0;
    off = align_up(off + w.p_bytes, 256);
    w.total = off < 256 ? 256 : off;
    w.ldd = align_up((size_t)N, 8);  // (the GEMM's epilogue reads whole 8-column pieces of a row)
    w.d_off = w.total;
    // (also for decode-sized bf16 batches, whose wide outputs may take the tiled path)
    w.d_bytes = (T > kDecodeMaxRows || (dtype == LORA_DTYPE_BF16 && T > 0)) ? (size_t)T * w.ldd * sizeof(float) : 0;
    w.sk_off = align_up(w.d_off + w.d_bytes, 256);
    const SplitK sk = choose_split_k(T, K, N, dtype);
    w.sk_bytes = sk.s > 1 ? (size_t)sk.s * (size_t)T * w.ldd * sizeof(float) : 0;
    w.total_preferred = align_up(w.sk_off + w.sk_bytes, 256);
    return w;
}

// (check_ws = false: the entry point that brings its own workspace; d->workspace is then not looked at)
int check_linear(const lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *d, bool need_ctx = true, bool check_ws = true) {
    if (!plan || !d) return LORA_ERR_INVALID_ARG;
    if (plan->magic != kPlanMagic || plan->T < 0 || !plan->scalars) return LORA_ERR_PLAN;
    if (plan->unit_rows != kShrinkRows && plan->unit_rows != kShrinkRowsSmall) return LORA_ERR_PLAN;
    if (d->dtype != LORA_DTYPE_BF16 && d->dtype != LORA_DTYPE_F32) return LORA_ERR_INVALID_ARG;
    if (d->flags != 0) return LORA_ERR_INVALID_ARG;
    const int ce = d->dtype == LORA_DTYPE_BF16 ? 8 : 4;
    if (d->K <= 0 || d->N <= 0 || (d->K & 7) != 0) return LORA_ERR_SHAPE;
    if (d->ldx < d->K || d->ldw < d->K || d->ldy < d->N) return LORA_ERR_SHAPE;
    if (d->ldx % ce || d->ldw % ce || d->ldy % ce) return LORA_ERR_ALIGNMENT;
    // the tiled kernels address X with 32-bit byte offsets from its start, W0 from a tile's first row
    const int64_t es = d->dtype == LORA_DTYPE_BF16 ? 2 : 4;
    if (plan->T * d->ldx * es >= (1ll << 32) || 256 * d->ldw * es >= (1ll << 32)) return LORA_ERR_SHAPE;
    if (plan->T > 0) {
        if (!d->X || !d->W0 || !d->Y) return LORA_ERR_INVALID_ARG;
        if (((uintptr_t)d->X | (uintptr_t)d->W0 | (uintptr_t)d->Y) & 15u) return LORA_ERR_ALIGNMENT;
        // Y must not overlap X, W0 or the workspace (extents from the leading dimensions)
        const uintptr_t y0 = (uintptr_t)d->Y, y1 = y0 + (uintptr_t)(((plan->T - 1) * d->ldy + d->N) * es);
        const uintptr_t x0 = (uintptr_t)d->X, x1 = x0 + (uintptr_t)(((plan->T - 1) * d->ldx + d->K) * es);
        const uintptr_t w0 = (uintptr_t)d->W0, w1 = w0 + (uintptr_t)(((int64_t)(d->N - 1) * d->ldw + d->K) * es);
        if ((y0 < x1 && x0 < y1) || (y0 < w1 && w0 < y1)) return LORA_ERR_INVALID_ARG;
        if (check_ws && d->workspace) {
            const uintptr_t s0 = (uintptr_t)d->workspace, s1 = s0 + d->workspace_bytes;
            if ((s0 < y1 && y0 < s1) || (s0 < x1 && x0 < s1) || (s0 < w1 && w0 < s1)) return LORA_ERR_INVALID_ARG;
        }
    }
    if (d->tbl) {
        if (d->tbl->n_adapters < plan->n_adapters) return LORA_ERR_INVALID_ARG;
        if (plan->n_adapters > 0 && (!d->tbl->A || !d->tbl->B || !d->tbl->scale)) return LORA_ERR_INVALID_ARG;
    }
    const WorkspaceLayout w = workspace_layout(plan->T, d->K, d->N, plan->r_max, d->dtype);
    if (plan->T > 0 && check_ws) {
        if (!d->workspace) return LORA_ERR_INVALID_ARG;
        if ((uintptr_t)d->workspace & 255u) return LORA_ERR_ALIGNMENT;
        if (d->workspace_bytes < w.total) return LORA_ERR_WORKSPACE_TOO_SMALL;
    }
    if (need_ctx && !ctx) return LORA_ERR_INVALID_ARG;  // last, so that the checks above run on a GPU-less host too
    return LORA_OK;
}

PlanView view_of(const lora_plan_t *plan) {
    PlanView v;
    v.perm = plan->perm;
    v.row_seg = plan->row_seg;
    v.row_adapter = plan->row_adapter;
    v.row_ext = plan->row_ext;
    v.seg_adapter = plan->seg_adapter;
    v.seg_indptr = plan->seg_indptr;
    v.seg_rank = plan->seg_rank;
    v.seg_ext = plan->seg_ext;
    v.seg_unit = plan->seg_unit;
    v.unit_rec = plan->unit_rec;
    v.ext_rec = plan->ext_rec;
    v.scalars = plan->scalars;
    return v;
}

bool has_adapters(const lora_plan_t *plan, const lora_linear_desc *d) {
    return d->tbl != nullptr && plan->n_adapters > 0 && plan->r_max > 0;
}

// Whether work on the stream is being captured; yes also where the runtime does not say (the legacy stream, for one, while a stream
// that synchronises with it is captured): the calls then do what is right under capture, and report what HIP says to that.
bool is_capturing(hipStream_t stream) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// What the launches' grids have room for: work units -- sum over the adapter segments of ceil(rows / unit_rows) -- and ranks in
// use, each by an upper bound.  Under stream capture it holds for every batch of the plan's sizes, because a captured launch may
// be replayed after plan_buf has been filled for another one.  Nothing but grids, and what they imply for the shape of the
// shrink's workgroups, depends on these bounds, and no result does: workspace offsets follow the sizes alone, a captured stage
// may follow an eager one, and V's sums are cut the same way in every shape.  An eager launch is for this plan, of which
// lora_plan() knows what it uses: no surplus workgroups (73 requests, a 7B decoder layer, 100 slots of up to rank 64: 237 -> 229 us).
struct PlanBounds {
    int64_t units, ext_rows;
};
PlanBounds bounds_of(const lora_plan_t *plan, hipStream_t stream) {
    int64_t segs = std::min<int64_t>(std::min<int64_t>(plan->n_adapters, plan->n_req), plan->T);
    int64_t ext_rows = segs * plan->r_max;
    if ((plan->seg_cap < segs || 8 * (int64_t)plan->ext_cap < ext_rows) && !is_capturing(stream)) {
        segs = std::min<int64_t>(segs, plan->seg_cap);
        ext_rows = std::min<int64_t>(ext_rows, 8 * (int64_t)plan->ext_cap);
    }
    return PlanBounds{plan->T / plan->unit_rows + segs, ext_rows};
}

// Decode path: when the reduction's own expand -- every row gathers its adapter's B_a for the workgroup's 16 columns,
// and every workgroup re-reduces V -- would move more than ~24 MB through 16-byte gathers (T x r_max x N x 2 bytes:
// 8 MB at 64 rows of rank 16 and 4096 columns), the second launch is the finishing kernel, which streams each used B_a
// once, unit by unit.  It rounds V to bf16, so it is for calls with a workspace of the preferred size only, as V in bf16 is
// everywhere: with less, V stays in fp32 (64 rows on 64 adapters of rank 128, 4096 -> 4096: 55 us against 39).
bool decode_adapters_heavy(const lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *d) {
    if (!has_adapters(plan, d)) return false;
    if (plan->unit_rows > kShrinkRowsSmall) return false;  // (does not happen at decode sizes)
    if (d->workspace_bytes < workspace_layout(plan->T, d->K, d->N, plan->r_max, d->dtype).total_preferred) return false;
    if (ctx->opt_expand_split == 0) return false;
    if (ctx->opt_expand_split == 1) return true;
    return 2.0e-6 * (double)plan->T * (double)plan->r_max * (double)d->N > 24.0;
}

// The two launches of the decode path share one argument block.  n > 1: several projections of the same X, their
// blocks of weight rows side by side in the first launch's grid and their column blocks in the second's.
DecodeArgs decode_args(const lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *const *descs, int n,
                       const GemmChoice &c) {
    const lora_linear_desc *d = descs[0];
    bool any_ad = false;
    for (int i = 0; i < n; ++i) any_ad = any_ad || has_adapters(plan, descs[i]);
    // ranks that a batch of these sizes can use at most: one adapter per request, per slot, per row
    const int64_t segs = std::min<int64_t>(std::min<int64_t>(plan->n_req, plan->n_adapters), plan->T);
    DecodeArgs a;
    a.plan = view_of(plan);
    a.X = d->X;
    a.ldx = d->ldx;
    a.T = (int32_t)plan->T;
    a.K = d->K;
    a.r_max = plan->r_max;
    a.n_sets = n > 1 ? n : 0;
    long nblk = 0;
    for (int i = 0; i < n; ++i) {
        const lora_linear_desc *di = descs[i];
        const WorkspaceLayout w = workspace_layout(plan->T, di->K, di->N, plan->r_max, di->dtype);
        const DecodeGeom g = decode_geom(plan->T, di->K, di->N, any_ad ? segs * plan->r_max : 0);
        const bool ad = has_adapters(plan, di);
        DecodeSet &st = a.set[i];
        st.W = di->W0;
        st.ldw = di->ldw;
        st.A = ad ? di->tbl->A : nullptr;
        st.B = ad ? di->tbl->B : nullptr;
        st.scale = ad ? di->tbl->scale : nullptr;
        st.Y = di->Y;
        st.ldy = di->ldy;
        st.P = reinterpret_cast<float *>(static_cast<unsigned char *>(di->workspace) + w.p_off);
        st.N = di->N;
        st.nbw = g.nbw;
        st.n_adapters = ad ? di->tbl->n_adapters : 0;
        st.blk0 = st.cb0 = st.fb0 = 0;
        a.nbe_cap = g.nbe_cap;
        a.nbe = any_ad ? (int32_t)((pb.ext_rows + 15) / 16) : 0;
        a.ks = g.ks;
        nblk += (long)a.nbe + g.nbw;
    }
    const DecodeSet &s0 = a.set[0];  // (one projection: the launch's own fields)
    a.W = s0.W;
    a.ldw = s0.ldw;
    a.A = s0.A;
    a.B = s0.B;
    a.scale = s0.scale;
    a.Y = s0.Y;
    a.ldy = s0.ldy;
    a.P = s0.P;
    a.N = s0.N;
    a.nbw = s0.nbw;
    a.n_adapters = s0.n_adapters;
    // waves per workgroup: whole rounds of one workgroup per CU, as little of the last round idle as possible
    const int maxw = kDecodeMaxWaves;
    long best = -1;
    a.waves = kDecodeMinWaves;
    for (int w = maxw; w >= kDecodeMinWaves; --w) {
        const long wgs = ((nblk + w - 1) / w) * a.ks;
        const long cost = ((wgs + ctx->num_cu - 1) / ctx->num_cu) * w;
        if (best < 0 || cost < best) {
            best = cost;
            a.waves = w;
        }
    }
    if (ctx->opt_decode_waves >= kDecodeMinWaves && ctx->opt_decode_waves <= maxw) a.waves = ctx->opt_decode_waves;
    return a;
}

// The second launch of the decode path: sums the slices, adds V B_a, stores Y.  Projections with much adapter work go
// through the finishing kernel, the others through the reduction: one launch of each at most.
int do_decode_second(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *const *descs, int n,
                     const DecodeArgs &a, const GemmChoice &c, hipStream_t stream) {
    DecodeArgs part[2] = {a, a};  // [0] reduction, [1] finishing kernel
    int cnt[2] = {0, 0};
    for (int i = 0; i < n; ++i) {
        const int k = decode_adapters_heavy(ctx, plan, descs[i]) ? 1 : 0;
        part[k].set[cnt[k]++] = a.set[i];
    }
    for (int k = 0; k < 2; ++k) {
        if (cnt[k] == 0) continue;
        part[k].n_sets = n > 1 ? cnt[k] : 0;
        KernelTimer timer;
        const bool timed = next_timer(ctx, kProfGemm, &timer);
        if (k == 0)
            LORA_HIP(launch_decode_reduce(part[k], c.tblk, stream, timed ? &timer : nullptr));
        else
            LORA_HIP(launch_decode_finish(part[k], c.tblk, (int)pb.units, stream, timed ? &timer : nullptr));
    }
    return LORA_OK;
}

int do_decode(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *const *descs, int n,
              const GemmChoice &c, hipStream_t stream) {
    const DecodeArgs a = decode_args(ctx, plan, pb, descs, n, c);
    KernelTimer t1;
    const bool timed1 = next_timer(ctx, kProfShrink, &t1);
    LORA_HIP(launch_decode_stream(a, c.tblk, stream, timed1 ? &t1 : nullptr));  // streams W0 and the used A_a against X
    return do_decode_second(ctx, plan, pb, descs, n, a, c, stream);
}

// Whether lora_plan() made the plan: it leaves what the batch uses in the capacities, lora_plan_device what any batch could (one
// segment more than slots; every segment at r_max).  A host plan that uses every slot at full rank, with rows that have no adapter
// besides, looks like the latter: nothing but a choice between equals may hang on this.
bool built_by_host(const lora_plan_t *plan) {
    const int64_t segs = std::min<int64_t>(plan->n_adapters, plan->n_req);
    return plan->seg_cap <= plan->n_adapters || 8 * (int64_t)plan->ext_cap < segs * plan->r_max;
}

// (multi: several projections of the same X that go through one launch)
int do_shrink(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *d, hipStream_t stream,
              const lora_linear_desc *const *multi = nullptr, int n_multi = 0) {
    if (n_multi == 0) {
        const GemmChoice c = choose_gemm(ctx, plan->T, d->K, d->N, d->dtype);
        if (c.variant == kGemmDecode) {  // decode-sized: the first launch streams W0 and the used A_a against X
            KernelTimer timer;
            const bool timed = next_timer(ctx, kProfShrink, &timer);
            LORA_HIP(launch_decode_stream(decode_args(ctx, plan, pb, &d, 1, c), c.tblk, stream, timed ? &timer : nullptr));
            return LORA_OK;
        }
    }
    bool ad = has_adapters(plan, d);
    for (int i = 0; i < n_multi; ++i) ad = ad || has_adapters(plan, multi[i]);
    if (!ad) return LORA_OK;
    const WorkspaceLayout w = workspace_layout(plan->T, d->K, d->N, plan->r_max, d->dtype);
    unsigned char *ws = static_cast<unsigned char *>(d->workspace);
    ShrinkArgs a;
    a.plan = view_of(plan);
    a.X = d->X;
    a.ldx = d->ldx;
    a.K = d->K;
    a.T = (int32_t)plan->T;
    a.A = ad && n_multi == 0 ? d->tbl->A : nullptr;
    a.scale = ad && n_multi == 0 ? d->tbl->scale : nullptr;
    a.V = ws + w.v_off;
    a.r_max = plan->r_max;
    a.n_adapters = ad && n_multi == 0 ? d->tbl->n_adapters : 0;
    a.n_sets = n_multi;
    for (int i = 0; i < n_multi; ++i) {
        const lora_linear_desc *di = multi[i];
        const bool adi = has_adapters(plan, di);
        const WorkspaceLayout wi = workspace_layout(plan->T, di->K, di->N, plan->r_max, di->dtype);
        a.set[i].A = adi ? di->tbl->A : nullptr;
        a.set[i].scale = adi ? di->tbl->scale : nullptr;
        a.set[i].V = static_cast<unsigned char *>(di->workspace) + wi.v_off;
        a.set[i].n_adapters = adi ? di->tbl->n_adapters : 0;
        a.set[i].pad_ = 0;
    }
    a.max_units = ad ? (int32_t)pb.units : 0;
    // With few units (decode-sized batches) a unit's ranks are dealt to several workgroups: every A_a
    // is streamed once either way, and it takes most of the chip to stream them at HBM speed.
    const int64_t wide_groups = (plan->r_max + kShrinkRanks - 1) / kShrinkRanks;
    const int64_t mid_groups = (plan->r_max + 15) / 16;
    // (every rank block of a unit reads the unit's rows of X again: only worth it while X is small)
    const bool small_x = plan->T <= 256;
    // A unit of at most 16 rows reads little of X beside its ranks' rows of A_a, so its ranks are dealt out as finely as keeps
    // one workgroup per CU, the workgroups of all projections counted (365 rows on 14 adapters of rank 16 and 32, K = 11008: 32
    // workgroups, 23.4 us, as one block of 32 ranks, 15-16 us as blocks of 8; 700 rows on 16 adapters of rank 16, three
    // projections of 4096 -> 4096: the layer 110 us with 354 workgroups, two blocks of 8 ranks each, 105 with 177).
    int fine = 0;
    const int64_t unit_sets = (int64_t)a.max_units * std::max(n_multi, 1);
    if (plan->unit_rows == kShrinkRowsSmall)
        for (int rb = 32; rb >= 8 && unit_sets * (((int64_t)plan->r_max + rb - 1) / rb) <= (int64_t)ctx->num_cu; rb /= 2) fine = rb;
    int rank_block = !ad                                                  ? kShrinkRanks
                     : !small_x ? (fine > 0 ? fine : a.max_units * wide_groups < (int64_t)ctx->num_cu && plan->r_max > 32 ? 32 : kShrinkRanks)
                     : a.max_units * mid_groups < 2 * (int64_t)ctx->num_cu  ? 8
                     : a.max_units * wide_groups < 2 * (int64_t)ctx->num_cu ? 16
                                                                            : kShrinkRanks;
    if (ctx->opt_shrink_rank_block > 0) rank_block = ctx->opt_shrink_rank_block;
    a.rank_block = rank_block;
    a.rank_groups = ad ? (plan->r_max + rank_block - 1) / rank_block : 1;
    // Workgroups of four waves, two per CU, when there are more than that many: one's chain of dependent loads rides on the
    // other's stream (eight and four waves, us: three projections of 4096 -> 4096, 1216 rows, 100 adapters of rank 8 to 64, 1008
    // workgroups, 34.3 / 30.1; gate and up, 672, 24.2 / 20.0; three projections of K = 2048, 1000 one-row adapters, 93.3 / 72.1).
    // Fewer workgroups stay at eight waves: a unit's stream is what lasts then (336 workgroups, K = 4096: 13.5 us against 17.3).
    // So does K from 16 KB a row on, for the same reason (1000 one-row adapters, K in bf16: 4096 56.3 / 55.2, 5120 69.8 / 69.2, 7168
    // 89.8 / 91.1, 8192 97.8 / 102.2, 11008 134.6 / 139.8; 300 adapters, two projections, 8192 69.4 / 79.6, 11008 90.5 / 101.8), K with
    // less than one stage of 128 bytes for each of a unit's eight slices, launches with X staged in LDS (small batches: units of a
    // few rows), of which either kind fits a CU once, and plans built on the device, whose grids are for every slot (300 of
    // 1000 in use: 25.7 / 29.7).  (Under capture a host plan's grid is an upper bound as well; the shape has to follow it, so that a
    // captured launch is the one that a batch using all of it would get.)
    a.xlds_bytes = ad && plan->T <= 256 ? 64 * 1024 : 0;
    const int64_t row_bytes = (int64_t)d->K * (d->dtype == LORA_DTYPE_BF16 ? 2 : 4);
    a.waves = built_by_host(plan) && row_bytes >= 8 * 128 && row_bytes < 16 * 1024 && a.xlds_bytes == 0 &&
                      (int64_t)a.max_units * a.rank_groups * std::max(n_multi, 1) > 2 * (int64_t)ctx->num_cu
                  ? 4
                  : 8;
    KernelTimer timer;
    const bool timed = next_timer(ctx, kProfShrink, &timer);
    LORA_HIP(launch_shrink(a, d->dtype, stream, timed ? &timer : nullptr));
    return LORA_OK;
}

// The adapter term of one projection: fused into the GEMM, or -- batches of many small segments, where an M tile
// of the fused kernel would hold dozens of adapters, a few rows each -- computed per segment by a weight-streaming
// kernel of its own into the workspace (fp32), which is launched here, and added by the GEMM to its accumulators;
// the second only if the caller's workspace has the room.  Describes the projection for the GEMM in *out.
// (collect: several projections in one launch -- the expand kernel's arguments are gathered there, not launched)
// (all_in_d: the whole adapter term through the expand kernel -- the caller has checked the workspace -- for a GEMM
// that adds nothing itself)
int prepare_set(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *d, int variant, hipStream_t stream,
                const KernelTimer *expand_timer, GemmSet *out, bool *split_out, ExpandArgs *collect = nullptr,
                bool all_in_d = false) {
    const WorkspaceLayout w = workspace_layout(plan->T, d->K, d->N, plan->r_max, d->dtype);
    unsigned char *ws = static_cast<unsigned char *>(d->workspace);
    const bool ad = has_adapters(plan, d);
    GemmSet g{};
    g.W = d->W0;
    g.ldw = d->ldw;
    g.Y = d->Y;
    g.ldy = d->ldy;
    g.V = ad ? ws + w.v_off : nullptr;
    g.B = ad ? d->tbl->B : nullptr;
    g.N = d->N;
    bool split = false;
    if (ad && w.d_bytes > 0 && (all_in_d || d->workspace_bytes >= w.total_preferred)) {
        const int64_t segs = plan->n_adapters < plan->n_req ? plan->n_adapters : plan->n_req;  // upper bound
        split = segs > 0 && plan->T / segs < 64;
        if (ctx->opt_expand_split >= 0) split = ctx->opt_expand_split == 1;
        if (all_in_d) split = true;
    }
    if (split) {
        ExpandArgs e;
        e.plan = view_of(plan);
        e.V = ws + w.v_off;
        e.B = d->tbl->B;
        e.D = reinterpret_cast<float *>(ws + w.d_off);
        e.ldd = (int64_t)w.ldd;
        e.r_max = plan->r_max;
        e.N = d->N;
        e.max_units = (int32_t)pb.units;  // as for the shrink grid
        e.unit_rows = plan->unit_rows;
        e.col_groups = 0;
        // The tiled GEMM keeps the long segments' term to itself (an extension stage per 64 ranks of each such segment
        // of an M tile, ~2 us each, against 8 bytes of D traffic per element and the units' reads of B_a saved: worth
        // it up to rank 64 -- C3 gate_proj 150 -> 140 us; at rank 128, C4, 428 -> 434 us) and takes the short
        // segments' from D; the other kernels take all of it from D.
        const bool tiled = plan->r_max <= 64 && !all_in_d;
        e.skip_long = tiled ? 1 : 0;
        if (collect != nullptr) {
            const int i = collect->n_sets;
            e.n_sets = 0;
            if (i == 0) *collect = e;
            collect->set[i] = ExpandSet{e.V, e.B, e.D, e.ldd, e.N, e.skip_long, 0, 0};
            collect->n_sets = i + 1;
        } else {
            KernelTimer et;
            const bool etimed = expand_timer != nullptr && next_timer(ctx, kProfExpand, &et);
            LORA_HIP(launch_expand(e, d->dtype, stream, etimed ? &et : nullptr));
        }
        if (tiled) {
            g.long_rows = kLongSegRows;
        } else {
            g.B = nullptr;
            g.V = nullptr;
        }
        g.D = e.D;
        g.ldd = e.ldd;
    }
    *out = g;
    *split_out = split;
    return LORA_OK;
}

int do_gemm(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *d, hipStream_t stream) {
    GemmChoice c = choose_gemm(ctx, plan->T, d->K, d->N, d->dtype);
    if (c.variant == kGemmDecode)
        return do_decode_second(ctx, plan, pb, &d, 1, decode_args(ctx, plan, pb, &d, 1, c), c, stream);
    KernelTimer timer, etimer;
    const bool timed = next_timer(ctx, kProfGemm, &timer);
    const WorkspaceLayout w = workspace_layout(plan->T, d->K, d->N, plan->r_max, d->dtype);
    SplitK sk = choose_split_k(plan->T, d->K, d->N, d->dtype, d->workspace_bytes > w.sk_off ? d->workspace_bytes - w.sk_off : 0);
    if (ctx->opt_gemm_split_k == 0 || (ctx->opt_gemm_variant >= 0 && ctx->opt_gemm_variant != sk.variant) ||
        (has_adapters(plan, d) && w.d_bytes == 0))
        sk = SplitK{1, 0, kGemmTile128x128};
    if (sk.s > 1) c.variant = sk.variant;
    GemmSet g;
    bool split = false;
    const int rc = prepare_set(ctx, plan, pb, d, c.variant, stream, timed ? &etimer : nullptr, &g, &split, nullptr, sk.s > 1);
    if (rc != LORA_OK) return rc;
    if (sk.s > 1) {  // partial products per stretch of K, then one launch that sums them, adds the adapter term and rounds
        GemmArgs a;
        a.plan = view_of(plan);
        a.X = d->X;
        a.ldx = d->ldx;
        a.W = g.W;
        a.ldw = g.ldw;
        a.Y = g.Y;
        a.ldy = g.ldy;
        a.V = nullptr;
        a.B = nullptr;
        a.D = nullptr;
        a.ldd = 0;
        a.r_max = plan->r_max;
        a.T = (int32_t)plan->T;
        a.K = d->K;
        a.N = d->N;
        a.split_k = sk.s;
        a.k_chunk = sk.k_chunk;
        a.P = reinterpret_cast<float *>(static_cast<unsigned char *>(d->workspace) + w.sk_off);
        a.ldp = (int64_t)w.ldd;
        LORA_HIP(launch_gemm_tile(a, d->dtype, c.variant, stream, timed ? &timer : nullptr));
        SplitReduceArgs r;
        r.plan = a.plan;
        r.P = a.P;
        r.ldp = a.ldp;
        r.split_k = sk.s;
        r.D = g.D;  // (null when the call has no adapters)
        r.ldd = g.ldd;
        r.Y = d->Y;
        r.ldy = d->ldy;
        r.T = a.T;
        r.N = d->N;
        KernelTimer rtimer;
        const bool rtimed = timed && next_timer(ctx, kProfGemm, &rtimer);
        LORA_HIP(launch_splitk_reduce(r, d->dtype, stream, rtimed ? &rtimer : nullptr));
        return LORA_OK;
    }
    GemmArgs a;
    a.plan = view_of(plan);
    a.X = d->X;
    a.ldx = d->ldx;
    a.W = g.W;
    a.ldw = g.ldw;
    a.Y = g.Y;
    a.ldy = g.ldy;
    a.V = g.V;
    a.B = g.B;
    a.D = g.D;
    a.ldd = g.ldd;
    a.long_rows = g.long_rows;
    a.r_max = plan->r_max;
    a.T = (int32_t)plan->T;
    a.K = d->K;
    a.N = d->N;
    const KernelTimer *tg = timed ? &timer : nullptr;
    LORA_HIP(launch_gemm_tile(a, d->dtype, c.variant, stream, tg));
    return LORA_OK;
}

// Several projections of the same X in one GEMM launch (their column tiles side by side in one grid: one ramp, one
// set of whole rounds of tiles for all of them).  0: this batch / these options take the projections one by one;
// 1: the tiled kernel (one launch of each kernel for all of them); 2: the decode path's two launches for all of them.
int multi_kind(const lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *const *descs, int n, GemmChoice *c) {
    int32_t ns[kMaxGemmSets];
    for (int i = 0; i < n; ++i) ns[i] = descs[i]->N;
    *c = choose_gemm(ctx, plan->T, descs[0]->K, descs[0]->N, descs[0]->dtype);
    if (c->variant == kGemmDecode) {
        for (int i = 1; i < n; ++i)
            if (choose_gemm(ctx, plan->T, descs[i]->K, descs[i]->N, descs[i]->dtype).variant != kGemmDecode) return 0;
        return 2;
    }
    *c = choose_gemm_sets(ctx, plan->T, descs[0]->K, ns, n, descs[0]->dtype);
    if (c->variant == kGemmDecode) return 0;
    return 1;
}

int do_gemm_multi(lora_ctx *ctx, const lora_plan_t *plan, const PlanBounds &pb, const lora_linear_desc *const *descs, int n,
                  const GemmChoice &c, hipStream_t stream) {
    GemmArgs a;
    a.plan = view_of(plan);
    a.X = descs[0]->X;
    a.ldx = descs[0]->ldx;
    a.W = nullptr;
    a.ldw = 0;
    a.Y = nullptr;
    a.ldy = 0;
    a.V = nullptr;
    a.B = nullptr;
    a.D = nullptr;
    a.ldd = 0;
    a.r_max = plan->r_max;
    a.T = (int32_t)plan->T;
    a.K = descs[0]->K;
    a.N = 0;
    a.n_sets = n;
    KernelTimer timer;
    const bool timed = next_timer(ctx, kProfGemm, &timer);
    ExpandArgs e;
    e.n_sets = 0;
    for (int i = 0; i < n; ++i) {
        bool split = false;
        const int rc = prepare_set(ctx, plan, pb, descs[i], c.variant, stream, nullptr, &a.set[i], &split, &e);
        if (rc != LORA_OK) return rc;
    }
    if (e.n_sets > 0) {  // one launch for every projection that takes it
        KernelTimer et;
        const bool etimed = timed && next_timer(ctx, kProfExpand, &et);
        LORA_HIP(launch_expand(e, descs[0]->dtype, stream, etimed ? &et : nullptr));
    }
    LORA_HIP(launch_gemm_tile(a, descs[0]->dtype, c.variant, stream, timed ? &timer : nullptr));
    return LORA_OK;
}

}  // namespace

// =========================================================================================================
extern "C" {

int lora_ctx_create(lora_ctx **out, int device_ordinal) {
    if (!out) return LORA_ERR_INVALID_ARG;
    *out = nullptr;
    if (device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    int count = 0;
    LORA_HIP(hipGetDeviceCount(&count));
    if (device_ordinal >= count) return LORA_ERR_INVALID_ARG;
    lora_ctx *ctx = new (std::nothrow) lora_ctx();
    if (!ctx) return LORA_ERR_INVALID_ARG;
    ctx->keys = new (std::nothrow) KeyScratch;
    if (!ctx->keys) {
        delete ctx;
        return LORA_ERR_INVALID_ARG;
    }
    ctx->device = device_ordinal;
    DeviceGuard guard(device_ordinal);
    hipError_t e = guard.err;
    hipDeviceProp_t prop;
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, device_ordinal);
    if (e == hipSuccess) {
        ctx->num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
        e = hipHostMalloc(reinterpret_cast<void **>(&ctx->ring), kRingSlots * kRingSlotInts * sizeof(int32_t), hipHostMallocDefault);
    }
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void **>(&ctx->tables), kTableSlots * (kPlanTableInts * sizeof(int32_t) + sizeof(uint32_t)), hipHostMallocDefault);
    if (e == hipSuccess) {
        ctx->table_done = reinterpret_cast<uint32_t *>(ctx->tables + (size_t)kTableSlots * kPlanTableInts);
        memset(ctx->table_done, 0, kTableSlots * sizeof(uint32_t));
    }
    for (int i = 0; i < kRingSlots && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&ctx->ring_event[i], hipEventDisableTiming);
    // per-device set-up of the kernels: dynamic-LDS grants of every instantiation (so that no launch has to make one,
    // under stream capture or from two threads at once), and this device's address of the static scratch array
    if (e == hipSuccess) e = init_plan_kernels();
    if (e == hipSuccess) e = init_gemm_tile_kernels();
    if (e == hipSuccess) e = init_decode_kernels();
    if (e == hipSuccess) e = init_shrink_kernels();
    if (e == hipSuccess) e = init_expand_kernels();
    if (e == hipSuccess) e = hipGetSymbolAddress(reinterpret_cast<void **>(&ctx->static_scratch), HIP_SYMBOL(scratch));
    if (e != hipSuccess) {
        for (int i = 0; i < kRingSlots; ++i)
            if (ctx->ring_event[i]) (void)hipEventDestroy(ctx->ring_event[i]);
        if (ctx->ring) (void)hipHostFree(ctx->ring);
        if (ctx->tables) (void)hipHostFree(ctx->tables);
        delete ctx->keys;
        delete ctx;
        return hip_fail(e);
    }
    *out = ctx;
    return LORA_OK;
}

int lora_ctx_destroy(lora_ctx *ctx) {
    if (!ctx) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    for (int i = 0; i < kRingSlots; ++i) {
        if (ctx->ring_event[i]) {
            if (ctx->ring_used[i]) (void)hipEventSynchronize(ctx->ring_event[i]);
            (void)hipEventDestroy(ctx->ring_event[i]);
        }
    }
    // (tables that a kernel may still read: freed only once the device is known to be through with them)
    bool idle = true;
    for (int i = 0; i < kTableSlots; ++i) idle = idle && table_free(ctx, i);
    if (!idle) idle = hipDeviceSynchronize() == hipSuccess;
    if (ctx->ring) (void)hipHostFree(ctx->ring);
    if (idle) (void)hipHostFree(ctx->tables);
    free_profiler(ctx);
    delete ctx->keys;
    delete ctx;
    return LORA_OK;
}

int lora_ctx_set_option(lora_ctx *ctx, const char *name, int value) {
    if (!ctx || !name) return LORA_ERR_INVALID_ARG;
    if (!strcmp(name, "gemm_variant")) {
        if (value >= kGemmVariantCount || value == 2 || (value >= 6 && value <= 8)) return LORA_ERR_INVALID_ARG;
        ctx->opt_gemm_variant = value;
    } else if (!strcmp(name, "decode_waves")) {
        if (value >= 0 && (value < kDecodeMinWaves || value > kDecodeMaxWaves)) return LORA_ERR_INVALID_ARG;
        ctx->opt_decode_waves = value;
    } else if (!strcmp(name, "decode_max_rows")) {
        ctx->opt_decode_max_rows = value;
    } else if (!strcmp(name, "plan_fused_rows")) {
        ctx->opt_plan_fused_rows = value;
    } else if (!strcmp(name, "gemm_split_k")) {
        if (value > 1) return LORA_ERR_INVALID_ARG;
        ctx->opt_gemm_split_k = value;
    } else if (!strcmp(name, "expand_split")) {
        if (value > 1) return LORA_ERR_INVALID_ARG;
        ctx->opt_expand_split = value;
    } else if (!strcmp(name, "plan_variant")) {
        if (value > 1) return LORA_ERR_INVALID_ARG;
        ctx->opt_plan_variant = value;
    } else if (!strcmp(name, "shrink_rank_block")) {
        if (value > 0 && value != 8 && value != 16 && value != 32 && value != 64) return LORA_ERR_INVALID_ARG;
        ctx->opt_shrink_rank_block = value;
    } else {
        return LORA_ERR_INVALID_ARG;
    }
    return LORA_OK;
}

int lora_plan_validate(const int32_t *req_adapter, const int32_t *req_ntok, int32_t n_req, const int32_t *adapter_rank,
                       int32_t n_adapters, int32_t r_max, int64_t T_expected, int32_t *n_seg_out, int64_t *ext_total_out) {
    return validate_batch(req_adapter, req_ntok, n_req, adapter_rank, n_adapters, r_max, T_expected, n_seg_out, ext_total_out);
}

size_t lora_plan_bytes(int32_t n_req, int64_t T, int32_t n_adapters, int32_t r_max) {
    if (!plan_sizes_ok(n_req, T, n_adapters, r_max)) return 0;
    return plan_layout(n_req, T, n_adapters, r_max).total_bytes;
}

int lora_plan(lora_ctx *ctx, const int32_t *req_adapter, const int32_t *req_ntok, int32_t n_req, const int32_t *adapter_rank,
              int32_t n_adapters, int32_t r_max, int64_t T_expected, void *plan_buf, size_t plan_buf_bytes,
              lora_stream_t stream_, lora_plan_t *out) {
    int32_t n_seg = 0;
    int64_t ext_total = 0;
    int rc = validate_batch(req_adapter, req_ntok, n_req, adapter_rank, n_adapters, r_max, T_expected, &n_seg, &ext_total);
    if (rc != LORA_OK) return rc;
    const PlanLayout L = plan_layout(n_req, T_expected, n_adapters, r_max);
    rc = check_plan_buf(plan_buf, plan_buf_bytes, L, out);
    if (rc != LORA_OK) return rc;
    if (!ctx) return LORA_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    int32_t *base = static_cast<int32_t *>(plan_buf);
    int32_t *staged = base + L.staged;
    const PlanBuildArgs a = plan_args(ctx, staged, staged + n_req, staged + 2 * (size_t)n_req, n_req, n_adapters, r_max, T_expected, L, base);
    // The host's table for the batches one workgroup can serve; the arrays themselves and the device's own builders for
    // larger ones, under stream capture (nothing runs that would report the table read), while every table waits to be read, and
    // when an option asks for one of those builders.
    bool built = false;
    const bool asked = ctx->opt_plan_variant >= 0 || ctx->opt_plan_fused_rows >= 0;
    if (!asked && n_req <= kApplyReq && T_expected <= kApplyRows && ext_total <= 8 * kApplyRows && !is_capturing(stream)) {
        std::lock_guard<std::mutex> lock(ctx->ring_mutex);
        const int slot = take_table(ctx);
        if (slot >= 0) {
            PlanTable t;
            t.data = ctx->tables + (size_t)slot * kPlanTableInts;
            t.done = ctx->table_done + slot;
            t.ticket = ++ctx->last_ticket;  // (no two launches share one, whatever became of them)
            t.n_req = n_req;
            t.n_seg = n_seg;
            build_table(req_adapter, req_ntok, adapter_rank, n_adapters, a, ctx->keys, ctx->tables + (size_t)slot * kPlanTableInts, &t);
            KernelTimer timer;
            const bool timed = next_timer(ctx, kProfPlanSegments, &timer);
            LORA_HIP(launch_plan_apply(a, t, stream, timed ? &timer : nullptr));
            ctx->table_ticket[slot] = t.ticket;  // (only now: a launch that failed enqueued nothing and will report nothing)
            ctx->table_next = (slot + 1) % kTableSlots;
            fill_plan(a, out);
            built = true;
        }
    }
    if (!built) {
        const size_t n_ints = 2 * (size_t)n_req + (size_t)n_adapters;
        if (n_ints > 0) {
            std::lock_guard<std::mutex> lock(ctx->ring_mutex);
            const int slot = ctx->ring_next;
            ctx->ring_next = (slot + 1) % kRingSlots;
            if (ctx->ring_used[slot]) LORA_HIP(hipEventSynchronize(ctx->ring_event[slot]));
            int32_t *host = ctx->ring + (size_t)slot * kRingSlotInts;
            if (n_req > 0) {
                memcpy(host, req_adapter, sizeof(int32_t) * (size_t)n_req);
                memcpy(host + n_req, req_ntok, sizeof(int32_t) * (size_t)n_req);
            }
            if (n_adapters > 0) memcpy(host + 2 * (size_t)n_req, adapter_rank, sizeof(int32_t) * (size_t)n_adapters);
            LORA_HIP(hipMemcpyAsync(staged, host, n_ints * sizeof(int32_t), hipMemcpyHostToDevice, stream));
            LORA_HIP(hipEventRecord(ctx->ring_event[slot], stream));
            ctx->ring_used[slot] = true;
        }
        rc = build_plan(ctx, a, stream, out);
        if (rc != LORA_OK) return rc;
    }
    // (the host knows what the batch uses: see bounds_of)
    out->seg_cap = n_seg;
    out->ext_cap = (int32_t)(ext_total >> 3);
    return LORA_OK;
}

int lora_plan_device(lora_ctx *ctx, const int32_t *req_adapter, const int32_t *req_ntok, int32_t n_req,
                     const int32_t *adapter_rank, int32_t n_adapters, int32_t r_max, int64_t T_expected, void *plan_buf,
                     size_t plan_buf_bytes, lora_stream_t stream_, lora_plan_t *out) {
    if (!plan_sizes_ok(n_req, T_expected, n_adapters, r_max)) return LORA_ERR_INVALID_ARG;
    if (n_req > 0 && (!req_adapter || !req_ntok)) return LORA_ERR_INVALID_ARG;
    if (n_adapters > 0 && !adapter_rank) return LORA_ERR_INVALID_ARG;
    const PlanLayout L = plan_layout(n_req, T_expected, n_adapters, r_max);
    int rc = check_plan_buf(plan_buf, plan_buf_bytes, L, out);
    if (rc != LORA_OK) return rc;
    if (!ctx) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    return build_plan(ctx, plan_args(ctx, req_adapter, req_ntok, adapter_rank, n_req, n_adapters, r_max, T_expected, L, static_cast<int32_t *>(plan_buf)),
                      static_cast<hipStream_t>(stream_), out);
}

int lora_plan_status(lora_ctx *ctx, const lora_plan_t *plan, lora_stream_t stream_, int32_t *n_seg_out) {
    if (!ctx || !plan) return LORA_ERR_INVALID_ARG;
    if (plan->magic != kPlanMagic || !plan->scalars) return LORA_ERR_PLAN;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    LORA_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream_)));
    int32_t sc[8];
    LORA_HIP(hipMemcpy(sc, plan->scalars, sizeof sc, hipMemcpyDeviceToHost));
    if (n_seg_out) *n_seg_out = sc[kScNSeg];
    return sc[kScStatus] != 0 ? sc[kScStatus] : sc[kScEvicted];
}

size_t lora_linear_workspace_bytes(int64_t T, int32_t K, int32_t N, int32_t r_max, int32_t dtype) {
    if (T < 0 || K <= 0 || N <= 0 || r_max < 0 || (dtype != LORA_DTYPE_BF16 && dtype != LORA_DTYPE_F32)) return 0;
    return workspace_layout(T, K, N, r_max, dtype).total;
}

size_t lora_linear_workspace_bytes_preferred(int64_t T, int32_t K, int32_t N, int32_t r_max, int32_t dtype) {
    if (T < 0 || K <= 0 || N <= 0 || r_max < 0 || (dtype != LORA_DTYPE_BF16 && dtype != LORA_DTYPE_F32)) return 0;
    return workspace_layout(T, K, N, r_max, dtype).total_preferred;
}

int lora_shrink(lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *desc, lora_stream_t stream) {
    int rc = check_linear(ctx, plan, desc);
    if (rc != LORA_OK) return rc;
    if (plan->T == 0) return LORA_OK;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return do_shrink(ctx, plan, bounds_of(plan, s), desc, s);
}

int lora_gemm_expand(lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *desc, lora_stream_t stream) {
    int rc = check_linear(ctx, plan, desc);
    if (rc != LORA_OK) return rc;
    if (plan->T == 0) return LORA_OK;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return do_gemm(ctx, plan, bounds_of(plan, s), desc, s);
}

int lora_linear(lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *desc, lora_stream_t stream) {
    int rc = check_linear(ctx, plan, desc);
    if (rc != LORA_OK) return rc;
    if (plan->T == 0) return LORA_OK;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const PlanBounds pb = bounds_of(plan, s);
    rc = do_shrink(ctx, plan, pb, desc, s);
    if (rc != LORA_OK) return rc;
    return do_gemm(ctx, plan, pb, desc, s);
}

int lora_linear_static(lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *desc, lora_stream_t stream) {
    if (!desc) return LORA_ERR_INVALID_ARG;
    if (desc->workspace != nullptr || desc->workspace_bytes != 0) return LORA_ERR_INVALID_ARG;
    if (!plan) return LORA_ERR_INVALID_ARG;
    // (sizes first, so that an oversized problem is reported as such whatever else is wrong with it)
    if (plan->T >= 0 && desc->K > 0 && desc->N > 0 && plan->r_max >= 0 &&
        (desc->dtype == LORA_DTYPE_BF16 || desc->dtype == LORA_DTYPE_F32) &&
        workspace_layout(plan->T, desc->K, desc->N, plan->r_max, desc->dtype).total > (size_t)LORA_STATIC_SCRATCH_BYTES)
        return LORA_ERR_WORKSPACE_TOO_SMALL;
    int rc = check_linear(ctx, plan, desc, true, false);
    if (rc != LORA_OK) return rc;
    lora_linear_desc d = *desc;
    d.workspace = ctx->static_scratch;
    d.workspace_bytes = LORA_STATIC_SCRATCH_BYTES;
    if (plan->T == 0) return LORA_OK;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const PlanBounds pb = bounds_of(plan, s);
    rc = do_shrink(ctx, plan, pb, &d, s);
    if (rc != LORA_OK) return rc;
    return do_gemm(ctx, plan, pb, &d, s);
}

int lora_linear_multi(lora_ctx *ctx, const lora_plan_t *plan, const lora_linear_desc *const *descs, int32_t n,
                      lora_stream_t stream) {
    if (!descs || n < 1 || n > LORA_MAX_MULTI) return LORA_ERR_INVALID_ARG;
    for (int i = 0; i < n; ++i) {
        if (!descs[i]) return LORA_ERR_INVALID_ARG;
        const int rc = check_linear(ctx, plan, descs[i], false);
        if (rc != LORA_OK) return rc;
        if (descs[i]->X != descs[0]->X || descs[i]->ldx != descs[0]->ldx || descs[i]->K != descs[0]->K ||
            descs[i]->dtype != descs[0]->dtype)
            return LORA_ERR_INVALID_ARG;
        for (int j = 0; j < i; ++j)
            if (plan->T > 0 && (descs[i]->Y == descs[j]->Y || descs[i]->workspace == descs[j]->workspace)) return LORA_ERR_INVALID_ARG;
    }
    if (!ctx) return LORA_ERR_INVALID_ARG;  // (last: the checks above run on a GPU-less host too)
    if (plan->T == 0) return LORA_OK;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const PlanBounds pb = bounds_of(plan, s);
    GemmChoice c;
    const int kind = n == 1 ? 0 : multi_kind(ctx, plan, descs, n, &c);
    if (kind == 0) {  // one after the other
        for (int i = 0; i < n; ++i) {
            int rc = do_shrink(ctx, plan, pb, descs[i], s);
            if (rc == LORA_OK) rc = do_gemm(ctx, plan, pb, descs[i], s);
            if (rc != LORA_OK) return rc;
        }
        return LORA_OK;
    }
    if (kind == 2) return do_decode(ctx, plan, pb, descs, n, c, s);
    const int rc = do_shrink(ctx, plan, pb, descs[0], s, descs, n);  // one launch: the single projection's grid once per projection
    if (rc != LORA_OK) return rc;
    return do_gemm_multi(ctx, plan, pb, descs, n, c, s);
}

int lora_profile_begin(lora_ctx *ctx, int max_launches) {
    if (!ctx || max_launches <= 0 || max_launches > (1 << 20)) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    if (max_launches > ctx->prof_cap) {
        free_profiler(ctx);
        for (int k = 0; k < kProfKinds; ++k) {
            ctx->prof_start[k] = new (std::nothrow) hipEvent_t[max_launches]();
            ctx->prof_stop[k] = new (std::nothrow) hipEvent_t[max_launches]();
            if (!ctx->prof_start[k] || !ctx->prof_stop[k]) return LORA_ERR_INVALID_ARG;
        }
        ctx->prof_cap = max_launches;
        for (int k = 0; k < kProfKinds; ++k)
            for (int i = 0; i < max_launches; ++i) {
                LORA_HIP(hipEventCreate(&ctx->prof_start[k][i]));
                LORA_HIP(hipEventCreate(&ctx->prof_stop[k][i]));
            }
    }
    for (int k = 0; k < kProfKinds; ++k) ctx->prof_used[k] = 0;
    ctx->prof_on = true;
    return LORA_OK;
}

int lora_profile_end(lora_ctx *ctx, lora_stream_t stream, double *avg_us, int32_t *counts) {
    if (!ctx || !avg_us || !counts) return LORA_ERR_INVALID_ARG;
    if (!ctx->prof_on) return LORA_ERR_INVALID_ARG;
    ctx->prof_on = false;
    DeviceGuard guard(ctx->device);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    LORA_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    for (int k = 0; k < kProfKinds; ++k) {
        double sum = 0.0;
        for (int i = 0; i < ctx->prof_used[k]; ++i) {
            float ms = 0.f;
            LORA_HIP(hipEventElapsedTime(&ms, ctx->prof_start[k][i], ctx->prof_stop[k][i]));
            sum += (double)ms * 1000.0;
        }
        counts[k] = ctx->prof_used[k];
        avg_us[k] = ctx->prof_used[k] > 0 ? sum / ctx->prof_used[k] : 0.0;
        ctx->prof_used[k] = 0;
    }
    return LORA_OK;
}

static_assert(sizeof(hipIpcMemHandle_t) == LORA_IPC_HANDLE_BYTES, "IPC handle size out of sync");

int lora_backbone_alloc(int device_ordinal, size_t bytes, void **dev_ptr_out) {
    if (!dev_ptr_out || bytes == 0 || device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    *dev_ptr_out = nullptr;
    DeviceGuard guard(device_ordinal);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    LORA_HIP(hipMalloc(dev_ptr_out, bytes));
    return LORA_OK;
}

int lora_backbone_free(int device_ordinal, void *dev_ptr) {
    if (!dev_ptr || device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(device_ordinal);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    LORA_HIP(hipFree(dev_ptr));
    return LORA_OK;
}

int lora_backbone_export(int device_ordinal, const void *dev_ptr, unsigned char handle_out[LORA_IPC_HANDLE_BYTES]) {
    if (!dev_ptr || !handle_out || device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(device_ordinal);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipIpcMemHandle_t h;
    LORA_HIP(hipIpcGetMemHandle(&h, const_cast<void *>(dev_ptr)));
    memcpy(handle_out, &h, sizeof h);
    return LORA_OK;
}

int lora_backbone_open(int device_ordinal, const unsigned char handle[LORA_IPC_HANDLE_BYTES], void **dev_ptr_out) {
    if (!handle || !dev_ptr_out || device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    *dev_ptr_out = nullptr;
    DeviceGuard guard(device_ordinal);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    hipIpcMemHandle_t h;
    memcpy(&h, handle, sizeof h);
    LORA_HIP(hipIpcOpenMemHandle(dev_ptr_out, h, hipIpcMemLazyEnablePeerAccess));
    return LORA_OK;
}

int lora_backbone_close(int device_ordinal, void *dev_ptr) {
    if (!dev_ptr || device_ordinal < 0) return LORA_ERR_INVALID_ARG;
    DeviceGuard guard(device_ordinal);
    if (guard.err != hipSuccess) return hip_fail(guard.err);
    LORA_HIP(hipIpcCloseMemHandle(dev_ptr));
    return LORA_OK;
}

const char *lora_gemm_kernel_name(lora_ctx *ctx, int64_t T, int32_t K, int32_t N, int32_t dtype) {
    static thread_local char buf[64];
    const GemmChoice c = choose_gemm(ctx, T, K, N, dtype);
    // (with a workspace of the preferred size and an adapter table, or none)
    const SplitK sk = choose_split_k(T, K, N, dtype);
    if (c.variant != kGemmDecode && sk.s > 1 && !(ctx && ctx->opt_gemm_split_k == 0) &&
        !(ctx && ctx->opt_gemm_variant >= 0 && ctx->opt_gemm_variant != sk.variant)) {
        const char *shape = sk.variant == kGemmTile128x128 ? "128x128" : sk.variant == kGemmTile192x128 ? "192x128" : "256x256";
        snprintf(buf, sizeof buf, "tile_%s_splitk%d", shape, sk.s);
        return buf;
    }
    switch (c.variant) {
        case kGemmDecode:
            snprintf(buf, sizeof buf, "decode_tb%d", c.tblk);
            break;
        case kGemmTile64x64:
            snprintf(buf, sizeof buf, "tile_64x64");
            break;
        case kGemmTile128x128:
            snprintf(buf, sizeof buf, "tile_128x128");
            break;
        case kGemmTile256x128:
            snprintf(buf, sizeof buf, "tile_256x128");
            break;
        case kGemmTile256x256w4:
            snprintf(buf, sizeof buf, "tile_256x256w4");
            break;
        case kGemmTile128x192:
            snprintf(buf, sizeof buf, "tile_128x192");
            break;
        case kGemmTile256x192:
            snprintf(buf, sizeof buf, "tile_256x192");
            break;
        case kGemmTile256x224:
            snprintf(buf, sizeof buf, "tile_256x224");
            break;
        case kGemmTile192x128:
            snprintf(buf, sizeof buf, "tile_192x128");
            break;
        default:
            snprintf(buf, sizeof buf, "unknown");
    }
    return buf;
}

const char *lora_strerror(int status) {
    switch (status) {
        case LORA_OK:
            return "ok";
        case LORA_ERR_INVALID_ARG:
            return "invalid argument";
        case LORA_ERR_BAD_ADAPTER_ID:
            return "adapter id outside [-1, n_adapters)";
        case LORA_ERR_LENGTH_MISMATCH:
            return "negative token count or token counts do not add up to T";
        case LORA_ERR_ADAPTER_NOT_RESIDENT:
            return "a used adapter is not resident (rank 0 or null weights)";
        case LORA_ERR_RANK_TOO_LARGE:
            return "a used adapter's rank exceeds r_max";
        case LORA_ERR_WORKSPACE_TOO_SMALL:
            return "plan buffer or workspace too small";
        case LORA_ERR_ALIGNMENT:
            return "pointer or row stride not aligned";
        case LORA_ERR_SHAPE:
            return "unsupported shape (K, N, leading dimension or rank)";
        case LORA_ERR_HIP:
            return "HIP runtime error";
        case LORA_ERR_PLAN:
            return "not a valid plan";
        default:
            return "unknown status";
    }
}

int lora_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"

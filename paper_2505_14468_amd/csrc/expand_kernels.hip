// Segmented LoRA expand as a kernel of its own, for batches of many small segments:
//
//     D[row, n] = sum_j V[row, j] * B_a[n, j]        for the rows of every adapter segment, in fp32
//
// (second half of the adapter product of paper section 4.4; the base GEMM that runs next adds D to
// its fp32 accumulators before it rounds and stores Y, once).  When an M tile of the fused GEMM holds dozens of adapters, every
// extension stage there serves a handful of rows, and the adapters' B matrices -- together larger
// than W0 in such a batch -- arrive through a two-deep, latency-bound pipeline.  Here the same work
// is a weight-streaming problem laid out like the shrink:
//
//   * a workgroup = one work unit of the plan's list (<= 64 rows of one segment, <= 16 in small plans) x 256 output
//     columns (128 to 1024 where the ranks are large);
//   * the unit's rows of V (<= 64 x r, a few KB) are staged in LDS once; as MFMA operand they are
//     read from there, so global loads carry B_a only;
//   * each of the 2 waves (4, 8) walks 16-column blocks; MFMA 16x16x32 with the 16 output columns as M
//     (operand rows = rows of B_a, contiguous along the rank) and 16 token rows as N; four groups
//     of loads (16 KB per wave) are in flight while one is multiplied, across block boundaries;
//   * steps come in pairs that share one 128-byte piece of every B_a row (step 2m takes the even
//     16-byte chunks, step 2m+1 the odd ones), so a load instruction covers whole cache lines;
//   * every (row, column) with an adapter belongs to exactly one unit, so D is stored, not accumulated;
//     rows without an adapter are never written and never read.  D costs 8 bytes of traffic per output
//     element with an adapter, against the B_a bytes streamed at HBM speed instead of through a
//     latency-bound pipeline; the host picks this path for batches of many small segments only;
//   * units of long segments (flagged in the work list) are skipped when the GEMM computes those itself;
//   * one launch can cover several projections of the same batch (ExpandSet), grid after grid.
#include "kernels.h"

namespace lora {
namespace {

// Workgroups of two waves: a unit is a chain of four dependent round trips (work list -> row map and adapter -> V and B_a ->
// stores) with a short stream in the middle, and what one CU gets through is how many of them run side by side.  1024, 512 and
// 256 columns a workgroup (eight, four, two waves): 1216 rows on 100 adapters of rank 8 to 64, gate and up 37.3 / 31.0 / 28.1 us,
// one 4096 -> 4096 16.6 / 15.0 / 14.2; 1500 one-token requests 18.8 / 17.0 / 16.0; 365 rows 7.9 / 5.8 / 5.6; 2048 rows on some 170
// adapters of rank 128, 5120 -> 13824 (714 MB of B_a and D) 170 / 163 / 164.
// Four or eight waves where the LDS for a unit's V leaves too few workgroups of two on a CU: see expand_waves.
constexpr int ex_cols(int waves, int blocks) { return waves * blocks * 16; }  // output columns per workgroup (16-column blocks per wave)
constexpr int kExGroup = 4;                                       // MFMA steps per load group
constexpr int kExRing = 4;                                        // load groups in flight per wave
constexpr int kExPad = 1;                                         // chunks of padding per staged row of V
constexpr size_t kLdsBytesPerCu = 160 * 1024;
// Four blocks per wave instead of eight where the rows of B_a are long: what a wave streams for eight lasts longer than a unit's
// set-up.  Eight and four, us: bf16 rank 128, 600 rows on 100 adapters, N 358 5.5 / 5.2, 2048 12.0 / 10.7, 4096 22.3 / 19.5, 11008 61.8
// / 57.2; fp32 rank 128, N 358 18.1 / 12.6, 749 22.4 / 16.1, 4096 53.5 / 50.2, 11008 129 / 124; but rank 16 to 32 bf16 4096 -> 4096, 1500
// rows 16.4 / 18.0, rank 8 to 64, 1216 rows 16.0 / 17.8, fp32 rank 16, 600 rows, N 4096 12.7 / 12.2, 1500 rows, N 2048 29.0 / 34.4.
constexpr int kExLongRow = 256;  // bytes

template <typename E, int WAVES, int NBLK, int TB>
__device__ __forceinline__ void expand_unit(const ExpandArgs &p, const E *Ba, int r, int slot0, int nrows, int nwg0,
                                            unsigned char *smem) {
    constexpr int CE = Elem<E>::CE;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int rchunks = r / CE;
    const int vstride = rchunks + kExPad;
    chunk_t *vs = reinterpret_cast<chunk_t *>(smem);
    const E *V = static_cast<const E *>(p.V);

    // rows of D this lane stores (rows past the unit: never stored)
    int64_t drow[TB];
    bool rok[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int t = tb * 16 + li;
        rok[tb] = t < nrows;
        drow[tb] = (int64_t)p.plan.perm[slot0 + min(t, nrows - 1)] * p.ldd;
    }
    const chunk_t *vrow[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) vrow[tb] = vs + min(tb * 16 + li, nrows - 1) * vstride;

    // MFMA steps over the rank: pairs of steps, lane group g takes chunks 2g (even step) and 2g+1 (odd step)
    // of each 8-chunk piece; chunks past the rank contribute zeros (the V operand is zeroed).
    const int steps = 2 * ((rchunks + 7) >> 3);
    const int groups = (steps + kExGroup - 1) / kExGroup;
    auto chunk_of = [&](int st) { return (st >> 1) * 8 + 2 * lg + (st & 1); };

    // this wave's column blocks, b = 0 .. NBLK-1 (those below N): pairs of adjacent blocks (32 columns:
    // a row's two stores fall into one 128-byte line), pair p of wave w at column 32 * (w + WAVES p)
    auto block_n0 = [&](int b) { return nwg0 + (2 * wave + (b & 1) + 2 * WAVES * (b >> 1)) * 16; };
    int nblk = 0;
#pragma unroll
    for (int b = 0; b < NBLK; ++b) nblk += block_n0(b) < p.N ? 1 : 0;
    const int total = nblk * groups;  // (block, group) pairs, walked in order

    auto load_group = [&](int q, chunk_t (&wf)[kExGroup]) {
        if (q < total) {
            const int b = q / groups, g = q - b * groups;
            const E *brow = Ba + (int64_t)min(block_n0(b) + li, p.N - 1) * r;  // columns past N: clamped, never stored
#pragma unroll
            for (int s = 0; s < kExGroup; ++s) {
                const int st = g * kExGroup + s;
                const int kc = chunk_of(st);
                wf[s] = load_chunk(brow + (int64_t)((st < steps && kc < rchunks) ? kc : 0) * CE);
            }
        }
    };
    f32x4_t acc[TB];
    auto mma_group = [&](int q, const chunk_t (&wf)[kExGroup]) {
        const int g = q % groups;
#pragma unroll
        for (int s = 0; s < kExGroup; ++s) {
            const int st = g * kExGroup + s;
            if (st < steps) {
                const int kc = chunk_of(st);
                const bool ok = kc < rchunks;
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    const chunk_t v = keep_if(ok, vrow[tb][ok ? kc : 0]);
                    Elem<E>::mma16(acc[tb], wf[s], v);
                }
            }
        }
    };
    // acc[tb][e] = D[n = n0 + lg*4 + e][t = tb*16 + li]: a lane stores 4 consecutive columns of one row
    auto flush_block = [&](int b) {
        const int n = block_n0(b) + lg * 4;
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            if (!rok[tb]) continue;
            float *dst = p.D + drow[tb] + n;
            if (n + 3 < p.N) {
                store4(dst, acc[tb][0], acc[tb][1], acc[tb][2], acc[tb][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < p.N) dst[e] = acc[tb][e];
            }
        }
    };

    // ---- stage the unit's rows of V (original row order in memory: gather through the row map) ----
    // V first: it comes from L2 and loads return in order -- behind B_a's loads from HBM it would arrive last.
    LORA_TS(p.trace, 2);  // row map read
    // (Four pieces per thread at a time, unguarded: a loop of one would be two round trips per piece.)
    constexpr int VP = 4;
    const int pieces = nrows * rchunks;
    for (int e0 = tid; e0 < pieces; e0 += VP * WAVES * 64) {
        chunk_t v[VP];
        int dst[VP];
#pragma unroll
        for (int u = 0; u < VP; ++u) {
            const int e = min(e0 + u * WAVES * 64, pieces - 1);
            const int t = e / rchunks, c = e - t * rchunks;
            dst[u] = t * vstride + c;
            v[u] = load_chunk(V + (int64_t)p.plan.perm[slot0 + t] * p.r_max + (int64_t)c * CE);
        }
#pragma unroll
        for (int u = 0; u < VP; ++u) vs[dst[u]] = v[u];  // (past the last piece: the last one again)
    }
    // ---- a ring of kExRing groups of B_a loads in flight per wave ----
    chunk_t ring[kExRing][kExGroup];
#pragma unroll
    for (int i = 0; i < kExRing; ++i) load_group(i, ring[i]);
    __syncthreads();
    LORA_TS(p.trace, 3);  // V staged
    for (int q0 = 0; q0 < total; q0 += kExRing) {
#pragma unroll
        for (int i = 0; i < kExRing; ++i) {
            const int q = q0 + i;
            if (q < total) {
                if (q % groups == 0) {
#pragma unroll
                    for (int tb = 0; tb < TB; ++tb) acc[tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
                mma_group(q, ring[i]);
                if ((q + 1) % groups == 0) flush_block(q / groups);
                load_group(q + kExRing, ring[i]);
            }
        }
    }
}

// The common shapes -- rank <= 128 (bf16) -- with every index a compile-time constant:
// S MFMA steps per 16-column block (2: at most 8 chunks of rank, 4: at most 16), the B_a loads of RING blocks in flight
// per wave (all of them: everything is requested before the first MFMA), the results of all NBLK blocks kept in
// registers and stored after the last load has been consumed.  Loads and stores are counted by one in-order
// counter, so a store issued between loads makes the next wait for a load wait for the store's acknowledgement
// from memory as well; and no load sits behind a branch, so that the compiler can count the loads in flight.  In the last group of
// columns, if it is not a whole one, the rows of B_a past N are clamped and their columns not stored.
template <typename E, int WAVES, int NBLK, int TB, int S, int RING0>
__device__ __forceinline__ void expand_unit_short(const ExpandArgs &p, const E *Ba, int r, int slot0, int nrows, int nwg0,
                                                  unsigned char *smem) {
    constexpr int CE = Elem<E>::CE;
    constexpr int RING = RING0 < NBLK ? RING0 : NBLK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int rchunks = r / CE;
    const int vstride = rchunks + kExPad;
    chunk_t *vs = reinterpret_cast<chunk_t *>(smem);
    const E *V = static_cast<const E *>(p.V);

    // ---- the unit's rows of V (at most 16 TB rows x 4 S chunks), requested first ----
    constexpr int VL = (TB * 16 * 4 * S + WAVES * 64 - 1) / (WAVES * 64);
    chunk_t vreg[VL];
    int vdst[VL];
#pragma unroll
    for (int u = 0; u < VL; ++u) {
        const int e = tid + u * (WAVES * 64);
        const bool ok = e < nrows * rchunks;
        const int t = ok ? e / rchunks : 0, c = ok ? e - t * rchunks : 0;
        vdst[u] = ok ? t * vstride + c : -1;
        vreg[u] = load_chunk(V + (int64_t)p.plan.perm[slot0 + t] * p.r_max + (int64_t)c * CE);
    }
    // ---- B_a: lane -> (column block_n0 + li, chunk of the step); chunks past the rank are read from chunk 0
    //      and meet a zeroed V operand ----
    auto block_n0 = [&](int b) { return nwg0 + (2 * wave + (b & 1) + 2 * WAVES * (b >> 1)) * 16; };
    int kc[S];
    bool kok[S];
#pragma unroll
    for (int st = 0; st < S; ++st) {
        const int c = (st >> 1) * 8 + 2 * lg + (st & 1);
        kok[st] = c < rchunks;
        kc[st] = kok[st] ? c : 0;
    }
    auto load_block = [&](int b, chunk_t (&wf)[S]) {
        const E *brow = Ba + (int64_t)min(block_n0(b) + li, p.N - 1) * r;
#pragma unroll
        for (int st = 0; st < S; ++st) wf[st] = load_chunk(brow + kc[st] * CE);
    };
    chunk_t ring[RING][S];
#pragma unroll
    for (int i = 0; i < RING; ++i) load_block(i, ring[i]);
    LORA_TS(p.trace, 2);
#pragma unroll
    for (int u = 0; u < VL; ++u)
        if (vdst[u] >= 0) vs[vdst[u]] = vreg[u];
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // LDS only: the B_a loads stay in flight
    LORA_TS(p.trace, 3);  // V staged

    // V operands of this lane: row tb * 16 + li (clamped), the step's chunk; the same for every block
    chunk_t vop[TB][S];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int st = 0; st < S; ++st) vop[tb][st] = keep_if(kok[st], vs[min(tb * 16 + li, nrows - 1) * vstride + kc[st]]);

    f32x4_t acc[NBLK][TB];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[b][tb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < S; ++st)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) Elem<E>::mma16(acc[b][tb], ring[b % RING][st], vop[tb][st]);
        if (b + RING < NBLK) load_block(b + RING, ring[b % RING]);
    }
    LORA_TS(p.trace, 4);
    // acc[b][tb][e] = D[n = block_n0(b) + lg*4 + e][t = tb*16 + li]: a lane stores 4 consecutive columns of one row
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int t = tb * 16 + li;
        if (t >= nrows) continue;
        float *drow = p.D + (int64_t)p.plan.perm[slot0 + t] * p.ldd;
        if (nwg0 + ex_cols(WAVES, NBLK) <= p.N) {
#pragma unroll
            for (int b = 0; b < NBLK; ++b) store4(drow + block_n0(b) + lg * 4, acc[b][tb][0], acc[b][tb][1], acc[b][tb][2], acc[b][tb][3]);
            continue;
        }
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const int n = block_n0(b) + lg * 4;
            if (n + 3 < p.N) {
                store4(drow + n, acc[b][tb][0], acc[b][tb][1], acc[b][tb][2], acc[b][tb][3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < p.N) drow[n + e] = acc[b][tb][e];
            }
        }
    }
}

// SMALL: every unit of the plan has at most 16 rows.  That instantiation keeps a quarter of the accumulators and
// half the loads in flight, fits 128 registers (4 waves per SIMD): twice as many workgroups share a CU, and a unit of a few
// rows is a chain of dependent round trips (work list, row map and adapter table, operands) more than it is a
// stream, and one workgroup's chain overlaps the others' loads.
template <typename E, int WAVES, int NBLK, bool SMALL>
__global__ __launch_bounds__(WAVES * 64, SMALL ? 4 : 2) void expand_kernel(ExpandArgs p0) {
    constexpr int COLS = ex_cols(WAVES, NBLK);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    LORA_TS(p0.trace, 0);
    // several projections of the same batch: the single-projection grids one after the other
    ExpandArgs p = p0;
    int bid = blockIdx.x;
    if (p0.n_sets > 0) {
        int si = 0;
        while (si + 1 < p0.n_sets && bid >= p0.set[si + 1].block0) ++si;
        bid -= p0.set[si].block0;
        p.V = p0.set[si].V;
        p.B = p0.set[si].B;
        p.D = p0.set[si].D;
        p.ldd = p0.set[si].ldd;
        p.N = p0.set[si].N;
        p.skip_long = p0.set[si].skip_long;
        p.col_groups = (p.N + COLS - 1) / COLS;
    }
    const int unit = bid / p.col_groups;
    const int cg = bid - unit * p.col_groups;
    // the grid is an upper bound of the unit count and the work list is that long
    const int4 rec = reinterpret_cast<const int4 *>(p.plan.unit_rec)[unit];
    const int status = p.plan.scalars[kScStatus], n_units = p.plan.scalars[kScNUnits];
    if (status != 0 || unit >= n_units) return;
    const int a = rec.x, r = rec.y & 0xffff, slot0 = rec.z, nrows = rec.w;
    if (a < 0 || r <= 0 || nrows <= 0) return;
    if (p.skip_long && (rec.y & kUnitLongFlag)) return;  // the GEMM computes this segment's term itself
    const E *Ba = static_cast<const E *>(p.B[a]);
    LORA_TS(p.trace, 1);  // work-list record read
    if (Ba == nullptr) {  // slot emptied after the plan was built: flag it, contribute nothing
        if (threadIdx.x == 0) atomicMin(&p.plan.scalars[kScEvicted], kErrNotResident);
        const int n_lo = cg * COLS, n_hi = min(n_lo + COLS, p.N);
        for (int e = threadIdx.x; e < nrows * (n_hi - n_lo); e += WAVES * 64) {
            const int t = e / (n_hi - n_lo), n = n_lo + e - t * (n_hi - n_lo);
            p.D[(int64_t)p.plan.perm[slot0 + t] * p.ldd + n] = 0.f;
        }
        return;
    }
    const int rchunks = r / Elem<E>::CE;
    if (rchunks <= 16) {  // at most 4 MFMA steps along the rank
        if constexpr (SMALL) {
            if (rchunks <= 8)
                expand_unit_short<E, WAVES, NBLK, 1, 2, 8>(p, Ba, r, slot0, nrows, cg * COLS, smem);
            else
                expand_unit_short<E, WAVES, NBLK, 1, 4, 4>(p, Ba, r, slot0, nrows, cg * COLS, smem);
        } else if (nrows <= 16) {
            if (rchunks <= 8)
                expand_unit_short<E, WAVES, NBLK, 1, 2, 8>(p, Ba, r, slot0, nrows, cg * COLS, smem);
            else
                expand_unit_short<E, WAVES, NBLK, 1, 4, 8>(p, Ba, r, slot0, nrows, cg * COLS, smem);
        } else {
            if (rchunks <= 8)
                expand_unit_short<E, WAVES, NBLK, 4, 2, 8>(p, Ba, r, slot0, nrows, cg * COLS, smem);
            else
                expand_unit_short<E, WAVES, NBLK, 4, 4, 4>(p, Ba, r, slot0, nrows, cg * COLS, smem);
        }
    } else if (SMALL || nrows <= 16) {
        expand_unit<E, WAVES, NBLK, 1>(p, Ba, r, slot0, nrows, cg * COLS, smem);
    } else {
        expand_unit<E, WAVES, NBLK, 4>(p, Ba, r, slot0, nrows, cg * COLS, smem);
    }
    LORA_TS(p.trace, 5);
}

}  // namespace

static constexpr size_t expand_smem_bytes(int r_max, int dtype, int unit_rows) {
    const int ce = dtype == 1 ? 8 : 4;
    return (size_t)unit_rows * (size_t)(r_max / ce + kExPad) * 16;
}

// Waves per workgroup: as few as let the workgroups whose rows of V fit a CU's LDS hold the waves that its registers do, 8 or
// 16 of the small form.  Two, four and eight waves, us: 2000 rows on 150 adapters, 2048 -> 4096, bf16 rank 512 (67 KB) 222 / 165 / 171,
// fp32 rank 256 (67 KB) 335 / 215 / 223, rank 512 (132 KB) 1012 / 565 / 421; 600 rows on 64 adapters, units of 16 rows, fp32 rank 512
// (33 KB) - / 118 / 117.  (With one such adapter in a pool of rank 16 the fewest are best: bf16 rank 512 31.9 / 32.9 / 36.4, fp32 rank
// 512 84.5 / 85.6 / 96.5.)
static int expand_waves(size_t smem, bool small) {
    const long wgs = (long)(kLdsBytesPerCu / smem), held = small ? 16 : 8;
    return wgs * 2 >= held ? 2 : wgs * 4 >= held ? 4 : 8;
}

template <typename E, int WAVES, int NBLK = 8>
static hipError_t init_expand() {
    // (ranks above ~480 need more than the default 64 KB of dynamic LDS: granted per kernel and device before the first launch)
    const int dtype = sizeof(E) == 2 ? 1 : 0;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(expand_kernel<E, WAVES, NBLK, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)expand_smem_bytes(kMaxRank, dtype, kShrinkRowsSmall));
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(expand_kernel<E, WAVES, NBLK, false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)expand_smem_bytes(kMaxRank, dtype, kShrinkRows));
    return e;
}
static_assert(kLdsBytesPerCu / expand_smem_bytes(kMaxRank, 1, kShrinkRows) * 4 >= 8, "bf16 needs four waves at most");
hipError_t init_expand_kernels() {
    hipError_t e = init_expand<__bf16, 2>();
    if (e == hipSuccess) e = init_expand<__bf16, 2, 4>();
    if (e == hipSuccess) e = init_expand<float, 2, 4>();
    if (e == hipSuccess) e = init_expand<__bf16, 4>();
    if (e == hipSuccess) e = init_expand<float, 2>();
    if (e == hipSuccess) e = init_expand<float, 4>();
    if (e == hipSuccess) e = init_expand<float, 8>();
    return e;
}

template <typename E, int WAVES, int NBLK = 8>
static hipError_t launch_expand_waves(const ExpandArgs &a, bool small, long grid, size_t smem, hipStream_t stream, const KernelTimer *timer) {
    const dim3 g((unsigned)grid), t(WAVES * 64);
    return small ? launch_kernel(expand_kernel<E, WAVES, NBLK, true>, g, t, smem, stream, timer, a)
                 : launch_kernel(expand_kernel<E, WAVES, NBLK, false>, g, t, smem, stream, timer, a);
}

hipError_t launch_expand(const ExpandArgs &a0, int dtype, hipStream_t stream, const KernelTimer *timer) {
    if (a0.max_units <= 0 || (a0.n_sets == 0 && a0.N <= 0)) return hipSuccess;
    ExpandArgs a = a0;
    const bool small = a.unit_rows <= kShrinkRowsSmall;
    const size_t smem = expand_smem_bytes(a.r_max, dtype, small ? kShrinkRowsSmall : kShrinkRows);
    const int waves = expand_waves(smem, small);
    int cols = 0;
    long grid = 0;
    auto lay_out = [&](int blocks) {
        cols = ex_cols(waves, blocks);
        if (a.n_sets > 0) {
            grid = 0;
            for (int i = 0; i < a.n_sets; ++i) {
                a.set[i].block0 = (int32_t)grid;
                grid += (long)a.max_units * ((a.set[i].N + cols - 1) / cols);
            }
        } else {
            a.col_groups = (a.N + cols - 1) / cols;
            grid = (long)a.max_units * a.col_groups;
        }
    };
    bool halves = waves == 2 && a.r_max * (dtype == 1 ? 2 : 4) >= kExLongRow;
    lay_out(halves ? 4 : 8);
    if (halves && grid * (waves * 64) >= (1l << 32)) {  // (a launch has fewer than 2^32 threads)
        halves = false;
        lay_out(8);
    }
    if (grid <= 0) return hipSuccess;
    auto launch = [&](const ExpandArgs &b) {
        if (halves)
            return dtype == 1 ? launch_expand_waves<__bf16, 2, 4>(b, small, grid, smem, stream, timer)
                              : launch_expand_waves<float, 2, 4>(b, small, grid, smem, stream, timer);
        if (dtype == 1)
            return waves == 2 ? launch_expand_waves<__bf16, 2>(b, small, grid, smem, stream, timer)
                              : launch_expand_waves<__bf16, 4>(b, small, grid, smem, stream, timer);
        return waves == 2   ? launch_expand_waves<float, 2>(b, small, grid, smem, stream, timer)
               : waves == 4 ? launch_expand_waves<float, 4>(b, small, grid, smem, stream, timer)
                            : launch_expand_waves<float, 8>(b, small, grid, smem, stream, timer);
    };
#ifdef LORA_TRACE
    return trace_launch("expand", grid, [&](long long *buf) {
        ExpandArgs b = a;
        b.trace = buf;
        return launch(b);
    });
#else
    return launch(a);
#endif
}

}  // namespace lora

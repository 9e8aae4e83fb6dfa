// The whole runtime flow of Sec. III-B -- gather features, evaluate the decision tree,
// run the chosen kernel -- as a few launches with no host round trip in between:
//
//   1. the feature reduction (one launch for a small matrix, two for a large one);
//      its finishing launch -- a single wave after a first pass, a workgroup for a small
//      matrix -- derives the feature vector on the device, walks the tree (handed over by
//      value in the kernel arguments) and leaves the chosen kernel id in device memory;
//   2. spmv_auto_kernel: one kernel that contains the five CSR schedules that need no
//      preprocessing; every workgroup reads the chosen id and runs that schedule's
//      body (the grid is sized for the reachable schedule that needs the most workgroups,
//      the rest exit);
//   3. from 2^23 nonzeros on (below, cut rows meet inside the product: Meet) spmv_auto_fixup_kernel: the carry
//      fix-up of merge path and of the nonzero split; exits at once unless one of them was chosen, and is not enqueued
//      at all if the host can tell from rows, cols and nnz that the tree cannot answer either.
// When the product's grid is small, steps 1 and 2 share a launch (or, for a small
// matrix, are one launch): see spmv_auto_fused_kernel.  When the known features leave the
// tree a single answer, step 1 is dropped: see spmv_auto_decided_kernel.
//
// The host only enqueues; feature collection costs the reduction kernel itself
// instead of a launch, a wait and a second launch.  The sequence has no host-side
// dependency on device data, so it can be captured in a HIP graph.
//
// The derivation of the floating-point features repeats the host's, operation by
// operation (exact integers, correctly rounded int -> fp64 conversions, one fp64
// division, one rounding to fp32), so both give the same bits.
#include "../../include/seer.h"
#include "features_bodies.hiph"
#include "select_bodies.hiph"
#include "spmv_bodies.hiph"

namespace seer {

// Finishing launch of the selection after a first pass: ONE wave folds the partials, derives
// the features, walks the tree and leaves the record -- no LDS, no barrier (as a workgroup of
// 1024 lanes that met in LDS atomics it took 4.4 us on the timeline).
template <int U>
__global__ __launch_bounds__(kWave) void features_select_wave_kernel(
    int rows, int cols, const int *__restrict__ rp, const FeatPartial *__restrict__ part, uint32_t n_part,
    AutoSel *__restrict__ sel, const AutoHeap heap, uint32_t reachable)
{
    const HeapRegs hr = heap_load(heap);
    const int64_t nnz = (int64_t)rp[rows] - (int64_t)rp[0];
    const FeatTotals t = fold_partials_wave<U>(part, n_part);
    select_in_wave(rows, cols, nnz, t, hr, reachable, sel);
}

// Finishing launch of the selection when it is a launch of its own: the workgroup folds the
// partials of the first pass (or, for a small matrix, reduces row_ptr itself), its first wave
// derives the features, walks the tree and leaves the record.
template <bool VEC>
__global__ __launch_bounds__(kFeatWG) void features_select_heap_kernel(
    int rows, int cols, const int *__restrict__ rp, const FeatPartial *__restrict__ part, uint32_t n_part,
    AutoSel *__restrict__ sel, const AutoHeap heap, uint32_t reachable)
{
    __shared__ FeatLds s;
    HeapRegs hr{};
    int64_t nnz = 0;
    if (threadIdx.x < kWave) {                       // requested before the reduction, used after it
        hr = heap_load(heap);
        nnz = (int64_t)rp[rows] - (int64_t)rp[0];
    }
    const FeatTotals t = features_total<VEC>(rows, rp, part, n_part, &s);
    if (threadIdx.x < kWave) select_in_wave(rows, cols, nnz, t, hr, reachable, sel);
}

template <bool VEC>
__global__ __launch_bounds__(kFeatWG) void features_select_kernel(
    int rows, int cols, const int *__restrict__ rp, const FeatPartial *__restrict__ part, uint32_t n_part,
    AutoSel *__restrict__ sel, const AutoTree tree, uint32_t reachable)
{
    __shared__ FeatLds s;
    __shared__ float s_f[SEER_NUM_FEATURES];
    const FeatTotals t = features_total<VEC>(rows, rp, part, n_part, &s);
    if (threadIdx.x == 0) select_on_device(rows, cols, rp, t, s_f, tree, reachable, sel);
}

static_assert(kFeatMaxParts * sizeof(FeatPartial) <= kAutoSelOffset && sizeof(AutoSel) <= kAutoCarryOffset - kAutoSelOffset,
              "workspace layout");

constexpr int kAutoLdsMpBm = mp_lds_words<kMpIptLarge>() > bm_lds_words<kBmChunk>() ? mp_lds_words<kMpIptLarge>()
                                                                                     : bm_lds_words<kBmChunk>();
constexpr int kAutoLds = kAutoLdsMpBm > bm_lds_words<kWoChunkLarge>() + 2 ? kAutoLdsMpBm
                                                                           : bm_lds_words<kWoChunkLarge>() + 2;
static_assert(bm_lds_words<kWoChunk>() + 2 <= kAutoLds, "CSR,WO's products and its two bounds share the overlay");

// This workgroup's share of schedule k (the same k in every workgroup of the grid).
// RANGED: with gathers ordered by column range (shape.ranges), as the stand-alone kernels.
// LONGS: long rows of CSR,WO may go apart (shape.longs; from 2^23 nonzeros on, where cut rows don't meet); an instance
// of its own, because what that form needs of the arguments leaves too few scalar registers for the others (67 were kept
// in vector lanes, 14 without; a band of 21, 29 M nonzeros, 60.0 and 58.7 us a step).
template <int IPT, bool VEC, bool RANGED = false, bool LONGS = false>
__device__ __forceinline__ void auto_dispatch(
    int k, int rows, int nnz, const int *__restrict__ rp, const int *__restrict__ ci,
    const float *__restrict__ va, const float *__restrict__ x, float *__restrict__ y,
    int *__restrict__ carry_row, float *__restrict__ carry_val, const AutoShape &shape, int remap, int *smem,
    bool no_longs = false /* as in AutoSel */)
{
    static_assert(mp_lds_words<IPT>() <= kAutoLds, "LDS overlay too small");
    const uint32_t n_tiles = shape.tiles[k];
    if (k == SEER_CSR_WM) {
        // The one schedule whose tiles can outnumber the grid (launch_auto caps its share):
        // a workgroup takes every gridDim-th block position; tile_of_block is one-to-one
        // on [0, span), so each tile is still visited exactly once.
        const uint32_t span = remap ? tiles_per_xcd(n_tiles) * kXCD : n_tiles;
        for (uint32_t vb = blockIdx.x; vb < span; vb += gridDim.x) {
            const uint32_t t = tile_of_block(vb, n_tiles, remap);
            if (t >= n_tiles) continue;
            switch (shape.wm_lanes) {
            case 2: wm_body<2>(rows, rp, ci, va, x, y, t); break;
            case 4: wm_body<4>(rows, rp, ci, va, x, y, t); break;
            case 8: wm_body<8>(rows, rp, ci, va, x, y, t); break;
            case 16: wm_body<16>(rows, rp, ci, va, x, y, t); break;
            case 32: wm_body<32>(rows, rp, ci, va, x, y, t); break;
            default: wm_body<64>(rows, rp, ci, va, x, y, t); break;
            }
        }
        return;
    }
    static_assert(RANGED || !LONGS, "long rows go apart where gathers go by range");
    if constexpr (LONGS) {
        if (k == SEER_CSR_WO && !no_longs) {      // (from 2^23 nonzeros on: the larger chunks)
            static_assert(bm_lds_words<kWoChunkLarge>() + 2 <= kAutoLds, "LDS overlay too small");
            wo_long_body<VEC, true>(rows, nnz, rp, ci, va, x, y, n_tiles, remap, reinterpret_cast<float *>(smem),
                                    reinterpret_cast<uint32_t *>(smem) + bm_lds_words<kWoChunkLarge>(), shape.ranges, shape.longs, shape.long_meet);
            return;
        }
    }
    const uint32_t tile = tile_of_block(blockIdx.x, n_tiles, k == SEER_CSR_TM ? (remap && shape.tm_remap) : remap);
    if (tile >= n_tiles) return;
    if (k == SEER_CSR_TM) {
        if (shape.tm_pair) tm_body<true, 2>(rows, nnz, rp, ci, va, x, y, tile);
        else if (shape.tm_short) tm_body<true>(rows, nnz, rp, ci, va, x, y, tile);
        else tm_body<false>(rows, nnz, rp, ci, va, x, y, tile);
    } else if (k == SEER_CSR_BM) {
        float *s_prod = reinterpret_cast<float *>(smem);
        if constexpr (RANGED) {
            static_assert(bm_lds_words<kRangedChunk>() <= kAutoLds, "LDS overlay too small");
            if (shape.bm_ranged) {
                GatherRanges g = shape.ranges;
                g.ticks = shape.bm_ticks;
                bm_body<kRangedChunk, VEC, true, false, false, false, 256, true>(rows, rp, ci, va, x, y, shape.bm_rows,
                                                                                 shape.bm_own_shift, tile, s_prod, g);
                return;
            }
        }
        if (shape.bm_rows <= (int)kWoGroupRows)
            bm_body<kBmChunk, VEC, true, true, false, true, 256>(rows, rp, ci, va, x, y, shape.bm_rows,
                                                                 shape.bm_own_shift, tile, s_prod);
        else   // (the host keeps bm_rows within kAutoBmMaxRows here)
            bm_body<kBmChunk, VEC, true, true, false, false, kAutoBmMaxRows>(rows, rp, ci, va, x, y, shape.bm_rows,
                                                                             shape.bm_own_shift, tile, s_prod);
    } else if (k == SEER_CSR_WO) {
        if (wo_chunk_of(nnz) == kWoChunkLarge)
            wo_body<kWoChunkLarge, VEC, true, RANGED>(rows, nnz, rp, ci, va, x, y, carry_row, carry_val, tile,
                                                      reinterpret_cast<float *>(smem),
                                                      reinterpret_cast<uint32_t *>(smem) + bm_lds_words<kWoChunkLarge>(),
                                                      shape.ranges);
        else
            wo_body<kWoChunk, VEC, true, RANGED>(rows, nnz, rp, ci, va, x, y, carry_row, carry_val, tile,
                                                 reinterpret_cast<float *>(smem),
                                                 reinterpret_cast<uint32_t *>(smem) + bm_lds_words<kWoChunk>(), shape.ranges, shape.meet);
    } else {
        GatherRanges g = shape.ranges;
        g.ticks = shape.mp_ticks;
        mp_body<IPT, VEC, true, RANGED>(rows, nnz, rp, ci, va, x, y, carry_row, carry_val, tile, smem, g, LONGS ? Meet{} : shape.meet);
    }
}

// Eight waves per SIMD take at most 80 scalar registers each (800 in all, in sixteens, sixteen of every wave's the trap handler's):
// with 85 a grid of 1024^2 under CSR,WM took 23.7 us a step instead of 19.2, under CSR,TM 15.6 instead of 15.2.
#define SEER_EIGHT_WAVES __attribute__((amdgpu_num_sgpr(80)))

template <int IPT, bool VEC, bool RANGED = false, bool LONGS = false>
__global__ SEER_EIGHT_WAVES __launch_bounds__(kWG, RANGED ? 8 : 1) void spmv_auto_kernel(
    int rows, int nnz, const int *__restrict__ rp, const int *__restrict__ ci,
    const float *__restrict__ va, const float *__restrict__ x, float *__restrict__ y,
    int *__restrict__ carry_row, float *__restrict__ carry_val, const AutoSel *__restrict__ sel,
    int remap, const AutoShape shape)
{
    __shared__ __attribute__((aligned(16))) int smem[kAutoLds];
    const int k = sel->kernel_id, no_longs = sel->no_longs;              // (one load)
    auto_dispatch<IPT, VEC, RANGED, LONGS>(k, rows, nnz, rp, ci, va, x, y, carry_row, carry_val, shape, remap, smem, no_longs != 0);
}

// The product when the host could decide alone: every leaf the tree can reach from rows,
// cols and nnz names the same kernel, so nothing is gathered.  Workgroup 0 leaves the record
// (valid = 2: no statistics, known features only).
template <int IPT, bool VEC, bool RANGED = false, bool LONGS = false>
__global__ SEER_EIGHT_WAVES __launch_bounds__(kWG, RANGED ? 8 : 1) void spmv_auto_decided_kernel(
    int rows, int nnz, const int *__restrict__ rp, const int *__restrict__ ci,
    const float *__restrict__ va, const float *__restrict__ x, float *__restrict__ y,
    int *__restrict__ carry_row, float *__restrict__ carry_val, AutoSel *__restrict__ sel,
    const AutoSel record, int remap, const AutoShape shape)
{
    __shared__ __attribute__((aligned(16))) int smem[kAutoLds];
    if (blockIdx.x == 0 && threadIdx.x == 0) *sel = record;
    auto_dispatch<IPT, VEC, RANGED, LONGS>(record.kernel_id, rows, nnz, rp, ci, va, x, y, carry_row, carry_val, shape, remap, smem);
}

// Selection inside the product's launch.  The first wave of every workgroup finishes the
// feature reduction for itself -- it folds the up to 64 partials a first pass left (lane <->
// partial, no LDS; for a matrix of at most kAutoFusedRows rows there is no first pass and the
// whole workgroup reduces row_ptr, out of L2 after the first workgroup touched it) -- derives
// the same feature vector, walks the same tree, and hands the kernel id to the other waves
// through LDS; then the workgroup runs its share of the chosen schedule.  The redundant work
// is a few hundred instructions of one wave behind one load of two kilobytes that hits L2,
// while a selection launch costs the path about three microseconds.  Workgroup 0 leaves the
// record for seer_spmv_auto_result and the fix-up kernel.
// Used for grids of up to about a thousand workgroups.  Beyond, it was measured slower than
// the separate launch (a 54 MB stencil: 24.4 us per step against 22.8; the product itself
// 17.2 against 13.0 us, and a first pass of 64 fat workgroups 6.3 against 4.6 us for 512).
// RPU: quads of offsets that a lane reduces per trip where there is no first pass.  Four are all there are of up
// to 4096 rows, and half of the code of eight, which every workgroup runs through for the first time:
// 4096 rows of 16 5.87 -> 5.53 us a step, 1003 rows of 100 6.15 -> 5.80; more rows would take a second trip (5000 14.2 -> 14.6).
template <int IPT, bool VEC, bool RPVEC, uint32_t RPU>
__global__ SEER_EIGHT_WAVES __launch_bounds__(kWG) void spmv_auto_fused_kernel(
    int rows, int cols, int nnz, const int *__restrict__ rp, const int *__restrict__ ci,
    const float *__restrict__ va, const float *__restrict__ x, float *__restrict__ y,
    int *__restrict__ carry_row, float *__restrict__ carry_val, const FeatPartial *__restrict__ part,
    uint32_t n_part, AutoSel *__restrict__ sel, const AutoHeap heap, int remap, const AutoShape shape)
{
    __shared__ __attribute__((aligned(16))) int smem[kAutoLds];
    __shared__ FeatLds s;
    __shared__ int s_k;
    const bool first_wave = threadIdx.x < kWave;
    HeapRegs hr{};
    int64_t nnz_dev = 0;
    FeatTotals t{INT32_MIN, INT32_MAX, 0, 0};
    if (first_wave) {
        hr = heap_load(heap);
        nnz_dev = (int64_t)rp[rows] - (int64_t)rp[0];
    }
    if (n_part == 0) {                                // block-uniform
        features_accumulate_strided<RPVEC, RPU>(rows, rp, threadIdx.x, kWG, t.mx, t.mn, t.sq, t.em);
        t = features_block_fold<kWG>(t.mx, t.mn, t.sq, t.em, &s);
    } else if (first_wave) {
        t = fold_partials_wave(part, n_part);
    }
    if (first_wave) {
        const int k = select_in_wave(rows, cols, nnz_dev, t, hr, shape.reachable, blockIdx.x == 0 ? sel : nullptr);
        if (threadIdx.x == 0) s_k = k;
    }
    __syncthreads();
    auto_dispatch<IPT, VEC>(s_k, rows, nnz, rp, ci, va, x, y, carry_row, carry_val, shape, remap, smem);
}

__global__ __launch_bounds__(kWG) void spmv_auto_fixup_kernel(
    int rows, uint32_t n_mp, uint32_t n_wo, const int *__restrict__ carry_row,
    const float *__restrict__ carry_val, float *__restrict__ y, const AutoSel *__restrict__ sel, bool longs)
{
    const int k = sel->kernel_id, no_longs = sel->no_longs;
    if (k != SEER_CSR_MP && (k != SEER_CSR_WO || (longs && no_longs == 0))) return;      // (beside long rows, cut rows meet)
    mp_fixup_body(rows, k == SEER_CSR_MP ? n_mp : n_wo, carry_row, carry_val, y, blockIdx.x * kWG + threadIdx.x);
}

size_t auto_workspace_bytes(int rows, int nnz)
{
    const size_t mp = mp_workspace_bytes(rows, nnz, kMpIptSmall);
    const size_t wo = carry_workspace_bytes(wo_num_tiles(rows, nnz));
    return kAutoCarryOffset + (mp > wo ? mp : wo);
}

size_t auto_slots_bytes(int rows, int nnz)
{
    const uint32_t mp = mp_num_tiles(rows, nnz, kMpIptSmall), wo = wo_num_tiles(rows, nnz);
    return meet_workspace_bytes(mp > wo ? mp : wo);
}

size_t auto_meet_workspace_bytes(int rows, int nnz)
{
    const size_t least = auto_workspace_bytes(rows, nnz), meet = kAutoCarryOffset + auto_slots_bytes(rows, nnz);
    return meet_applies(rows, nnz) && meet > least ? meet : least;
}

// The first pass ahead of a product that selects for itself: at most kAutoFusedParts
// partials, sixteen rows (four 16-byte loads in flight) per lane and trip; workgroups of
// 1024 lanes once 256-lane ones would need more than one trip.
constexpr uint32_t kAutoFusedOneTrip = kAutoFusedParts * kFeatPartWG * 16u;
static uint32_t launch_fused_partials(const SpmvArgs &a, FeatPartial *part, bool rp_vec, hipStream_t st)
{
    const uint32_t rows = (uint32_t)a.rows;
    if (rows <= kAutoFusedOneTrip) {
        const uint32_t n = (rows + kFeatPartWG * 16u - 1u) / (kFeatPartWG * 16u);
        if (rp_vec) hipLaunchKernelGGL((features_partial_kernel<true, kFeatPartWG, 4>), dim3(n), dim3(kFeatPartWG), 0, st, a.rows, a.rp, part);
        else hipLaunchKernelGGL((features_partial_kernel<false, kFeatPartWG>), dim3(n), dim3(kFeatPartWG), 0, st, a.rows, a.rp, part);
        return n;
    }
    uint32_t n = (rows + kFeatWG * 16u - 1u) / (kFeatWG * 16u);
    n = n > kAutoFusedParts ? kAutoFusedParts : n;
    if (rp_vec) hipLaunchKernelGGL((features_partial_kernel<true, kFeatWG, 4>), dim3(n), dim3(kFeatWG), 0, st, a.rows, a.rp, part);
    else hipLaunchKernelGGL((features_partial_kernel<false, kFeatWG>), dim3(n), dim3(kFeatWG), 0, st, a.rows, a.rp, part);
    return n;
}

void launch_auto(const SpmvArgs &a, const AutoTree &tree, const AutoHeap *heap, const AutoShape &given, bool vec,
                 const AutoPolicy &policy, const AutoSel *decided, void *workspace, void *long_workspace, hipStream_t st)
{
    AutoShape shape = given;
    char *ws = static_cast<char *>(workspace);
    FeatPartial *part = reinterpret_cast<FeatPartial *>(ws);
    AutoSel *sel = reinterpret_cast<AutoSel *>(ws + kAutoSelOffset);
    const uint32_t n_mp = shape.tiles[SEER_CSR_MP], n_wo = shape.tiles[SEER_CSR_WO];
    const uint32_t n_carry = n_mp > n_wo ? n_mp : n_wo;
    const size_t one = carry_workspace_bytes(n_carry) / 2;
    int *carry_row = reinterpret_cast<int *>(ws + kAutoCarryOffset);
    float *carry_val = reinterpret_cast<float *>(ws + kAutoCarryOffset + one);
    const auto reachable = [&](int k) { return ((shape.reachable >> k) & 1u) != 0; };

    // One workgroup per tile of the reachable schedule with the most tiles -- except CSR,WM,
    // whose tiles (64/G rows per wave) can be several times the others': its share is capped at
    // kAutoWmGrid workgroups, or the others' maximum if that is more, and they loop, so that a
    // grid that runs another schedule does not launch thousands of workgroups to no purpose.
    // Where the others alone would let the selection run inside the product's launch, CSR,WM's tiles do not
    // stand in its way: the cap is that launch's limit then (20 011 rows of 20, 1251 of them: 10.8 us a step with
    // a selection launch, now 10.1; a band of 61, 7001 rows, where CSR,WM is chosen and loops: 9.8 and 8.5; 300 x 300 grid 9.0
    // and 8.7).  Only for as many rows as the first pass reads in one trip: a tree of CSR,BM and CSR,WM alone
    // on 250 003 rows of 0 to 6 entries 10.2 and 9.8 us where CSR,BM is chosen, 9.8 to 10.1 and 9.9 where CSR,WM is, on 500 003
    // rows 14.7 and 15.3, 14.6 and 16.8.
    uint32_t grid = 0, wm_grid = 0;
    for (int k = 0; k < SEER_NUM_DIRECT_KERNELS; ++k) {
        if (!reachable(k)) continue;
        const uint32_t g = a.remap ? tiles_per_xcd(shape.tiles[k]) * kXCD : shape.tiles[k];
        if (k == SEER_CSR_WM) wm_grid = g;
        else grid = g > grid ? g : grid;
    }
    if (reachable(SEER_CSR_WM)) {
        const uint32_t least = heap && !shape.ranges.count && grid <= (uint32_t)policy.fused_grid && !decided &&
                                       (uint32_t)a.rows <= kAutoFusedOneTrip
                                   ? (uint32_t)policy.fused_grid : kAutoWmGrid;
        const uint32_t cap = grid > least ? grid : least;
        const uint32_t g = wm_grid < cap ? wm_grid : cap;
        grid = g > grid ? g : grid;
    }
    // The fix-up launch is only enqueued where cut rows do not meet inside the product.  It finds nothing to do unless merge path
    // or the nonzero split ran: it is left out, too, if the tree cannot get to one of them from what the host knows.
    const bool carries = !shape.meet.slots && (reachable(SEER_CSR_MP) || reachable(SEER_CSR_WO));

    if (decided) {
        if (long_workspace && decided->kernel_id == SEER_CSR_WO)
            shape.longs = launch_long(a, LongSelect{}, long_workspace, st);
#define SEER_DECIDED_LAUNCH(...)                                                                           \
    hipLaunchKernelGGL((spmv_auto_decided_kernel<__VA_ARGS__>), dim3(grid), dim3(kWG), 0, st, a.rows, a.nnz, a.rp, \
                       a.ci, a.va, a.x, a.y, carry_row, carry_val, sel, *decided, a.remap, shape)
        if (shape.longs.skip) {
            if (shape.mp_ipt == kMpIptSmall) SEER_DECIDED_LAUNCH(kMpIptSmall, true, true, true);
            else SEER_DECIDED_LAUNCH(kMpIptLarge, true, true, true);
        } else if (shape.ranges.count) {
            if (shape.mp_ipt == kMpIptSmall) SEER_DECIDED_LAUNCH(kMpIptSmall, true, true);
            else SEER_DECIDED_LAUNCH(kMpIptLarge, true, true);
        } else if (shape.mp_ipt == kMpIptSmall) {
            if (vec) SEER_DECIDED_LAUNCH(kMpIptSmall, true); else SEER_DECIDED_LAUNCH(kMpIptSmall, false);
        } else {
            if (vec) SEER_DECIDED_LAUNCH(kMpIptLarge, true); else SEER_DECIDED_LAUNCH(kMpIptLarge, false);
        }
#undef SEER_DECIDED_LAUNCH
        if (carries && !shape.longs.skip)
            launch_carry_fixup(a.rows, decided->kernel_id == SEER_CSR_MP ? n_mp : n_wo, carry_row, carry_val, a.y, st);
        return;
    }

    const bool rp_vec = (reinterpret_cast<uintptr_t>(a.rp) & 15u) == 0;
    if (heap && !shape.ranges.count && (grid <= (uint32_t)policy.fused_grid || a.rows <= policy.fused_max_rows)) {
        // one launch for a small matrix; else a first pass that leaves a few partials
        const uint32_t n_part = a.rows > policy.fused_rows ? launch_fused_partials(a, part, rp_vec, st) : 0u;
#define SEER_FUSED_LAUNCH(I, V, R) SEER_FUSED_LAUNCH_BY(I, V, R, 8)
#define SEER_FUSED_LAUNCH_BY(I, V, R, U)                                                                    \
    hipLaunchKernelGGL((spmv_auto_fused_kernel<I, V, R, U>), dim3(grid), dim3(kWG), 0, st, a.rows, a.cols, a.nnz, \
                       a.rp, a.ci, a.va, a.x, a.y, carry_row, carry_val, part, n_part, sel, *heap, a.remap, shape)
        if (shape.mp_ipt == kMpIptSmall && vec && rp_vec && a.rows <= (int)(kWG * 16u)) {
            SEER_FUSED_LAUNCH_BY(kMpIptSmall, true, true, 4);
        } else if (shape.mp_ipt == kMpIptSmall) {
            if (vec) { if (rp_vec) SEER_FUSED_LAUNCH(kMpIptSmall, true, true); else SEER_FUSED_LAUNCH(kMpIptSmall, true, false); }
            else     { if (rp_vec) SEER_FUSED_LAUNCH(kMpIptSmall, false, true); else SEER_FUSED_LAUNCH(kMpIptSmall, false, false); }
        } else {
            if (vec) { if (rp_vec) SEER_FUSED_LAUNCH(kMpIptLarge, true, true); else SEER_FUSED_LAUNCH(kMpIptLarge, true, false); }
            else     { if (rp_vec) SEER_FUSED_LAUNCH(kMpIptLarge, false, true); else SEER_FUSED_LAUNCH(kMpIptLarge, false, false); }
        }
#undef SEER_FUSED_LAUNCH
#undef SEER_FUSED_LAUNCH_BY
        if (carries)
            hipLaunchKernelGGL(spmv_auto_fixup_kernel, dim3((n_carry + kWG - 1) / kWG), dim3(kWG), 0, st, a.rows, n_mp,
                               n_wo, carry_row, carry_val, a.y, sel, false);
        return;
    }

    // Where CSR,WO may have long rows to leave out, the first pass lists them, too, and the launch that cuts them selects: a matrix
    // without such rows has one launch more than without the stage.
    const bool longs = long_workspace && reachable(SEER_CSR_WO), long_select = longs && heap && policy.select_wave;
    if (long_select) shape.longs = launch_long(a, LongSelect{heap, part, sel, shape.reachable, policy.long_all != 0}, long_workspace, st);
    const uint32_t n_part = features_num_parts(a.rows, policy.part_rows);
    if (n_part && !long_select) launch_feature_partials(a.rows, a.rp, part, n_part, rp_vec, st);
    const bool one_wave = heap && n_part && policy.select_wave;
#define SEER_WAVE_LAUNCH(U)                                                                                 \
    hipLaunchKernelGGL(features_select_wave_kernel<U>, dim3(1), dim3(kWave), 0, st, a.rows, a.cols, a.rp, part, n_part, sel, \
                       *heap, shape.reachable)
#define SEER_SELECT_LAUNCH(V)                                                                               \
    if (heap)                                                                                               \
        hipLaunchKernelGGL(features_select_heap_kernel<V>, dim3(1), dim3(kFeatWG), 0, st, a.rows, a.cols, a.rp, part, \
                           n_part, sel, *heap, shape.reachable);                                            \
    else                                                                                                    \
        hipLaunchKernelGGL(features_select_kernel<V>, dim3(1), dim3(kFeatWG), 0, st, a.rows, a.cols, a.rp, part, n_part, \
                           sel, tree, shape.reachable)
    if (long_select) {
    } else if (one_wave) {
        if (fold_eight(n_part)) SEER_WAVE_LAUNCH(8); else SEER_WAVE_LAUNCH(4);
    } else if (rp_vec) {
        SEER_SELECT_LAUNCH(true);
    } else {
        SEER_SELECT_LAUNCH(false);
    }
#undef SEER_WAVE_LAUNCH
#undef SEER_SELECT_LAUNCH

    if (longs && !long_select) shape.longs = launch_long(a, LongSelect{nullptr, nullptr, sel, 0, policy.long_all != 0}, long_workspace, st);
#define SEER_AUTO_LAUNCH(...)                                                                              \
    hipLaunchKernelGGL((spmv_auto_kernel<__VA_ARGS__>), dim3(grid), dim3(kWG), 0, st, a.rows, a.nnz, a.rp, a.ci, \
                       a.va, a.x, a.y, carry_row, carry_val, sel, a.remap, shape)
    if (shape.longs.skip) {
        if (shape.mp_ipt == kMpIptSmall) SEER_AUTO_LAUNCH(kMpIptSmall, true, true, true);
        else SEER_AUTO_LAUNCH(kMpIptLarge, true, true, true);
    } else if (shape.ranges.count) {
        if (shape.mp_ipt == kMpIptSmall) SEER_AUTO_LAUNCH(kMpIptSmall, true, true);
        else SEER_AUTO_LAUNCH(kMpIptLarge, true, true);
    } else if (shape.mp_ipt == kMpIptSmall) {
        if (vec) SEER_AUTO_LAUNCH(kMpIptSmall, true); else SEER_AUTO_LAUNCH(kMpIptSmall, false);
    } else {
        if (vec) SEER_AUTO_LAUNCH(kMpIptLarge, true); else SEER_AUTO_LAUNCH(kMpIptLarge, false);
    }
#undef SEER_AUTO_LAUNCH
    if (carries)
        hipLaunchKernelGGL(spmv_auto_fixup_kernel, dim3((n_carry + kWG - 1) / kWG), dim3(kWG), 0, st, a.rows, n_mp,
                           n_wo, carry_row, carry_val, a.y, sel, longs);
}

} // namespace seer

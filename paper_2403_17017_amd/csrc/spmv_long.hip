// The long rows of CSR,WO's largest matrices, with slabs of x in LDS.
// In a matrix of hundreds of millions of nonzeros and skewed row lengths most nonzeros lie in
// rows of thousands of entries with columns all over x, and CSR,WO gathers them out of L2, one
// 128-byte request each (Zipf rows, s = 1.6, 2 M columns, 480 M nonzeros: 200 G/s, a third of the rate at
// which the entries could be read).  Here such rows are cut into slabs of x that LDS holds (2^15 columns)
// without any preparation: a search per row and slab finds the cuts, one launch takes the pieces
// of a slab in all long rows with that slab in LDS, a last one adds up each row's pieces, in
// slab order.  CSR,WO takes the rest: it is told per chunk which entries belong to a long row.
//
// A row is long from 32 entries per slab on, if it crosses a chunk boundary, and if its columns at a
// quarter, half and three quarters of it are within a sixteenth of x of where ascending columns spread
// evenly would be: then its pieces are of about equal size, and the tasks below are balanced.
// The cuts are right for any order of columns: a cut is a place in the row, cuts never descend
// (each is raised to the ones before it), and an entry whose column lies outside the slab of its piece
// is gathered from x.
// 472 M nonzeros, Zipf s = 1.6: list 10 us, cuts 80, products 598 (nine tenths of the nonzeros, read at 5.7 TB/s),
// CSR,WO over the rest and the sums 415; all of them by CSR,WO 2370.  Tried: rows from 16 entries per slab on, the same
// with twice the scratch memory; a wave per piece from 128 entries on, 1289 in all against 1255 at the time.
// CSR,WO over the rest took 513 while every chunk had a workgroup, to find nothing in four of five, and its gather
// ranges lasted as long as full chunks need.
#include "features_bodies.hiph"
#include "select_bodies.hiph"
#include "spmv_bodies.hiph"

namespace seer {

constexpr uint32_t kLongShift = 15;
constexpr uint32_t kLongCols = 1u << kLongShift;    // columns per slab: 128 KB of LDS
constexpr uint32_t kLongWG = 1024;
constexpr uint32_t kLongGrid = 256;                 // workgroups of long_multiply_kernel: one per CU
constexpr uint32_t kLongCutGrid = 512;              // ... of long_cut_kernel: two per CU
constexpr uint32_t kLongListWG = 512;
constexpr uint32_t kLongRows = 4096;                // rows per workgroup of long_list_kernel
// Rows by the length of their pieces: 8 lanes, 16 lanes and a wave take a piece of class 0 (32 entries on
// average and more), 1 (64) and 2 (256).
constexpr uint32_t kLongClasses = 3;
__host__ __device__ inline uint32_t long_class_piece(uint32_t k) { return k == 0 ? 32u : k == 1 ? 64u : 256u; }

struct LongRow { uint32_t row, start, end, pad; };

static uint32_t long_slabs(int cols) { return ((uint32_t)cols + kLongCols - 1u) >> kLongShift; }

// ---- 1: the long rows of every 4096 rows into the workgroup's part of a list, and the words per chunk of
// CSR,WO to zero.  A part is placed by the nonzeros before it, so that none runs into the next and nothing is
// counted by atomics (a list per class filled that way took 13 us and a launch to clear its counters, 2 M rows; this 9).
__host__ __device__ inline uint32_t long_part(uint32_t nnz_before, uint32_t least, uint32_t part) { return nnz_before / least + part; }

struct LongPart { uint32_t n[kLongClasses], first, entries, whole, pad[2]; };   // rows of each class, where they lie in the list;
                                                                                // their entries and the chunks that hold nothing else
static_assert(sizeof(LongPart) == 32, "two 16-byte loads");

// FEATURES: the pass over the offsets leaves the feature partials (features_partial_kernel), too.  VEC: row_ptr lies on 16 bytes.
template <bool FEATURES, bool VEC>
__global__ __launch_bounds__(kLongListWG) void long_list_kernel(
    int rows, uint32_t cols, uint32_t n_slabs, const int *__restrict__ rp, const int *__restrict__ ci,
    LongPart *__restrict__ parts, LongRow *__restrict__ list, LongNumbers *__restrict__ numbers, uint32_t *__restrict__ skip_words,
    uint32_t n_skip, FeatPartial *__restrict__ features, const AutoSel *__restrict__ sel)
{
    // a row found: its place in the part, later its class and its number in that class, too
    constexpr uint32_t kClassAt = 12, kNumberAt = 14;
    static_assert(kLongRows == 1u << kClassAt && kLongClasses < 4u, "12 + 2 + 13 bits");
    __shared__ uint32_t s_row[kLongRows], s_n, s_class[kLongClasses], s_entries, s_whole;
    if (sel && sel->kernel_id != SEER_CSR_WO) return;
    const uint32_t r0 = blockIdx.x * kLongRows, tid = threadIdx.x, r1 = min(r0 + kLongRows, (uint32_t)rows);
    if (tid == 0) s_n = s_entries = s_whole = 0;
    if (blockIdx.x == 0 && tid == 0) *numbers = LongNumbers{};
    if (tid < kLongClasses) s_class[tid] = 0;
    for (uint32_t i = blockIdx.x * kLongListWG + tid; i < n_skip; i += gridDim.x * kLongListWG) skip_words[i] = 0;
    __syncthreads();
    const uint32_t least = long_class_piece(0) * n_slabs;
    int32_t mx = INT32_MIN, mn = INT32_MAX;
    uint64_t sq = 0;
    uint32_t em = 0;
    const auto take = [&](uint32_t at, uint32_t a, uint32_t e) {
        if constexpr (FEATURES) take_row((int32_t)(e - a), mx, mn, sq, em);
        if (e - a >= least && a / kWoChunkLarge != (e - 1u) / kWoChunkLarge) s_row[atomicAdd(&s_n, 1u)] = at;
    };
    if constexpr (VEC) {                                        // four rows per load, and the next one's offset
        constexpr uint32_t U = kLongRows / 4u / kLongListWG;
        v4i v[U];
        int next[U];
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            const uint32_t r = min(r0 + 4u * (j * kLongListWG + tid), (uint32_t)rows & ~3u);
            const bool in = r + 4u <= r1;
            v[j] = in ? *reinterpret_cast<const v4i *>(rp + r) : v4i{0, 0, 0, 0};
            next[j] = in ? rp[r + 4u] : 0;
        }
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            const uint32_t at = 4u * (j * kLongListWG + tid);
            if (r0 + at + 4u > r1) continue;
            take(at, (uint32_t)v[j].x, (uint32_t)v[j].y);
            take(at + 1u, (uint32_t)v[j].y, (uint32_t)v[j].z);
            take(at + 2u, (uint32_t)v[j].z, (uint32_t)v[j].w);
            take(at + 3u, (uint32_t)v[j].w, (uint32_t)next[j]);
        }
        const uint32_t at = ((r1 - r0) & ~3u) + tid;            // the last three rows of the matrix
        if (r0 + at < r1) take(at, (uint32_t)rp[r0 + at], (uint32_t)rp[r0 + at + 1u]);
    } else {
        for (uint32_t at = tid; r0 + at < r1; at += kLongListWG) take(at, (uint32_t)rp[r0 + at], (uint32_t)rp[r0 + at + 1u]);
    }
    FeatTotals t{};
    if constexpr (FEATURES) {
        __shared__ FeatLds s_feat;
        t = features_block_fold<kLongListWG>(mx, mn, sq, em, &s_feat);
    }
    __syncthreads();
    const uint32_t n = s_n;
    for (uint32_t i = tid; i < n; i += kLongListWG) {
        const uint32_t at = s_row[i], a = (uint32_t)rp[r0 + at], e = (uint32_t)rp[r0 + at + 1u], len = e - a;
        bool spread = true;
#pragma unroll
        for (uint32_t q = 1; q < 4; ++q) {
            const int64_t want = (int64_t)(cols / 4u) * q, got = ci[a + (uint32_t)((uint64_t)len * q / 4u)];
            spread = spread && (got > want ? got - want : want - got) <= (int64_t)(cols / 16u);
        }
        uint32_t k = kLongClasses, j = 0;
        if (spread) {
            k = len >= long_class_piece(2) * n_slabs ? 2u : len >= long_class_piece(1) * n_slabs ? 1u : 0u;
            j = atomicAdd(&s_class[k], 1u);
            atomicAdd(&s_entries, len);
            atomicAdd(&s_whole, (e - 1u) / kWoChunkLarge - a / kWoChunkLarge - 1u);
        }
        s_row[i] = at | k << kClassAt | j << kNumberAt;
    }
    __syncthreads();
    const uint32_t first = long_part(r0 < r1 ? (uint32_t)rp[r0] : 0u, least, blockIdx.x);
    if (FEATURES && tid == 0) features[blockIdx.x] = FeatPartial{t.mx, t.mn, t.sq, t.em, s_entries};
    if (tid == 0) parts[blockIdx.x] = LongPart{{s_class[0], s_class[1], s_class[2]}, first, s_entries, s_whole, {0, 0}};
    for (uint32_t i = tid; i < n; i += kLongListWG) {
        const uint32_t w = s_row[i], k = w >> kClassAt & 3u, row = r0 + (w & (kLongRows - 1u));
        if (k == kLongClasses) continue;
        const uint32_t before = (k > 0u ? s_class[0] : 0u) + (k > 1u ? s_class[1] : 0u);
        list[first + before + (w >> kNumberAt)] = LongRow{row, (uint32_t)rp[row], (uint32_t)rp[row + 1u], 0u};
    }
}

// ---- 2: the cuts.  The parts of the list, class by class, make one order of all long rows: number j of the
// first part's class 0 row, then the next part's ..., then class 1, class 2.  Every workgroup finds
// the parts' first numbers for itself (s_from).  Returns N, the number of long rows, and their entries and whole
// chunks.  kLongWG lanes; parts > 0.
constexpr uint32_t kLongWaves = kLongWG / kWave, kLongSums = (kLongClasses + 2u) * kLongWaves;
constexpr uint32_t kLongParts = 1024;                // of the list, at most: 4 M rows (long_rows_fit)
__device__ __forceinline__ uint32_t long_numbers(
    uint32_t parts, const LongPart *__restrict__ of, uint32_t *s_from /* LDS [kLongClasses * parts + 1] */,
    uint32_t *s_w /* LDS [kLongSums] */, uint32_t *s_n /* LDS [kLongClasses]: rows of each class */,
    uint32_t &entries, uint32_t &whole)
{
    constexpr uint32_t E = kLongParts / kLongWG;
    const uint32_t tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    LongPart c[E];                                               // of consecutive parts, all fetched at once
#pragma unroll
    for (uint32_t i = 0; i < E; ++i) {
        c[i] = of[min(tid * E + i, parts - 1u)];
        if (tid * E + i >= parts) c[i] = LongPart{};
    }
    constexpr uint32_t K = kLongClasses + 2u;                    // (the last two: sums only)
    uint32_t v[K][E], incl[K], sum[K];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
        sum[k] = 0;
#pragma unroll
        for (uint32_t i = 0; i < E; ++i) {
            v[k][i] = sum[k];
            sum[k] += k < kLongClasses ? c[i].n[k] : k == kLongClasses ? c[i].entries : c[i].whole;
        }
        incl[k] = sum[k];
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t up = (uint32_t)__shfl_up((int)incl[k], off);
            if ((int)lane >= off) incl[k] += up;
        }
        if (lane == kWave - 1) s_w[k * kLongWaves + wave] = incl[k];
    }
    __syncthreads();
    uint32_t run = 0;
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
        uint32_t before = run + incl[k] - sum[k], all = 0;
#pragma unroll
        for (uint32_t w = 0; w < kLongWaves; ++w) {
            const uint32_t of_wave = s_w[k * kLongWaves + w];
            before += w < wave ? of_wave : 0u;
            all += of_wave;
        }
        if (k < kLongClasses) {
#pragma unroll
            for (uint32_t i = 0; i < E; ++i)
                if (tid * E + i < parts) s_from[k * parts + tid * E + i] = before + v[k][i];
            if (tid == 0) s_n[k] = all;
            run += all;
        } else if (k == kLongClasses) {
            entries = all;
        } else {
            whole = all;
        }
    }
    if (tid == 0) s_from[kLongClasses * parts] = run;
    __syncthreads();
    return run;
}

// Wave <-> row, lane <-> slab: cut[s * N + j] = first place of slab s in row j.  The search begins where the
// column would be if the row's columns were spread evenly, comes nearer twice by the distance of the column
// found, then widens in steps that double; every one ends at the row's ends at the latest.  The words per
// chunk are set here, too, and the rows listed by number for the last pass.
// SELECT: the selection is made here (every workgroup for itself if there are long rows, the first one leaves the
// record), from one partial per part.  Where the device selects, here or before, long rows of fewer than kLongLeast entries
// together stay where they are: cutting them and a launch for their pieces take some 25 us, a gather saved 4.5 ps (4 M rows, Zipf s = 2.0, 12 M such entries:
// 300 and 280 us a step; s = 2.3, 0.6 M: 140 and 179).
constexpr uint32_t kLongLeast = 1u << 23;
struct LongFeatures { int rows; const int *rp; const FeatPartial *part; uint32_t reachable, least /* entries of long rows for them to go apart */; };

template <bool SELECT>
__global__ __launch_bounds__(kLongWG) void long_cut_kernel(
    uint32_t cols, uint32_t nnz, uint32_t n_slabs, uint32_t parts, const int *__restrict__ ci, const LongPart *__restrict__ of,
    const LongRow *__restrict__ list, LongNumbers *__restrict__ numbers, uint32_t ticks, uint32_t *__restrict__ rows_by_number,
    uint32_t *__restrict__ cut, LongSkip *__restrict__ skip, AutoSel *__restrict__ sel, const LongFeatures f, const AutoHeap heap)
{
    __shared__ uint32_t s_from[kLongClasses * kLongParts + 1], s_w[kLongSums], s_n[kLongClasses];
    if (!SELECT && sel && sel->kernel_id != SEER_CSR_WO) return;
    if constexpr (SELECT) {
        // The first wave selects; of too few long rows the first workgroup says that there are none, the others have nothing to do.
        if (threadIdx.x < kWave) {
            const HeapRegs hr = heap_load(heap);
            const int64_t nnz_dev = (int64_t)f.rp[f.rows] - (int64_t)f.rp[0];
            uint32_t in_all = 0;
            const FeatTotals t = fold_partials_wave<8, true>(f.part, parts, &in_all);
            const bool few = in_all < f.least;
            bool go = !few;
            if (!few || blockIdx.x == 0)
                go = select_in_wave(f.rows, (int)cols, nnz_dev, t, hr, f.reachable, blockIdx.x == 0 ? sel : nullptr) == SEER_CSR_WO && !few;
            if (threadIdx.x == 0) {
                s_w[0] = go;
                if (blockIdx.x == 0 && !go) {
                    numbers->all = 0;
                    sel->no_longs = 1;
                }
            }
        }
        __syncthreads();
        if (s_w[0] == 0) return;
        __syncthreads();
    }
    uint32_t entries = 0, whole = 0;
    const uint32_t N = long_numbers(parts, of, s_from, s_w, s_n, entries, whole);
    if (!SELECT && sel && entries < f.least) {                   // (their number is zero since the launch before)
        if (blockIdx.x == 0 && threadIdx.x == 0) sel->no_longs = 1;
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        for (uint32_t k = 0; k < kLongClasses; ++k) numbers->n[k] = s_n[k];
        numbers->all = N;
        // A turn over the ranges has to last as long as the gathers under way take, and the chunks of CSR,WO that have something
        // left are no longer full (Zipf, s = 1.6: 24 000 of 119 000, of 4096 entries 2000).
        const uint32_t chunks = (nnz + kWoChunkLarge - 1u) / kWoChunkLarge, left = max(chunks - min(whole, chunks), 1u);
        numbers->ticks = max((uint32_t)((uint64_t)ticks * (nnz - entries) / ((uint64_t)left * kWoChunkLarge)), 1u);
    }
    const uint32_t lane = threadIdx.x % kWave, waves = gridDim.x * kLongWaves;
    for (uint32_t j = blockIdx.x + threadIdx.x / kWave * gridDim.x; j < N; j += waves) {      // (few rows: on all CUs)
        uint32_t lo_f = 0, hi_f = kLongClasses * parts;         // the last part whose first number is at most j
        while (lo_f + 1u < hi_f) {
            const uint32_t mid = (lo_f + hi_f) / 2u;
            if (s_from[mid] <= j) lo_f = mid; else hi_f = mid;
        }
        const uint32_t k = lo_f / parts, part = lo_f - k * parts;
        const LongPart c = of[part];
        const LongRow r = list[c.first + (k > 0u ? c.n[0] : 0u) + (k > 1u ? c.n[1] : 0u) + (j - s_from[lo_f])];
        const uint32_t len = r.end - r.start;
        if (lane == 0) rows_by_number[j] = r.row;
        {
            const uint32_t first = r.start / kWoChunkLarge, last = (r.end - 1u) / kWoChunkLarge;
            if (lane == 0) {
                // (chunk 0 still has the empty rows before its first nonzero to write)
                if (r.start % kWoChunkLarge == 0 && r.start > 0u) skip[first].head = kLongWhole | kWoChunkLarge;
                else skip[first].tail = (uint16_t)(kWoChunkLarge - r.start % kWoChunkLarge);
                skip[last].head = (uint16_t)(r.end - last * kWoChunkLarge);
            }
            for (uint32_t t = first + 1u + lane; t < last; t += kWave) skip[t].head = kLongWhole | kWoChunkLarge;
        }
        const float scale = (float)len / (float)cols;
        uint32_t most = r.start;                                // of the cuts before these 64
        for (uint32_t s0 = 0; s0 <= n_slabs; s0 += kWave) {
            const uint32_t s = s0 + lane;
            uint32_t at = r.start;
            if (s >= n_slabs) {
                at = r.end;
            } else if (s > 0) {
                const int key = (int)(s << kLongShift);         // (s < n_slabs: below cols)
                uint32_t lo = r.start, hi = r.end, step = 4;    // the cut is in [lo, hi]
                int p = (int)((float)key * scale);              // from the row's start
                p = min(max(p, 0), (int)len - 1);
                int c = ci[r.start + (uint32_t)p];
#pragma unroll
                for (int near = 0; near < 2; ++near) {
                    p = min(max(p + (int)((float)(key - c) * scale), 0), (int)len - 1);
                    c = ci[r.start + (uint32_t)p];
                }
                if (c < key) {
                    lo = r.start + (uint32_t)p + 1u;
                    while (lo < hi) {                           // (each turn raises lo or ends)
                        const uint32_t q = min(lo + step, r.end - 1u);
                        if (ci[q] >= key) { hi = q; break; }
                        lo = q + 1u;
                        step *= 2u;
                    }
                } else {
                    hi = r.start + (uint32_t)p;
                    while (lo < hi) {                           // (each turn lowers hi or ends)
                        const uint32_t q = hi - lo > step ? hi - step : lo;
                        if (ci[q] < key) { lo = q + 1u; break; }
                        hi = q;
                        step *= 2u;
                    }
                }
                while (lo < hi) {
                    const uint32_t mid = lo + (hi - lo) / 2u;
                    if (ci[mid] < key) lo = mid + 1u; else hi = mid;
                }
                at = lo;
            }
            at = max(at, most);
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t up = (uint32_t)__shfl_up((int)at, off);
                if ((int)lane >= off) at = max(at, up);
            }
            if (s <= n_slabs) cut[(size_t)s * N + j] = at;
            most = (uint32_t)__shfl((int)at, kWave - 1);
        }
    }
}

// ---- 3: the pieces.  Task (slab, q) takes every Q-th row's piece in the slab; G lanes take a piece, four
// entries a lane at a time, twice.
template <uint32_t G>
__device__ __forceinline__ void long_pieces(
    uint32_t j0, uint32_t n, uint32_t q, uint32_t Q, uint32_t N, uint32_t s, uint32_t c0, uint32_t nc, uint32_t nnz,
    const int *__restrict__ ci, const float *__restrict__ va, const float *__restrict__ x, const float *__restrict__ s_x,
    const uint32_t *__restrict__ cut, float *__restrict__ part, uint32_t *s_next /* LDS; G = 64 */)
{
    constexpr uint32_t U = 2, kGroups = kLongWG / G;
    const uint32_t lg = threadIdx.x % G, group = threadIdx.x / G;
    const uint32_t *lo = cut + (size_t)s * N + j0, *hi = lo + N;
    const uint32_t stride = Q * kGroups;
    // Pieces for a whole wave differ the most in length, 256 to 3300 entries: a wave takes the next one when it is through with
    // the last.  With every sixteenth piece for each wave: 472 M nonzeros 680 us instead of 598, 53 M 106 and 96, 46 M 66 and 61.
    const auto grab = [&] {
        uint32_t g = 0;
        if (threadIdx.x % kWave == 0) g = atomicAdd(s_next, 1u);
        return q + Q * (uint32_t)__builtin_amdgcn_readfirstlane((int)g);
    };
    uint32_t i = G == kWave ? grab() : q + Q * group;
    uint32_t a = i < n ? lo[i] : 0u, e = i < n ? hi[i] : 0u;
    // whole waves go on together (the sum below is over lanes): until no group of the wave has a piece
    while (__ballot(i < n)) {
        const uint32_t next = G == kWave ? grab() : i + stride;
        const uint32_t na = next < n ? lo[next] : 0u, ne = next < n ? hi[next] : 0u;
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (uint32_t k0 = a + 4u * lg; k0 < e; k0 += 4u * G * U) {
            v4i c[U];
            v4f v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t k = k0 + u * 4u * G;
                c[u] = v4i{0, 0, 0, 0};
                v[u] = v4f{0.f, 0.f, 0.f, 0.f};
                if (k + 4u <= nnz) {
                    if (k < e) {
                        c[u] = __builtin_nontemporal_load(reinterpret_cast<const v4i_a4 *>(ci + k));
                        v[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f_a4 *>(va + k));
                    }
                } else {                                        // the last three entries of the matrix
                    if (k < e) { c[u].x = ci[k]; v[u].x = va[k]; }
                    if (k + 1u < e) { c[u].y = ci[k + 1u]; v[u].y = va[k + 1u]; }
                    if (k + 2u < e) { c[u].z = ci[k + 2u]; v[u].z = va[k + 2u]; }
                }
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t k = k0 + u * 4u * G;
                const uint32_t cc[4] = {(uint32_t)c[u].x, (uint32_t)c[u].y, (uint32_t)c[u].z, (uint32_t)c[u].w};
                const float vv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (uint32_t w = 0; w < 4; ++w) {
                    if (k + w >= e) continue;
                    const uint32_t o = cc[w] - c0;
                    const float xv = o < nc ? s_x[o] : x[cc[w]];
                    t[w] += vv[w] * xv;
                }
            }
        }
        const float sum = group_sum<(int)G>((t[0] + t[1]) + (t[2] + t[3]));
        if (i < n && lg == 0) part[(size_t)s * N + j0 + i] = sum;
        i = next;
        a = na;
        e = ne;
    }
}

__global__ __launch_bounds__(kLongWG) void long_multiply_kernel(
    uint32_t cols, uint32_t nnz, uint32_t n_slabs, uint32_t Q, const int *__restrict__ ci, const float *__restrict__ va,
    const float *__restrict__ x, LongNumbers *__restrict__ numbers, const uint32_t *__restrict__ cut,
    float *__restrict__ part, const LongSkip *__restrict__ skip, uint32_t chunks, uint32_t *__restrict__ active,
    const AutoSel *__restrict__ sel)
{
    __shared__ __attribute__((aligned(16))) float s_x[kLongCols];
    __shared__ uint32_t s_next;
    if (sel && sel->kernel_id != SEER_CSR_WO) return;
    const uint32_t n[kLongClasses] = {numbers->n[0], numbers->n[1], numbers->n[2]}, N = numbers->all, tid = threadIdx.x;
    if (N == 0) return;
    // The chunks that have something left are listed, workgroup after workgroup as they come (which workgroup of CSR,WO takes
    // a chunk does not show in y); one addition each to the common count, for these are served one after the other.
    uint32_t *s_w = reinterpret_cast<uint32_t *>(s_x);
    for (uint32_t c0 = blockIdx.x * kLongWG; c0 < chunks; c0 += gridDim.x * kLongWG) {
        const uint32_t c = c0 + tid, lane = tid % kWave;
        const bool in = c < chunks && (skip[c].head & kLongWhole) == 0;
        const uint64_t left = __ballot(in);
        if (lane == 0) s_w[tid / kWave] = (uint32_t)__popcll(left);
        __syncthreads();
        if (tid < kWave) {
            const uint32_t mine = lane < kLongWaves ? s_w[lane] : 0u;
            uint32_t incl = mine;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t up = (uint32_t)__shfl_up((int)incl, off);
                if ((int)lane >= off) incl += up;
            }
            uint32_t base = 0;
            if (lane == kWave - 1) base = atomicAdd(&numbers->active, incl);
            base = (uint32_t)__builtin_amdgcn_readlane((int)base, kWave - 1);
            if (lane < kLongWaves) s_w[lane] = base + incl - mine;
        }
        __syncthreads();
        if (in) active[s_w[tid / kWave] + (uint32_t)__popcll(left & ((1ull << lane) - 1ull))] = c;
        __syncthreads();
    }
    for (uint32_t task = tile_of_block(blockIdx.x, gridDim.x, 1); task < n_slabs * Q; task += gridDim.x) {
        const uint32_t s = task / Q, q = task - s * Q;
        const uint32_t c0 = s << kLongShift, nc = min(cols - c0, kLongCols);
        __syncthreads();                                        // the slab before has been used
        if (tid == 0) s_next = 0;
        {
            v4f t[kLongCols / 4u / kLongWG];
#pragma unroll
            for (uint32_t m = 0; m < kLongCols / 4u / kLongWG; ++m) {
                const uint32_t k = 4u * (m * kLongWG + tid);
                t[m] = v4f{0.f, 0.f, 0.f, 0.f};
                if (k + 4u <= nc) {
                    t[m] = *reinterpret_cast<const v4f_a4 *>(x + c0 + k);
                } else {
                    if (k < nc) t[m].x = x[c0 + k];
                    if (k + 1u < nc) t[m].y = x[c0 + k + 1u];
                    if (k + 2u < nc) t[m].z = x[c0 + k + 2u];
                }
            }
#pragma unroll
            for (uint32_t m = 0; m < kLongCols / 4u / kLongWG; ++m)
                *reinterpret_cast<v4f *>(s_x + 4u * (m * kLongWG + tid)) = t[m];
        }
        __syncthreads();
        long_pieces<64>(n[0] + n[1], n[2], q, Q, N, s, c0, nc, nnz, ci, va, x, s_x, cut, part, &s_next);
        long_pieces<16>(n[0], n[1], q, Q, N, s, c0, nc, nnz, ci, va, x, s_x, cut, part, &s_next);
        long_pieces<8>(0u, n[0], q, Q, N, s, c0, nc, nnz, ci, va, x, s_x, cut, part, &s_next);
    }
}

// ------------------------------------------------------------------ host side
static size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }

struct LongLayout { size_t slots, numbers, counts, skip, active, list, rows, cut, part, total; uint32_t parts, skip_words; };
static LongLayout long_layout(int rows, uint32_t nnz, uint32_t n_slabs)
{
    LongLayout L;
    const size_t tiles = ((size_t)nnz + kWoChunkLarge - 1) / kWoChunkLarge;
    const size_t most = nnz / (long_class_piece(0) * n_slabs);                        // long rows
    size_t o = 0;
    L.parts = ((uint32_t)rows + kLongRows - 1) / kLongRows;
    L.skip_words = (uint32_t)(tiles * sizeof(LongSkip) / 4);
    L.slots = o;     o += pad256(auto_slots_bytes(rows, (int)nnz));      // (first: the callers know them there)
    L.numbers = o;   o += 256;
    L.counts = o;    o += pad256((size_t)L.parts * sizeof(LongPart));
    L.skip = o;      o += pad256((size_t)L.skip_words * 4);
    L.active = o;    o += pad256(tiles * 4);
    L.list = o;      o += pad256((most + L.parts) * sizeof(LongRow));
    L.rows = o;      o += pad256(most * 4 + 4);
    L.cut = o;       o += pad256(((size_t)n_slabs + 1) * most * 4 + 4);
    L.part = o;      o += pad256((size_t)n_slabs * most * 4 + 4);
    L.total = o;
    return L;
}

bool long_rows_fit(int rows) { return rows > 0 && ((uint32_t)rows + kLongRows - 1) / kLongRows <= kLongParts; }
size_t long_workspace_bytes(int rows, int cols, int nnz) { return long_layout(rows, (uint32_t)nnz, long_slabs(cols)).total; }
// For any number of slabs from two on: 24 bytes per long row, of which there are at most nnz / 64, and 8 bytes for
// each of at most nnz / 32 pieces.
size_t long_workspace_most(int rows, int nnz)
{
    const size_t n = (size_t)nnz, parts = ((size_t)rows + kLongRows - 1) / kLongRows;
    return auto_slots_bytes(rows, nnz) + 24 * (n / 64) + 8 * (n / 32) + (n / kWoChunkLarge + 1) * (sizeof(LongSkip) + 4) + 48 * parts + 8192;
}

LongStage launch_long(const SpmvArgs &a, const LongSelect &select, void *workspace, hipStream_t st)
{
    const uint32_t S = long_slabs(a.cols), nnz = (uint32_t)a.nnz;
    const LongLayout L = long_layout(a.rows, nnz, S);
    char *base = static_cast<char *>(workspace);
    LongNumbers *numbers = reinterpret_cast<LongNumbers *>(base + L.numbers);
    LongPart *of = reinterpret_cast<LongPart *>(base + L.counts);
    LongSkip *skip = reinterpret_cast<LongSkip *>(base + L.skip);
    uint32_t *active = reinterpret_cast<uint32_t *>(base + L.active);
    LongRow *list = reinterpret_cast<LongRow *>(base + L.list);
    uint32_t *rows = reinterpret_cast<uint32_t *>(base + L.rows), *cut = reinterpret_cast<uint32_t *>(base + L.cut);
    float *part = reinterpret_cast<float *>(base + L.part);
    const bool vec = (reinterpret_cast<uintptr_t>(a.rp) & 15u) == 0;
    const AutoSel *made = select.heap ? nullptr : select.sel;    // (for the first two launches)
#define SEER_LIST_LAUNCH(F, V)                                                                                       \
    hipLaunchKernelGGL((long_list_kernel<F, V>), dim3(L.parts), dim3(kLongListWG), 0, st, a.rows, (uint32_t)a.cols, S, a.rp, a.ci, of, list, \
                       numbers, reinterpret_cast<uint32_t *>(skip), L.skip_words, select.part, made)
    if (select.heap) { if (vec) SEER_LIST_LAUNCH(true, true); else SEER_LIST_LAUNCH(true, false); }
    else             { if (vec) SEER_LIST_LAUNCH(false, true); else SEER_LIST_LAUNCH(false, false); }
#undef SEER_LIST_LAUNCH
    const LongFeatures f{a.rows, a.rp, select.part, select.reachable, select.all ? 1u : kLongLeast};
#define SEER_CUT_LAUNCH(S_, H)                                                                                       \
    hipLaunchKernelGGL(long_cut_kernel<S_>, dim3(kLongCutGrid), dim3(kLongWG), 0, st, (uint32_t)a.cols, nnz, S, L.parts, a.ci, \
                       static_cast<const LongPart *>(of), static_cast<const LongRow *>(list), numbers, a.ranges.ticks, rows, cut, skip, \
                       select.sel, f, H)
    if (select.heap) SEER_CUT_LAUNCH(true, *select.heap); else SEER_CUT_LAUNCH(false, AutoHeap{});
#undef SEER_CUT_LAUNCH
    // tasks per slab: so many that the tasks fill whole rounds of the grid best
    uint32_t Q = 1;
    double best = 0.0;
    for (uint32_t q = 1; q <= 8; ++q) {
        const uint32_t tasks = S * q, rounds = (tasks + kLongGrid - 1) / kLongGrid;
        const double filled = (double)tasks / ((double)rounds * kLongGrid);
        if (rounds <= 4 && filled > best + 0.01) { best = filled; Q = q; }
    }
    hipLaunchKernelGGL(long_multiply_kernel, dim3(kLongGrid), dim3(kLongWG), 0, st, (uint32_t)a.cols, nnz, S, Q, a.ci, a.va,
                       a.x, numbers, static_cast<const uint32_t *>(cut), part, static_cast<const LongSkip *>(skip), L.skip_words, active,
                       made);
    return LongStage{skip, numbers, active, rows, part, S};
}

} // namespace seer

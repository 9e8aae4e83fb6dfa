// CSR,S in bins -- the column-slabbed schedule for large matrices, with the slab of x in LDS.
// A gather out of L2 is one 128-byte request however little of the line is wanted, and the
// chip serves about 230 G of them a second, whatever the slab; LDS serves a wave's 64 gathers
// in a few cycles.  So x is cut into slabs that fit LDS (2^15 columns, 128 KB), and since most
// rows then have an entry or two per slab, products are not summed into rows where they are made:
//
//   * the nonzeros are cut into chunks of about 15 K (kBinNominal), on a row's start where one
//     lies within kBinMost - kBinNominal entries before the cut, else inside the row;
//   * preparation: the entries of (slab, chunk) form a bucket.  A run of entries of one row in it
//     (long rows have such runs) is taken sixteen and four at a time, so a bucket has three parts:
//     single entries, and fours and sixteens, of which only the sum will be kept.  Each part
//     is padded to groups of 16 entries; values and 16-bit columns within the slab lie slab
//     after slab, bucket after bucket;
//   * bins_multiply_kernel: a workgroup holds one slab of x in LDS, streams its entries and
//     writes products and sums to p, where they lie chunk after chunk, bucket after bucket (the
//     place of every group is kept beside the entries; a bucket begins on 64 bytes of p);
//   * bins_sum_kernel: a workgroup puts a chunk's part of p into row order in LDS (16-bit
//     places kept by the preparation) and sums the rows from there, as CSR,WO does.
//
// 16 bytes are moved per single entry (6 read + 4 written, 6 read), 7 to 9 where rows have runs,
// beside rows and padding, and that bounds both kernels where rows are even: 40 M nonzeros, 2 M columns, rows of 20: 427 MB in
// 84 us (5.1 TB/s, a third of it written) and 258 MB in 43 us (6.0 TB/s); the form with slabs in L2 takes
// 210 + 5 + 13 us, bound by its gathers.  Where they are not, the row sums are bound by the longest row of a wave: of a chunk of
// several hundred rows a lane adds up one of up to 128 products by itself, longer ones go to the whole wave one after
// the other (Zipf rows, s = 1.85, 47 M nonzeros: 110 MB in 39 us, 2.8 TB/s; the products 405 MB in 87, 4.6 TB/s).  Zipf rows (s = 1.9), 62 M nonzeros, 4 M columns: 129 + 58 + 5 us
// and 372 + 6 + 18.  Preparation, kernels alone, 40 M: 170 (sort) + 162 (fill) + 20 us, against about 480.
// Tried: without the sums of fours and sixteens, Zipf 133 + 109 us; the parts of all buckets of a slab
// one after the other, so that a bucket's p is written at three times, 134 instead of 129; streaming stores
// of p, 82 -> 95 us; four quads ahead, the same; p in 16 MB that stay in the last-level cache, 82 -> 77, not
// worth the launches and slabs that it takes to do so; stores left out for the measurement, 48.
#include "spmv_bodies.hiph"

namespace seer {

constexpr uint32_t kBinCols = 1u << kBinShift;      // columns per slab: 128 KB of x
constexpr uint32_t kBinNominal = 15360;             // nonzeros per chunk, where rows allow
constexpr uint32_t kBinMost = 16384;                // ... and at most: 64 KB of products, two workgroups per CU
constexpr uint32_t kBinGroup = 16;                  // entries per group
constexpr uint32_t kBinWG = 1024;
constexpr uint32_t kBinWaves = kBinWG / kWave;
constexpr uint32_t kBinGrid = 256;                  // workgroups of bins_multiply_kernel: one per CU (its LDS)
constexpr uint32_t kBinPartShift = 30;              // a group's place in p: words, and above them its part
constexpr uint32_t kBinNone = 0xFFFFu;              // place of a padding entry
constexpr uint32_t kBinAhead = kBinMost / kBinWG;   // entries per lane of the preparation
constexpr uint32_t kBinRounds = 4;                  // ... of which so many are fetched together
static_assert(kBinMost % kBinWG == 0 && kBinMost < kBinNone, "whole rounds, 16-bit places");

// The parts of a bucket, in the order in which they lie in it.
constexpr uint32_t kSingles = 0, kFours = 1, kSixteens = 2, kParts = 3;
__device__ __forceinline__ uint32_t bins_unit(uint32_t part) { return 1u << (2u * part); }

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Words of p (and entries of perm) per chunk: in every slab single entries are padded to 16, fours to 4,
// and the bucket's words to 16.
__host__ __device__ inline uint32_t bins_stride(uint32_t n_slabs) { return (kBinMost + 33u * n_slabs + 15u) & ~15u; }
// Entries of a chunk with all padding: 15 per slab for single entries, 12 for fours.
__host__ __device__ inline uint32_t bins_entry_stride(uint32_t n_slabs) { return (kBinMost + 27u * n_slabs + 15u) & ~15u; }

struct BinChunk {                                   // what the products need to know of a chunk
    uint32_t first_row, first_nnz;                  // the rows before first_row end at or before first_nnz
    uint32_t slots;                                 // sums and products of the chunk
    uint32_t cut;                                   // 1: first_row begins in an earlier chunk
};

// Exclusive prefix sum of v over the first waves of a workgroup of kBinWG lanes; the total
// comes back in *total.  s_w: LDS [kBinWaves].
__device__ __forceinline__ uint32_t bins_block_scan(uint32_t v, uint32_t *s_w, uint32_t *total)
{
    const uint32_t lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)incl, off);
        if ((int)lane >= off) incl += up;
    }
    if (lane == kWave - 1) s_w[wave] = incl;
    __syncthreads();
    uint32_t waves = s_w[lane % kBinWaves];                     // the sums of the waves, summed up by sixteen lanes
#pragma unroll
    for (int off = 1; off < (int)kBinWaves; off <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)waves, off, (int)kBinWaves);
        if ((int)(lane % kBinWaves) >= off) waves += up;
    }
    *total = (uint32_t)__builtin_amdgcn_readlane((int)waves, kBinWaves - 1);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)waves, __builtin_amdgcn_readfirstlane((int)wave - 1)) : 0u;
    return before + incl - v;
}

// Groups of a bucket's part before it in the chunk (*loc), and the words of p before it (*word), from
// the groups of the lane's own part (lane <-> slab * kParts + part; others: 0 groups).  A
// group is 16 words of single entries, 4 of fours, one of sixteens.  s_tmp: LDS [kBinWG].  Returns the chunk's
// groups in *total and its words.
__device__ __forceinline__ uint32_t bins_places(uint32_t groups, uint32_t *s_tmp, uint32_t *s_w, uint32_t *loc, uint32_t *word,
                                                uint32_t *total)
{
    const uint32_t tid = threadIdx.x, part = tid % kParts;
    uint32_t words = groups * (kBinGroup / bins_unit(part));
    s_tmp[tid] = words;
    *loc = bins_block_scan(groups, s_w, total);                 // (a barrier inside)
    if (part == kSixteens) words = ((s_tmp[tid - 2u] + s_tmp[tid - 1u] + words + kBinGroup - 1u) & ~(kBinGroup - 1u)) -
                                   s_tmp[tid - 2u] - s_tmp[tid - 1u];
    __syncthreads();                                            // (s_w is used again)
    uint32_t all;
    *word = bins_block_scan(words, s_w, &all);
    return all;
}

// ---- preparation 1: where the chunks begin, a wave for each.  kBinLooks of the waves also look at
// 256 consecutive entries and vote if these share lines of x, fewer than one line per two entries: in
// such a matrix (bands, stencils, blocks) gathers out of L1 and L2 cost next to nothing, and
// the other form is the faster one.  Long rows share lines, too, but have runs, which take less than half of a
// single entry's bytes here: where at most four descents are among the 256, fewer than 32 lines are asked for
// (Zipf rows, s = 1.6, 2 M columns, 471 M nonzeros, products and preparation: the other form 1586 and 3979 us, this
// 978 and 3789).
constexpr uint32_t kBinLines = 128, kBinLinesInRow = 32, kBinFewRows = 4;
constexpr uint32_t kBinLooks = 64;
// The wave of chunk k looks (its vote: number k / apart); so many of the votes exist.
__device__ __forceinline__ uint32_t bins_apart(uint32_t n_chunks) { return max(1u, n_chunks / kBinLooks); }
__device__ __forceinline__ bool bins_looks(uint32_t k, uint32_t n_chunks, uint32_t nnz)
{
    const uint32_t apart = bins_apart(n_chunks);
    return k % apart == 0 && k / apart < kBinLooks && k < n_chunks && k * kBinNominal + 256u <= nnz;
}

__global__ __launch_bounds__(kWG) void bins_table_kernel(
    int rows, uint32_t nnz, uint32_t n_chunks, const int *__restrict__ rp, const int *__restrict__ ci,
    BinChunk *__restrict__ table, uint32_t *__restrict__ counts_end, uint32_t *__restrict__ votes)
{
    __shared__ uint32_t s_seen[kWG / kWave][32];
    const uint32_t k = blockIdx.x * (kWG / kWave) + threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (k > n_chunks) return;                                   // wave-uniform
    const uint32_t t = k * kBinNominal;
    if (bins_looks(k, n_chunks, nnz)) {
        uint32_t *seen = s_seen[threadIdx.x / kWave];           // the wave's own: no barrier
        if (lane < 32u) seen[lane] = 0;
        __builtin_amdgcn_wave_barrier();
        uint32_t descents = 0;                                  // ends of rows, or nearly so
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t i = t + u * kWave + lane;
            const int c = ci[i];
            const uint32_t h = (((uint32_t)c >> 5) * 0x9E3779B1u) >> 22;                           // 1024 buckets of lines
            atomicOr(&seen[h >> 5], 1u << (h & 31u));
            descents += (uint32_t)__popcll(__ballot(c < ci[i ? i - 1u : 0u]));
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t lines = wave_fold(lane < 32u ? (uint32_t)__popc((int)seen[lane]) : 0u, [](uint32_t a, uint32_t b) { return a + b; });
        if (lane == 0) votes[k / bins_apart(n_chunks)] = lines < (descents <= kBinFewRows ? kBinLinesInRow : kBinLines) ? 1u : 0u;
    }
    if (k == 0 || k == n_chunks) {
        if (lane == 0) {
            table[k] = k ? BinChunk{(uint32_t)rows, nnz, 0u, 0u} : BinChunk{0u, 0u, 0u, 0u};
            if (k == 0) *counts_end = 0;
        }
        return;
    }
    const uint32_t lo = rows_ending_by(t, (uint32_t)rows, nnz, rp, lane);
    const uint32_t a = lo < (uint32_t)rows ? (uint32_t)rp[lo] : nnz;
    if (lane == 0) {
        const bool whole = t - a <= kBinMost - kBinNominal;
        table[k] = BinChunk{lo, whole ? a : t, 0u, whole ? 0u : 1u};
    }
}

// A chunk's rows are one workgroup's, empty ones among them, 0.43 ns each in a product and 0.6 to 1.2 in the
// preparation: a long run of empty rows holds up everything (12 M nonzeros, 4 M columns, 15 M empty rows in one place: 6497 us a
// product and 9600 to 18 100 of preparation, the other form 119 and 900).  most_rows is where that takes what
// the form gains: with so many in one chunk the other form is taken.
//
// What was seen, into pinned host memory: whether the other form is to be taken (max_len) and whether some row is cut
// (min_len).  The host waits for that before it enqueues the rest: a matrix that is not for this form then pays for these
// two launches and the wait, 15 us at 10 M nonzeros and 24 at 200 M (57 and 83 with the rest enqueued, too, to return
// at once, a prefix sum run for nothing and the flags copied to the host; where the form is taken 10 us less, as well).
__global__ __launch_bounds__(kBinWG) void bins_judge_kernel(
    uint32_t n_chunks, uint32_t nnz, const BinChunk *__restrict__ table, const uint32_t *__restrict__ votes, uint32_t most_rows,
    int always, uint32_t *__restrict__ bad, FeatureRaw *__restrict__ mailbox, uint64_t seq)
{
    const uint32_t tid = threadIdx.x;
    bool cut = false, empty = false;
    for (uint32_t k = tid; k < n_chunks; k += kBinWG) {
        cut |= table[k].cut != 0;
        empty |= table[k + 1u].first_row - table[k].first_row > most_rows;
    }
    const bool any_cut = __syncthreads_or(cut ? 1 : 0) != 0, any_empty = __syncthreads_or(empty ? 1 : 0) != 0;
    if (tid >= kBinLooks) return;
    static_assert(kBinLooks == kWave, "a vote per lane of one wave");
    const bool looked = tid < n_chunks && bins_looks(tid * bins_apart(n_chunks), n_chunks, nnz);
    const uint32_t looks = (uint32_t)__popcll(__ballot(looked)), local = (uint32_t)__popcll(__ballot(looked && votes[tid] != 0));
    if (tid != 0) return;
    *bad = 0;                                                   // (for the next kernels)
    mailbox->max_len = (2u * local > looks || any_empty) && !always ? 1 : 0;
    mailbox->min_len = any_cut ? 1 : 0;
    __threadfence_system();
    *reinterpret_cast<volatile uint64_t *>(&mailbox->seq) = seq;
}

// ---- preparation 2: a chunk's entries sorted by slab and part.  Leaves the groups per bucket and part
// (counts [n_slabs][n_chunks][kParts], for the prefix sum) and the chunk's words of p; order: for every entry
// in that order its number in the chunk; perm: for every word of the chunk's p its place in row order
// ("slot"); row_slot: the first slot of every row.  *bad: some row's columns do not ascend or lie outside
// the matrix.  A wave takes 1024 consecutive entries, 64 at a time (a run does not go on from one 64 to the
// next), and counts them by itself, so that all places depend on the matrix alone.
struct BinEntry {                                               // one entry among the 64 that its wave looks at
    uint32_t slab, part, sub;                                   // sub: its number within its sixteen or four
    bool bad;
    bool runs;                                                  // some run among the 64 has four entries (wave-uniform)
};
// All lanes of a wave together; `prev`: the column before lane 0's, handed on to the next 64.
__device__ __forceinline__ BinEntry bins_entry(
    uint32_t c, uint32_t &prev, bool in, bool starts_row, uint32_t lane, uint32_t cols, uint32_t n_slabs)
{
    const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp((int)prev, (int)c, 0x138, 0xF, 0xF, false);
    prev = (uint32_t)__builtin_amdgcn_readlane((int)c, kWave - 1);
    BinEntry r;
    r.bad = in && (c >= cols || ((int)c < (int)before && !starts_row));
    r.slab = min(c >> kBinShift, n_slabs - 1u);
    // the run of one row and one slab that the lane is in: n entries from lane - o on
    const bool opens = !in || starts_row || lane == 0 || r.slab != min(before >> kBinShift, n_slabs - 1u);
    const uint64_t open = __ballot(opens);
    r.part = kSingles;
    r.sub = 0;
    r.runs = (~open & ~open >> 1 & ~open >> 2) != 0;
    if (!r.runs) return r;                                      // (nearly always where rows are short: half of the work)
    const uint64_t upto = open & (~0ull >> (63u - lane)), after = lane == 63u ? 0ull : open >> (lane + 1u);
    const uint32_t o = lane - (63u - (uint32_t)__clzll((long long)upto));
    const uint32_t n = o + (after ? (uint32_t)__ffsll((long long)after) : 64u - lane);
    r.part = o < (n & ~15u) ? kSixteens : o < (n & ~3u) ? kFours : kSingles;
    r.sub = o & (bins_unit(r.part) - 1u);
    return r;
}

__global__ __launch_bounds__(kBinWG, 8) void bins_sort_kernel(
    int rows, int cols, uint32_t n_slabs, uint32_t n_chunks, const int *__restrict__ rp, const int *__restrict__ ci,
    BinChunk *__restrict__ table, uint32_t *__restrict__ counts, uint32_t *__restrict__ chunk_words,
    uint16_t *__restrict__ perm, uint16_t *__restrict__ order, uint16_t *__restrict__ row_slot, uint32_t *__restrict__ any_bad)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    const uint32_t entry_stride = bins_entry_stride(n_slabs), nb = kParts * n_slabs;
    uint32_t *s_order = lds;                                    // [entry_stride / 2]: pairs of 16-bit numbers
    uint64_t *s_lead = reinterpret_cast<uint64_t *>(s_order + entry_stride / 2u);   // [kBinMost / 64]: which entries open a slot
    uint32_t *s_before = reinterpret_cast<uint32_t *>(s_lead + kBinMost / 64u);     // [kBinMost / 64]: slots before these 64
    uint32_t *s_starts = s_before + kBinMost / 64u;             // [kBinMost / 32]: bit k: entry k starts a row
    uint32_t *s_w = s_starts + kBinMost / 32u;                  // [kBinWaves]
    uint32_t *s_tmp = s_w + kBinWaves;                          // [kBinWG]
    uint32_t *s_loc = s_tmp + kBinWG;                           // [nb]: entries of the chunk before each bucket's part
    uint32_t *s_word = s_loc + nb;                              // [nb]: its words of p before it
    uint32_t *s_hist = s_word + nb;                             // [kBinWaves][nb]: units of each wave, then its next place
    uint16_t *s_of = reinterpret_cast<uint16_t *>(s_hist + kBinWaves * nb);         // [entry_stride / kBinGroup]: whose group
    const uint32_t tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const uint32_t chunk = tile_of_block(blockIdx.x, n_chunks, 1);
    if (chunk >= n_chunks) return;
    const BinChunk t0 = table[chunk], t1 = table[chunk + 1];
    const uint32_t b = t0.first_nnz, len = t1.first_nnz - b;

    const uint32_t first = wave * (kBinAhead * kWave);          // this wave's entries
    // Calls look(i, in, entry) for the wave's entries, 64 at a time: once to count, once to place.  The columns
    // come four rounds at a time, the second time out of L2: kept in registers, all sixteen rounds and
    // what the compiler finds to share between the two looks take more than 64 of them.
    const auto look_at_all = [&](auto look) {
        uint32_t prev = 0;                                      // column of the entry before the wave's first
        if (first < len && b + first > 0u) prev = (uint32_t)ci[b + first - 1u];
        uint32_t ahead[kBinRounds];
        const auto fetch = [&](uint32_t m0) {
#pragma unroll
            for (uint32_t u = 0; u < kBinRounds; ++u) {
                const uint32_t i = first + (m0 + u) * kWave + lane;
                ahead[u] = i < len ? (uint32_t)ci[b + i] : 0u;
            }
        };
        fetch(0);
#pragma unroll 1
        for (uint32_t m0 = 0; m0 < kBinAhead; m0 += kBinRounds) {
            uint32_t c[kBinRounds];
#pragma unroll
            for (uint32_t u = 0; u < kBinRounds; ++u) c[u] = ahead[u];
            if (m0 + kBinRounds < kBinAhead) fetch(m0 + kBinRounds);
#pragma unroll
            for (uint32_t u = 0; u < kBinRounds; ++u) {
                const uint32_t i = first + (m0 + u) * kWave + lane;
                const bool in = i < len, starts = in && ((s_starts[i >> 5] >> (i & 31u)) & 1u);
                look(i, in, bins_entry(c[u], prev, in, starts, lane, (uint32_t)cols, n_slabs));
            }
        }
    };
#pragma unroll 1
    for (uint32_t i = tid; i < kBinWaves * nb; i += kBinWG) s_hist[i] = 0;
#pragma unroll 1
    for (uint32_t i = tid; i < kBinMost / 32u; i += kBinWG) s_starts[i] = 0;
#pragma unroll 1
    for (uint32_t i = tid; i < entry_stride / 2u; i += kBinWG) s_order[i] = 0xFFFFFFFFu;
    __syncthreads();
    const uint32_t row_end = t1.first_row + t1.cut;             // rows that begin here, beside the cut first one
#pragma unroll 1
    for (uint32_t r = t0.first_row + t0.cut + tid; r < row_end; r += kBinWG) {
        const uint32_t at = (uint32_t)rp[r] - b;
        if (at < len) atomicOr(&s_starts[at >> 5], 1u << (at & 31u));
    }
    __syncthreads();
    bool bad = false;
    look_at_all([&](uint32_t i, bool in, const BinEntry &e) {
        bad |= e.bad;
        const bool opens = in && e.sub == 0;
        if (opens) atomicAdd(&s_hist[wave * nb + e.slab * kParts + e.part], 1u);
        const uint64_t lead = __ballot(opens);
        if (lane == 0) s_lead[i / kWave] = lead;
    });
    __syncthreads();
    // units to groups, a lane per slab and part; slots before each 64 entries
    const uint32_t my_unit = bins_unit(tid % kParts);
    uint32_t groups = 0;
    if (tid < nb) {
        uint32_t n = 0;
#pragma unroll 4
        for (uint32_t w = 0; w < kBinWaves; ++w) n += s_hist[w * nb + tid];
        groups = (n * my_unit + kBinGroup - 1u) / kBinGroup;
        counts[((size_t)(tid / kParts) * n_chunks + chunk) * kParts + tid % kParts] = groups;
    }
    uint32_t loc, word, total, slots;
    const uint32_t words = bins_places(groups, s_tmp, s_w, &loc, &word, &total);
    uint16_t *my_perm = perm + (size_t)chunk * bins_stride(n_slabs);
    if (tid < nb) {
        s_loc[tid] = loc * kBinGroup;
        s_word[tid] = word;
        uint32_t n = loc * kBinGroup;                           // a wave's next place in the order
#pragma unroll 4
        for (uint32_t w = 0; w < kBinWaves; ++w) {
            const uint32_t mine = s_hist[w * nb + tid];
            s_hist[w * nb + tid] = n;
            n += mine * my_unit;
        }
#pragma unroll 1
        for (uint32_t g = 0; g < groups; ++g) s_of[loc + g] = (uint16_t)tid;
        if (tid % kParts == kSixteens)                          // the words that only fill up the bucket's last 16
#pragma unroll 1
            for (uint32_t w = word + groups; w & (kBinGroup - 1u); ++w) my_perm[w] = (uint16_t)kBinNone;
    }
    __syncthreads();                                            // (s_w is used again)
    {
        const uint32_t mine = tid < kBinMost / kWave ? (uint32_t)__popcll(s_lead[tid]) : 0u;
        const uint32_t before = bins_block_scan(mine, s_w, &slots);
        if (tid < kBinMost / kWave) s_before[tid] = before;
    }
    uint16_t *s_out = reinterpret_cast<uint16_t *>(s_order);
    look_at_all([&](uint32_t i, bool in, const BinEntry &e) {
        uint32_t at = 0;
        if (in && e.sub == 0)
            at = atomicAdd(&s_hist[wave * nb + e.slab * kParts + e.part], bins_unit(e.part));
        if (e.runs) at = (uint32_t)__shfl((int)at, (int)(lane - e.sub)) + e.sub;
        if (in) s_out[at] = (uint16_t)i;
    });
    __syncthreads();
    const auto slot_of = [&](uint32_t i) {
        return s_before[i / kWave] + (uint32_t)__popcll(s_lead[i / kWave] & ((1ull << (i % kWave)) - 1ull));
    };
#pragma unroll 1
    for (uint32_t r = t0.first_row + t0.cut + tid; r < row_end; r += kBinWG) {
        const uint32_t at = (uint32_t)rp[r] - b;                // (a last, empty row may begin where the chunk ends)
        row_slot[r] = (uint16_t)(at < len ? slot_of(at) : slots);
    }
    {
        v4u *out = reinterpret_cast<v4u *>(order + (size_t)chunk * entry_stride);
#pragma unroll 1
        for (uint32_t i = tid; i < total * (kBinGroup / 8u); i += kBinWG) out[i] = reinterpret_cast<const v4u *>(s_order)[i];
    }
    // perm, four entries of the order at a time: as many words of single entries, one word of fours, and of a
    // sixteen one for its first four
    const auto slot_or_none = [&](uint32_t i) { return i == kBinNone ? kBinNone : slot_of(i); };
#pragma unroll 1
    for (uint32_t k = 4u * tid; k < total * kBinGroup; k += 4u * kBinWG) {
        const uint32_t bucket = s_of[k / kBinGroup], part = bucket % kParts, rel = k - s_loc[bucket];
        const v2u four = *reinterpret_cast<const v2u *>(s_out + k);
        uint16_t *to = my_perm + s_word[bucket] + rel / bins_unit(part);
        const uint32_t first = slot_or_none(four.x & 0xFFFFu);
        if (part == kSingles)
            *reinterpret_cast<v2u *>(to) = v2u{first | slot_or_none(four.x >> 16) << 16,
                                               slot_or_none(four.y & 0xFFFFu) | slot_or_none(four.y >> 16) << 16};
        else if (part == kFours || (rel & 15u) == 0)
            *to = (uint16_t)first;
    }
    if (tid == 0) {
        chunk_words[chunk] = words;
        table[chunk].slots = slots;
    }
    if (bad) *any_bad = 1;
}

// ---- preparation 3, with the buckets' first groups known (starts): values and 16-bit columns into
// their buckets, each group's place in p beside them.  The chunk's values, then its columns, lie in LDS
// in CSR order, so that they are read and written in whole lines.
__global__ __launch_bounds__(kBinWG, 8) void bins_fill_kernel(
    uint32_t n_slabs, uint32_t n_chunks, const int *__restrict__ ci, const float *__restrict__ va,
    const BinChunk *__restrict__ table, const uint32_t *__restrict__ starts,
    const uint16_t *__restrict__ order, const uint32_t *__restrict__ bad, float *__restrict__ out_va, uint16_t *__restrict__ out_ci, uint32_t *__restrict__ out_to)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    float *s_val = reinterpret_cast<float *>(lds);              // [kBinMost]
    uint32_t *s_w = lds + kBinMost;                             // [kBinWaves]
    uint32_t *s_to = s_w + kBinWaves;                           // [entry stride / kBinGroup]: the chunk's groups among all
    uint32_t *s_place = s_to + bins_entry_stride(n_slabs) / kBinGroup;              // the same: their places in p
    const uint32_t stride = bins_stride(n_slabs), entry_stride = bins_entry_stride(n_slabs);
    const uint32_t tid = threadIdx.x;
    const uint32_t chunk = tile_of_block(blockIdx.x, n_chunks, 1);
    if (chunk >= n_chunks || *bad) return;                      // (bad: the form is refused, and that 160 us sooner at 40 M)
    const uint32_t b = table[chunk].first_nnz, len = table[chunk + 1].first_nnz - b;
    float v[kBinAhead];
    uint32_t c[kBinAhead];
#pragma unroll
    for (uint32_t m = 0; m < kBinAhead; ++m) {
        const uint32_t i = m * kBinWG + tid;
        v[m] = i < len ? __builtin_nontemporal_load(va + b + i) : 0.f;
    }
#pragma unroll
    for (uint32_t m = 0; m < kBinAhead; ++m) {
        const uint32_t i = m * kBinWG + tid;
        c[m] = i < len ? (uint32_t)__builtin_nontemporal_load(ci + b + i) : 0u;
    }
    uint32_t at = 0, groups = 0;
    if (tid < kParts * n_slabs) {
        const uint32_t *from = starts + ((size_t)(tid / kParts) * n_chunks + chunk) * kParts + tid % kParts;
        at = from[0];
        groups = from[1] - at;
    }
    uint32_t loc, word, total;
    bins_places(groups, lds, s_w, &loc, &word, &total);
    {
        const uint32_t part = tid % kParts, each = kBinGroup / bins_unit(part);
#pragma unroll 1
        for (uint32_t g = 0; g < groups; ++g) {
            s_to[loc + g] = at + g;
            s_place[loc + g] = (chunk * stride + word + g * each) | part << kBinPartShift;
        }
    }
    __syncthreads();                                            // (lds held the groups' words)
#pragma unroll
    for (uint32_t m = 0; m < kBinAhead; ++m) s_val[m * kBinWG + tid] = v[m];
    __syncthreads();
    const v2u *places = reinterpret_cast<const v2u *>(order + (size_t)chunk * entry_stride);
    const uint32_t quads = total * (kBinGroup / 4u);
#pragma unroll 1
    for (uint32_t q = tid; q < quads; q += kBinWG) {
        const v2u pl = places[q];
        const uint32_t i0 = pl.x & 0xFFFFu, i1 = pl.x >> 16, i2 = pl.y & 0xFFFFu, i3 = pl.y >> 16;
        const uint32_t to = s_to[q / 4u];
        v4f o;
        o.x = i0 != kBinNone ? s_val[i0 & (kBinMost - 1u)] : 0.f;
        o.y = i1 != kBinNone ? s_val[i1 & (kBinMost - 1u)] : 0.f;
        o.z = i2 != kBinNone ? s_val[i2 & (kBinMost - 1u)] : 0.f;
        o.w = i3 != kBinNone ? s_val[i3 & (kBinMost - 1u)] : 0.f;
        *reinterpret_cast<v4f *>(out_va + (size_t)to * kBinGroup + 4u * (q % 4u)) = o;
        if (q % 4u == 0) out_to[to] = s_place[q / 4u];
    }
    __syncthreads();
    uint32_t *s_col = lds;
#pragma unroll
    for (uint32_t m = 0; m < kBinAhead; ++m) s_col[m * kBinWG + tid] = c[m] & (kBinCols - 1u);
    __syncthreads();
#pragma unroll 1
    for (uint32_t q = tid; q < quads; q += kBinWG) {
        const v2u pl = places[q];
        const uint32_t i0 = pl.x & 0xFFFFu, i1 = pl.x >> 16, i2 = pl.y & 0xFFFFu, i3 = pl.y >> 16;
        const uint32_t to = s_to[q / 4u];
        v2u o;
        o.x = (i0 != kBinNone ? s_col[i0 & (kBinMost - 1u)] : 0u) | (i1 != kBinNone ? s_col[i1 & (kBinMost - 1u)] : 0u) << 16;
        o.y = (i2 != kBinNone ? s_col[i2 & (kBinMost - 1u)] : 0u) | (i3 != kBinNone ? s_col[i3 & (kBinMost - 1u)] : 0u) << 16;
        *reinterpret_cast<v2u *>(out_ci + (size_t)to * kBinGroup + 4u * (q % 4u)) = o;
    }
}

// Whether the form is refused, into pinned host memory (max_len).
__global__ void bins_report_kernel(const uint32_t *__restrict__ bad, FeatureRaw *__restrict__ mailbox, uint64_t seq)
{
    mailbox->max_len = (int32_t)*bad;
    __threadfence_system();
    *reinterpret_cast<volatile uint64_t *>(&mailbox->seq) = seq;
}

// ---- the products.  A workgroup takes an equal share of the groups, slab after slab; a group's four
// quads go to four lanes.  One workgroup of 1024 lanes per CU is all the slab leaves room for, so every
// lane has kMulAhead quads of the next trip under way while it gathers for this one.
constexpr uint32_t kMulAhead = 2;
struct BinQuads {
    v4f v[kMulAhead];
    v2u c[kMulAhead];
    uint32_t to[kMulAhead];
};
__device__ __forceinline__ void bins_load(BinQuads &r, uint32_t q0, uint32_t end, const float *__restrict__ va,
                                          const uint16_t *__restrict__ ci, const uint32_t *__restrict__ to)
{
#pragma unroll
    for (uint32_t u = 0; u < kMulAhead; ++u) {
        const uint32_t q = min(q0 + u * kBinWG, end - 1u);
        r.v[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(va) + q);
        r.c[u] = __builtin_nontemporal_load(reinterpret_cast<const v2u *>(ci) + q);
        r.to[u] = __builtin_nontemporal_load(to + q / 4u);
    }
}

__global__ __launch_bounds__(kBinWG) void bins_multiply_kernel(
    int cols, uint32_t n_slabs, uint32_t n_chunks, const float *__restrict__ x, const uint32_t *__restrict__ starts,
    const float *__restrict__ va, const uint16_t *__restrict__ ci, const uint32_t *__restrict__ to, float *__restrict__ p)
{
    __shared__ __attribute__((aligned(16))) float s_x[kBinCols];
    __shared__ uint32_t s_start[kBinMaxSlabs + 1];
    const uint32_t tid = threadIdx.x;
    if (tid <= n_slabs) s_start[tid] = starts[(size_t)tid * n_chunks * kParts];
    __syncthreads();
    const uint32_t total = s_start[n_slabs], share = tile_of_block(blockIdx.x, kBinGrid, 1);
    uint32_t g = (uint32_t)((uint64_t)total * share / kBinGrid);
    const uint32_t g_end = (uint32_t)((uint64_t)total * (share + 1u) / kBinGrid);
    for (uint32_t s = 0; s < n_slabs && g < g_end; ++s) {       // block-uniform
        const uint32_t next = s_start[s + 1u];
        if (next <= g) continue;
        const uint32_t end = min(next, g_end) * (kBinGroup / 4u);
        uint32_t q = g * (kBinGroup / 4u) + tid;
        BinQuads now;
        bins_load(now, q, end, va, ci, to);
        __syncthreads();                                        // the slab before has been used
        const uint32_t c0 = s << kBinShift, n = min((uint32_t)cols - c0, kBinCols);
        {
            v4f t[kBinCols / 4u / kBinWG];
#pragma unroll
            for (uint32_t m = 0; m < kBinCols / 4u / kBinWG; ++m) {
                const uint32_t k = 4u * (m * kBinWG + tid);
                if (k + 4u <= n) {
                    t[m] = *reinterpret_cast<const v4f_a4 *>(x + c0 + k);
                } else {
                    t[m].x = k < n ? x[c0 + k] : 0.f;
                    t[m].y = k + 1u < n ? x[c0 + k + 1u] : 0.f;
                    t[m].z = k + 2u < n ? x[c0 + k + 2u] : 0.f;
                    t[m].w = 0.f;
                }
            }
#pragma unroll
            for (uint32_t m = 0; m < kBinCols / 4u / kBinWG; ++m)
                *reinterpret_cast<v4f *>(s_x + 4u * (m * kBinWG + tid)) = t[m];
        }
        __syncthreads();
        for (;;) {
            const uint32_t q_next = q + kMulAhead * kBinWG;
            const bool more = q_next - tid < end;               // block-uniform
            BinQuads ahead;
            if (more) bins_load(ahead, q_next, end, va, ci, to);
#pragma unroll
            for (uint32_t u = 0; u < kMulAhead; ++u) {
                v4f o;
                o.x = now.v[u].x * s_x[now.c[u].x & 0xFFFFu];
                o.y = now.v[u].y * s_x[now.c[u].x >> 16];
                o.z = now.v[u].z * s_x[now.c[u].y & 0xFFFFu];
                o.w = now.v[u].w * s_x[now.c[u].y >> 16];
                const uint32_t qu = q + u * kBinWG;
                float *dst = p + (now.to[u] & ((1u << kBinPartShift) - 1u));
                const uint32_t part = now.to[u] >> kBinPartShift;
                if (part == kSingles) {
                    if (qu < end) *reinterpret_cast<v4f *>(dst + 4u * (qu % 4u)) = o;
                } else {                                        // (the four lanes of a group stay together)
                    const float four = (o.x + o.y) + (o.z + o.w);
                    if (part == kFours) {
                        if (qu < end) dst[qu % 4u] = four;
                    } else {
                        const float sixteen = group_sum<4>(four);
                        if (qu < end && qu % 4u == 0) *dst = sixteen;
                    }
                }
            }
            if (!more) break;
            now = ahead;
            q = q_next;
        }
        g = min(next, g_end);
    }
}

// ---- the sums.  A workgroup per chunk; rows that the chunk boundary cuts leave a carry, as in CSR,WO.
// Sum of s[a .. b), b > a, by one lane: eight partial sums (with four, as the other schedules have, rows of
// 20 are 4 % further from the exact sums than in the other form, which adds them up slab by slab).
__device__ __forceinline__ float bins_slice_sum(const float *__restrict__ s, uint32_t a, uint32_t b)
{
    float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint32_t k = a;
    for (; k + 8u <= b; k += 8u) {
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) t[j] += s[k + j];
    }
    float u[7];
#pragma unroll
    for (uint32_t j = 0; j < 7; ++j) u[j] = s[min(k + j, b - 1u)];      // what is left, fetched together
#pragma unroll
    for (uint32_t j = 0; j < 7; ++j) t[j] += k + j < b ? u[j] : 0.f;
    return ((t[0] + t[4]) + (t[2] + t[6])) + ((t[1] + t[5]) + (t[3] + t[7]));
}

// One batch of up to kBinWG >> gshift rows: the 2^gshift lanes that share i take row i (if `in`), whose slots are
// [a, b).  A row of more than `most` slots per lane is taken by the whole wave: most is four times the mean, so
// that of skewed rows no lane walks a long one while 63 wait, and even ones stay with their lanes.
__device__ __forceinline__ void bins_rows(
    bool in, uint32_t i, uint32_t a, uint32_t b, uint32_t hi, uint32_t lane, uint32_t gshift, uint32_t most,
    const float *__restrict__ s_prod, float *__restrict__ y, float *__restrict__ carry_val, uint32_t chunk)
{
    const uint32_t L = 1u << gshift, sub = lane & (L - 1u);
    const bool has = in && b > a, is_long = has && b - a > most << gshift;
    float sum = 0.f;
    if (gshift == 0) {                                          // block-uniform
        if (has && !is_long) sum = bins_slice_sum(s_prod, a, b);
    } else {
        if (has && !is_long) {
            float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
            uint32_t k = a + sub;
            for (; k + 3u * L < b; k += 4u * L) {
                t0 += s_prod[k];
                t1 += s_prod[k + L];
                t2 += s_prod[k + 2u * L];
                t3 += s_prod[k + 3u * L];
            }
            for (; k < b; k += L) t0 += s_prod[k];
            sum = (t0 + t1) + (t2 + t3);
        }
        sum = group_sum_by_shift(sum, gshift);                  // every lane of the wave is here
    }
    uint64_t todo = __ballot(is_long && sub == 0);
    while (todo) {                                              // wave-uniform
        const int src = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        const uint32_t la = (uint32_t)__shfl((int)a, src), lb = (uint32_t)__shfl((int)b, src);
        float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
        uint32_t k = la + lane;
        for (; k + 3u * kWave < lb; k += 4u * kWave) {
            t0 += s_prod[k];
            t1 += s_prod[k + kWave];
            t2 += s_prod[k + 2u * kWave];
            t3 += s_prod[k + 3u * kWave];
        }
        for (; k < lb; k += kWave) t0 += s_prod[k];
        const float t = group_sum<64>((t0 + t1) + (t2 + t3));
        if ((int)lane == src) sum = t;
    }
    if (in && sub == 0) {
        if (i < hi) y[i] = sum;
        else carry_val[chunk] = sum;                            // the row cut by the end of the chunk
    }
}

__global__ __launch_bounds__(kBinWG) void bins_sum_kernel(
    int rows, uint32_t n_chunks, uint32_t stride, const BinChunk *__restrict__ table,
    const uint32_t *__restrict__ chunk_words, const uint16_t *__restrict__ row_slot, const uint16_t *__restrict__ perm,
    const float *__restrict__ p, float *__restrict__ y, int *__restrict__ carry_row, float *__restrict__ carry_val)
{
    __shared__ __attribute__((aligned(16))) float s_prod[kBinMost];
    const uint32_t tid = threadIdx.x, lane = tid % kWave;
    const uint32_t chunk = tile_of_block(blockIdx.x, n_chunks, 1);
    if (chunk >= n_chunks) return;
    const BinChunk t0 = table[chunk], t1 = table[chunk + 1u];
    const uint32_t lo = t0.first_row, hi = t1.first_row, slots = t0.slots;
    const uint32_t quads = chunk_words[chunk] / 4u;
    const v2u *places = reinterpret_cast<const v2u *>(perm + (size_t)chunk * stride);
    const v4f *products = reinterpret_cast<const v4f *>(p + (size_t)chunk * stride);
    const uint32_t n_rows = hi - lo + t1.cut;                   // the rows that end here and the one cut by the chunk's end
    uint32_t gshift = 0;                                        // log2 of the lanes per row, if all rows fit one batch
    if (n_rows <= kBinWG / 2u) gshift = min(6u, 31u - (uint32_t)__clz((int)(kBinWG / max(n_rows, 1u))));
    const uint32_t most = min(max(4u * slots / max(n_rows, 1u), 32u), 128u);
    const auto slot_of = [&](uint32_t r) -> uint32_t {          // first slot of row lo + r; of the row after the last: the end
        return r == 0 ? 0u : r < n_rows ? (uint32_t)row_slot[lo + r] : slots;
    };
    constexpr uint32_t NB = 4;                                  // batches of rows whose slots are fetched ahead: of rows of two or three
    uint32_t ra[NB], rb[NB];                                    // entries a chunk has several
#pragma unroll
    for (uint32_t k = 0; k < NB; ++k) {
        if (k * kBinWG >= n_rows) break;                        // block-uniform
        const uint32_t r = (tid >> gshift) + k * kBinWG;
        ra[k] = r < n_rows ? slot_of(r) : 0u;
        rb[k] = r < n_rows ? slot_of(r + 1u) : 0u;
    }
    constexpr uint32_t U = 4;
    for (uint32_t q0 = tid; q0 < quads; q0 += U * kBinWG) {
        v2u pl[U];
        v4f pr[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t q = min(q0 + u * kBinWG, quads - 1u);
            pl[u] = __builtin_nontemporal_load(places + q);
            pr[u] = products[q];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (q0 + u * kBinWG >= quads) break;
            const uint32_t i0 = pl[u].x & 0xFFFFu, i1 = pl[u].x >> 16, i2 = pl[u].y & 0xFFFFu, i3 = pl[u].y >> 16;
            if (i0 < kBinMost) s_prod[i0] = pr[u].x;
            if (i1 < kBinMost) s_prod[i1] = pr[u].y;
            if (i2 < kBinMost) s_prod[i2] = pr[u].z;
            if (i3 < kBinMost) s_prod[i3] = pr[u].w;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < NB; ++k) {
        if (k * kBinWG >= n_rows) break;                        // block-uniform
        const uint32_t r = (tid >> gshift) + k * kBinWG;
        bins_rows(r < n_rows, lo + r, ra[k], rb[k], hi, lane, gshift, most, s_prod, y, carry_val, chunk);
    }
    for (uint32_t base = NB * kBinWG; base < n_rows; base += kBinWG) {    // mostly empty rows
        const uint32_t r = base + tid;
        const bool in = r < n_rows;
        const uint32_t a = in ? slot_of(r) : 0u, e = in ? slot_of(r + 1u) : 0u;
        bins_rows(in, lo + r, a, e, hi, lane, 0u, most, s_prod, y, carry_val, chunk);
    }
    if (tid == 0) carry_row[chunk] = t1.cut ? (int)hi : rows;
}

// ------------------------------------------------------------------ host side
static size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }

uint32_t bins_num_slabs(int cols) { return cols > 0 ? ((uint32_t)cols + kBinCols - 1u) >> kBinShift : 0u; }
static uint32_t bins_num_chunks(int nnz) { return nnz > 0 ? ((uint32_t)nnz + kBinNominal - 1u) / kBinNominal : 1u; }

// The slabs' counters fit the preparation's LDS, and a place in p fits beside its part.
bool bins_fit(int cols, int nnz)
{
    const uint32_t S = bins_num_slabs(cols);
    return S <= kBinMaxSlabs && (uint64_t)bins_num_chunks(nnz) * bins_stride(S) <= 1ull << kBinPartShift;
}

// Where things lie in plan_mem, from the sizes alone: the entries' values, 16-bit columns and
// groups' places, perm, the rows' first slots, the buckets' first groups (counts before that), words of p
// per chunk, the chunk table; then what only the preparation uses: order (the votes before that), the prefix
// sum's scratch, a flag.
struct BinsLayout {
    uint32_t n_chunks, stride;
    size_t n_buckets, max_groups;
    size_t va, ci, to, perm, row_slot, starts, chunk_words, table, order, scan, flag, total;
};
// Twice the chunks' mean, and so many beyond that as a product gains in time by this form: runs of 128 Ki empty rows
// among 12 M nonzeros 108 us, the other form 94 (without a run 54 and 93), 256 Ki among 40 M 246 and 279, 512 Ki 357
// and 278, 256 Ki among 60 M 349 and 432, 512 Ki 500 and 433.  Where rows are many but spread evenly all chunks take as
// long: 100 M rows, 12 M nonzeros, 128 K rows a chunk, 337 and 339.
static uint32_t bins_most_rows(int rows, int nnz) { return 2u * ((uint32_t)rows / bins_num_chunks(nnz)) + (uint32_t)nnz / 160u; }

static BinsLayout bins_layout(uint32_t n_slabs, int rows, int nnz)
{
    BinsLayout L;
    L.n_chunks = bins_num_chunks(nnz);
    L.stride = bins_stride(n_slabs);
    L.n_buckets = (size_t)n_slabs * kParts * L.n_chunks;
    const size_t padded = L.n_buckets / kParts < (size_t)nnz ? L.n_buckets / kParts : (size_t)nnz;
    L.max_groups = ((size_t)nnz + 27u * padded) / kBinGroup + 1u;   // (padding as in bins_entry_stride)
    size_t o = 0;
    L.va = o;           o += pad256(L.max_groups * kBinGroup * 4);
    L.ci = o;           o += pad256(L.max_groups * kBinGroup * 2);
    L.to = o;           o += pad256(L.max_groups * 4);
    L.perm = o;         o += pad256((size_t)L.n_chunks * L.stride * 2);
    L.row_slot = o;     o += pad256((size_t)rows * 2);
    L.starts = o;       o += pad256((L.n_buckets + 1) * 4);
    L.chunk_words = o;  o += pad256((size_t)L.n_chunks * 4);
    L.table = o;        o += pad256(((size_t)L.n_chunks + 1) * sizeof(BinChunk));
    L.order = o;        o += pad256((size_t)L.n_chunks * bins_entry_stride(n_slabs) * 2);
    L.scan = o;         o += pad256(scan_scratch_words(L.n_buckets + 1) * 4 + 4);
    L.flag = o;         o += 256;
    L.total = o;
    return L;
}

size_t bins_plan_bytes(int rows, int cols, int nnz) { return bins_layout(bins_num_slabs(cols), rows, nnz).total; }

size_t bins_workspace_bytes(uint32_t n_slabs, int nnz)
{
    const uint32_t n = bins_num_chunks(nnz);
    return pad256((size_t)n * bins_stride(n_slabs) * 4) + carry_workspace_bytes(n);
}

void launch_bins_judge(int rows, int cols, int nnz, const int *rp, const int *ci, void *plan_mem, bool always,
                       FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st)
{
    const BinsLayout L = bins_layout(bins_num_slabs(cols), rows, nnz);
    char *base = static_cast<char *>(plan_mem);
    uint32_t *starts = reinterpret_cast<uint32_t *>(base + L.starts), *votes = reinterpret_cast<uint32_t *>(base + L.order);
    BinChunk *table = reinterpret_cast<BinChunk *>(base + L.table);
    hipLaunchKernelGGL(bins_table_kernel, dim3(L.n_chunks / (kWG / kWave) + 1u), dim3(kWG), 0, st, rows, (uint32_t)nnz,
                       L.n_chunks, rp, ci, table, starts + L.n_buckets, votes);
    hipLaunchKernelGGL(bins_judge_kernel, dim3(1), dim3(kBinWG), 0, st, L.n_chunks, (uint32_t)nnz,
                       static_cast<const BinChunk *>(table), static_cast<const uint32_t *>(votes), bins_most_rows(rows, nnz),
                       always ? 1 : 0,
                       reinterpret_cast<uint32_t *>(base + L.flag), mailbox_dev, seq);
}

void launch_bins_prepare(int rows, int cols, int nnz, const int *rp, const int *ci, const float *va, void *plan_mem,
                         FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st)
{
    const uint32_t S = bins_num_slabs(cols);
    const BinsLayout L = bins_layout(S, rows, nnz);
    char *base = static_cast<char *>(plan_mem);
    uint32_t *starts = reinterpret_cast<uint32_t *>(base + L.starts);
    uint32_t *chunk_words = reinterpret_cast<uint32_t *>(base + L.chunk_words);
    BinChunk *table = reinterpret_cast<BinChunk *>(base + L.table);
    uint16_t *order = reinterpret_cast<uint16_t *>(base + L.order);
    uint16_t *perm = reinterpret_cast<uint16_t *>(base + L.perm);
    uint32_t *bad = reinterpret_cast<uint32_t *>(base + L.flag);
    const dim3 grid(tiles_per_xcd(L.n_chunks) * kXCD);
    const size_t sort_lds = (size_t)bins_entry_stride(S) * 2 + kBinMost / 64u * 12u + kBinMost / 32u * 4u +
                            (kBinWaves + kBinWG + (size_t)(2u + kBinWaves) * kParts * S) * 4 +
                            bins_entry_stride(S) / kBinGroup * 2u;
    hipLaunchKernelGGL(bins_sort_kernel, grid, dim3(kBinWG), sort_lds, st, rows, cols, S, L.n_chunks, rp, ci, table, starts,
                       chunk_words, perm, order, reinterpret_cast<uint16_t *>(base + L.row_slot), bad);
    launch_scan_exclusive(starts, L.n_buckets + 1, reinterpret_cast<uint32_t *>(base + L.scan), st);
    const size_t fill_lds = (kBinMost + kBinWaves + 2u * (bins_entry_stride(S) / kBinGroup)) * 4;
    hipLaunchKernelGGL(bins_fill_kernel, grid, dim3(kBinWG), fill_lds, st, S, L.n_chunks, ci, va,
                       static_cast<const BinChunk *>(table), static_cast<const uint32_t *>(starts),
                       static_cast<const uint16_t *>(order), static_cast<const uint32_t *>(bad),
                       reinterpret_cast<float *>(base + L.va), reinterpret_cast<uint16_t *>(base + L.ci),
                       reinterpret_cast<uint32_t *>(base + L.to));
    hipLaunchKernelGGL(bins_report_kernel, dim3(1), dim3(1), 0, st, static_cast<const uint32_t *>(bad), mailbox_dev, seq);
}

void launch_bins(const SpmvArgs &a, uint32_t n_slabs, bool cut_rows, const void *plan_mem, void *workspace, hipStream_t st)
{
    const BinsLayout L = bins_layout(n_slabs, a.rows, a.nnz);
    const char *base = static_cast<const char *>(plan_mem);
    float *p = static_cast<float *>(workspace);
    char *carry = static_cast<char *>(workspace) + pad256((size_t)L.n_chunks * L.stride * 4);
    int *carry_row = reinterpret_cast<int *>(carry);
    float *carry_val = reinterpret_cast<float *>(carry + carry_workspace_bytes(L.n_chunks) / 2);
    hipLaunchKernelGGL(bins_multiply_kernel, dim3(kBinGrid), dim3(kBinWG), 0, st, a.cols, n_slabs, L.n_chunks, a.x,
                       reinterpret_cast<const uint32_t *>(base + L.starts), reinterpret_cast<const float *>(base + L.va),
                       reinterpret_cast<const uint16_t *>(base + L.ci), reinterpret_cast<const uint32_t *>(base + L.to), p);
    hipLaunchKernelGGL(bins_sum_kernel, dim3(tiles_per_xcd(L.n_chunks) * kXCD), dim3(kBinWG), 0, st, a.rows, L.n_chunks,
                       L.stride, reinterpret_cast<const BinChunk *>(base + L.table),
                       reinterpret_cast<const uint32_t *>(base + L.chunk_words),
                       reinterpret_cast<const uint16_t *>(base + L.row_slot),
                       reinterpret_cast<const uint16_t *>(base + L.perm), static_cast<const float *>(p), a.y, carry_row,
                       carry_val);
    if (cut_rows) launch_carry_fixup(a.rows, L.n_chunks, carry_row, carry_val, a.y, st);
}

} // namespace seer

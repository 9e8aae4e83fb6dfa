// Host-side declarations shared by the kernel files and the C ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/seer.h"
#include "meet.hiph"

namespace seer {

constexpr int kBmMaxRows = 2048;  // most rows one CSR,BM workgroup owns (8 per lane, bounds in registers)
constexpr int kAutoBmMaxRows = 1024;   // ... inside the combined kernel (4 per lane: keeps it at eight waves per SIMD)
constexpr int kBmChunk = 2048;    // products staged in LDS per CSR,BM pass (4096 is the other choice)
constexpr int kRangedChunk = 4096;   // ... and with its gathers ordered by column range
constexpr int kMpIptSmall = 7;    // merge items per thread, small problems (tile = 1792 items)
constexpr int kMpIptLarge = 15;   // merge items per thread, large problems (tile = 3840 items)

// Gathers ordered in time by column range (ranged_chunk_finish): x is cut into `count` ranges
// of range_bytes = 2^shift bytes, and the chip turns to the next one every `ticks` of the
// constant-rate clock.  count == 0: gathers in the order of the entries.  Cells of 2^cell_shift
// bytes, at most 64, a power of two of them to a range, tell how much of x a wave touches;
// few_cells of them are little enough for an L2.
struct GatherRanges {
    uint32_t count, shift, range_bytes, ticks, x_bytes;
    uint32_t cell_shift, few_cells;
};

// Entries of a chunk of CSR,WO that belong to rows summed elsewhere (spmv_long.hip): the first `head`
// (kLongWhole: all of them, and the row goes on) and the last `tail`.
struct LongSkip { uint16_t head, tail; };
constexpr uint16_t kLongWhole = 0x8000u;
// What CSR,WO is told of them: a word per chunk (null: no entry is left out), and, if there are such rows, the ticks of the
// gather ranges, whose turn lasts as long as what is left needs, and the chunks that have something left.
struct LongNumbers { uint32_t n[3], all, ticks, active; };     // rows of each class, all of them; as above; how many chunks
struct LongStage {
    const LongSkip *skip = nullptr;
    LongNumbers *numbers = nullptr;
    const uint32_t *active = nullptr;
    const uint32_t *rows = nullptr;          // the long rows by number, and their pieces' sums
    const float *part = nullptr;
    uint32_t slabs = 0;
};

struct SpmvArgs {
    int rows, cols, nnz;
    const int *rp, *ci;
    const float *va, *x;
    float *y;
    int remap;  // 1: tiles laid out contiguously per XCD
    int nt;     // 1: matrix streams are loaded with the non-temporal hint (keeps x in L2)
    GatherRanges ranges = GatherRanges{};   // count > 0 only where the 16-byte loads are used, too
    LongStage longs = LongStage{};          // CSR,WO with ranges only
    Meet meet = Meet{};                     // CSR,MP and CSR,WO: only where meet_applies()
};

bool tm_short_rows(int rows, int nnz);
int tm_rows_per_lane(int rows, int nnz);
uint32_t tm_num_tiles(int rows, int nnz);
void launch_tm(const SpmvArgs &a, hipStream_t st);
void launch_wm(const SpmvArgs &a, int lanes_per_row, hipStream_t st);
void launch_bm(const SpmvArgs &a, int rows_per_block, int chunk, bool vec, hipStream_t st);

// merge path: ipt is kMpIptSmall or kMpIptLarge
uint32_t mp_num_tiles(int rows, int nnz, int ipt);
size_t mp_workspace_bytes(int rows, int nnz, int ipt);
void launch_mp(const SpmvArgs &a, int ipt, bool vec, void *workspace, hipStream_t st);

// work oriented (nonzero split); shares the carry arrays' layout and the fix-up with merge path
uint32_t wo_num_tiles(int rows, int nnz);
void launch_wo(const SpmvArgs &a, bool vec, void *workspace, hipStream_t st);
size_t carry_workspace_bytes(uint32_t n_tiles);
// Cut rows meet inside the product (no carries, no fix-up launch) below 2^23 nonzeros and at up to 2^25 rows (so that the
// slots fit seer_spmv_auto_static's array), if
// the workspace has the room: with workspaces of the sizes that the size functions give, every path to CSR,MP or CSR,WO adds a row
// up in the same order; with less, but room for carries, each goes on as before there were meetings, in the order of the fix-up.
// From 2^23 nonzeros on, the wait for an exchange at the end of every workgroup, over several generations of them, is more than
// the launch where columns are near each other.  Products and steps at those sizes, us with the launch and with meetings: a band of 61 (61 M
// nonzeros), CSR,WO 94 and 102, CSR,MP 127 and 136; a band of 21 (40 M) 80 and 83; rows of 10 000 (30 M) 151 and 158.5; 8 M short
// rows (23 M) 146.2 and 147.4; scattered columns, 10 M 67.5 and 66.8, 20 M 145.0 and 144.5, Zipf rows (32 M) 219.2 and 217.4.
inline bool meet_applies(int rows, int nnz) { return nnz < (1 << 23) && rows <= (1 << 25); }
inline size_t meet_workspace_bytes(uint32_t n_tiles) { return (size_t)n_tiles * kMeetWords * 8; }
void launch_carry_fixup(int rows, uint32_t n_tiles, const int *carry_row, const float *carry_val, float *y,
                        hipStream_t st);

// adaptive (row blocks found by a preprocessing pass).  plan_mem: adaptive_plan_bytes();
// carry_ws: carry_workspace_bytes(adaptive_num_tiles()) or null when the plan has no split row
uint32_t adaptive_num_tiles(int rows, int nnz);
size_t adaptive_plan_bytes(int rows, int nnz);
int *adaptive_split_flag(void *plan_mem, int rows, int nnz);
void launch_adaptive_plan(int rows, int nnz, const int *rp, void *plan_mem, bool want_flag, hipStream_t st);
void launch_adaptive(const SpmvArgs &a, bool vec, const void *plan_mem, void *carry_ws, hipStream_t st);

// ELL,TM: plan_mem holds the ELL columns, then the ELL values (ell_plan_bytes())
uint32_t ell_rows_pad(int rows);
size_t ell_plan_bytes(int rows, int width);
// with_shift: behind the arrays lie ell_shift_bytes() more, the distances from row to column of every 64 rows, and a
// sample, from which launch_ell_judge says whether products are to use them (the mailbox's max_len)
size_t ell_shift_bytes(int rows, int width);
struct FeatureRaw;
void launch_ell_judge(int rows, int width, void *plan_mem, FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st);
void launch_ell_convert(int rows, int width, const int *rp, const int *ci, const float *va, void *plan_mem,
                        bool with_shift, hipStream_t st);
void launch_ell(const SpmvArgs &a, int width, bool with_shift, const void *plan_mem, hipStream_t st);

// COO,WM: plan_mem holds the row index of every nonzero; carry_ws: carry_workspace_bytes(coo_num_intervals())
uint32_t coo_num_intervals(int rows, int nnz);
size_t coo_plan_bytes(int rows, int nnz);
void launch_coo_convert(int rows, const int *rp, void *plan_mem, hipStream_t st);
void launch_coo(const SpmvArgs &a, bool runs /* lane-owned runs of triples (the default form) */, const void *plan_mem,
                void *carry_ws, hipStream_t st);

// CSR,S: plan_mem holds the kept virtual rows' offsets, each row's list of pieces, the slabbed
// col_idx and values, then the preprocessing's scratch (slab_plan_bytes());
// workspace: slab_workspace_bytes() (one partial per kept virtual row, then CSR,WO's carries)
constexpr int kSlabShift = 19;              // a slab of x: 2^19 columns = 2 MiB, half of one XCD's L2
uint32_t slab_count(int rows, int cols, int shift);     // 0: the form does not apply (one slab, or too many virtual rows)
size_t slab_plan_bytes(int rows, int cols, int nnz, int shift);
size_t slab_workspace_bytes(uint32_t n_kept, int nnz);
int *slab_flag(void *plan_mem, int rows, int cols, int nnz, int shift);
const uint32_t *slab_kept_count(const void *plan_mem, int rows, int cols, int nnz, int shift);
void launch_slab_count(int rows, int cols, int nnz, int shift, const int *rp, const int *ci, void *plan_mem, hipStream_t st);
void launch_slab_fill(int rows, int cols, int nnz, int shift, uint32_t n_kept, const int *rp, const int *ci, const float *va,
                      void *plan_mem, hipStream_t st);
void launch_slab(const SpmvArgs &a, uint32_t n_slabs, uint32_t n_kept, const void *plan_mem, void *workspace, hipStream_t st);

// exclusive prefix sum over n words in place (a total below 2^32), and the words of scratch it takes
size_t scan_scratch_words(size_t n);
void launch_scan_exclusive(uint32_t *data, size_t n, uint32_t *scratch, hipStream_t st);

// CSR,S in bins: the slabs of x lie in LDS.  plan_mem: bins_plan_bytes(); workspace:
// bins_workspace_bytes() (the products, then carries)
constexpr int kBinShift = 15;               // 2^15 columns, 128 KB of LDS
constexpr uint32_t kBinMaxSlabs = 256;      // at most (the preparation's counters, 3 per wave and slab, lie in LDS, too)
uint32_t bins_num_slabs(int cols);
bool bins_fit(int cols, int nnz);           // the form can hold a matrix of these sizes
size_t bins_plan_bytes(int rows, int cols, int nnz);
size_t bins_workspace_bytes(uint32_t n_slabs, int nnz);
// In two steps, each of which leaves its answer in a mailbox.  The first: max_len 1: the other form is faster for the
// matrix (not if `always`), min_len 1: some row is cut, so that products leave carries.  The second, only if the first
// says 0: max_len 1: columns do not ascend in a row, or lie outside the matrix.
void launch_bins_judge(int rows, int cols, int nnz, const int *rp, const int *ci, void *plan_mem, bool always,
                       FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st);
void launch_bins_prepare(int rows, int cols, int nnz, const int *rp, const int *ci, const float *va, void *plan_mem,
                         FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st);
void launch_bins(const SpmvArgs &a, uint32_t n_slabs, bool cut_rows, const void *plan_mem, void *workspace, hipStream_t st);

// feature reduction
struct FeatureRaw {           // written by the device into pinned host memory
    int32_t max_len, min_len;
    int32_t first, last;      // row_ptr[0], row_ptr[rows]
    uint64_t sum_sq, empty;
    uint64_t seq;             // call counter echoed back (host checks it moved)
};
size_t features_workspace_bytes(int rows);
void launch_features(int rows, const int *rp, void *workspace, FeatureRaw *mailbox_dev,
                     uint64_t seq, hipStream_t st);

// CSR,BM: when a block owns fewer rows than it has lanes, every 2^shift-th lane owns one
inline int bm_own_shift(int rows_per_block)
{
    int shift = 0;
    while ((rows_per_block << (shift + 1)) <= 256) ++shift;
    return shift;
}

// ---- asynchronous path: selection on the device, one combined SpMV kernel
constexpr int kAutoMaxNodes = 127;          // a depth-6 binary tree; fits the 4 KB kernel-argument block
struct AutoTree {                           // passed to the kernel by value
    int32_t n_nodes, pad;
    seer_node nodes[kAutoMaxNodes];
};
// A tree of depth <= 6 laid out as a complete binary tree (slot i has children 2i + 1 and
// 2i + 2): one wave can then load every node at once, evaluate all comparisons in parallel
// and find the leaf with bit operations, instead of one dependent load per level.
constexpr int kHeapInternal = 63;           // slots 0..62 can be internal nodes, 63..126 are leaves
struct AutoHeap {                           // passed to the kernel by value (896 bytes)
    int32_t feature[64];                    // -1: the slot is a leaf (or not reachable)
    double threshold[64];
    int8_t klass[128];                      // kernel id of every slot that is a leaf
};
bool flatten_tree(const seer_tree *tree, AutoHeap *heap);   // false: deeper than 6 levels of comparisons

struct AutoSel {                            // what the selection leaves in the workspace
    int32_t kernel_id, valid;               // valid: 1 gathered on the device; 2 decided on the host, no statistics
    int32_t no_longs, pad;                  // 1: no long rows of CSR,WO go apart (0: their numbers say which)
    int64_t rows, cols, nnz;
    int32_t max_len, min_len;
    uint64_t sum_sq, empty;
    float f[SEER_NUM_FEATURES];
};
// The long rows of CSR,WO with slabs of x in LDS.  select.sel: null: CSR,WO it is; else the selection.  select.heap: null: it
// has been made (nothing is done unless it says CSR,WO); else it is made here: the first pass leaves the feature partials in
// select.part, too, and the next launch the selection.  Where there is a selection, long rows of few entries together stay
// (select.all: however few they have, they go).  What CSR,WO (chunks of
// kWoChunkLarge entries) is told lies in the workspace, which begins with the slots where its cut rows meet: beside long rows it
// leaves no carries, and it writes the long rows' y.
struct FeatPartial;
struct LongSelect {
    const AutoHeap *heap = nullptr;
    FeatPartial *part = nullptr;
    AutoSel *sel = nullptr;
    uint32_t reachable = 0;
    bool all = false;
};
bool long_rows_fit(int rows);                           // rows the stage can list
size_t long_workspace_bytes(int rows, int cols, int nnz);
size_t long_workspace_most(int rows, int nnz);          // for any number of columns
LongStage launch_long(const SpmvArgs &a, const LongSelect &select, void *workspace, hipStream_t st);

struct AutoShape {                          // launch shapes, all from rows and nnz alone
    uint32_t tiles[SEER_NUM_DIRECT_KERNELS];
    int wm_lanes, bm_rows, bm_own_shift, mp_ipt;
    int tm_short;                           // CSR,TM fetches the first eight entries of a row at once (mean row length <= 8)
    int tm_pair;                            // ... and takes two rows per lane (tiles of 512 rows)
    int tm_remap;                           // CSR,TM's tile order: 1 XCD-contiguous, 0 round-robin
    GatherRanges ranges;                    // as in SpmvArgs; ticks: CSR,WO's
    uint32_t bm_ticks, mp_ticks;
    int bm_ranged;                          // CSR,BM orders its gathers, too
    uint32_t reachable;                     // bit k: the tree can answer kernel k given rows, cols and nnz (never 0)
    LongStage longs;                        // as in SpmvArgs
    Meet meet, long_meet;                   // as in SpmvArgs; for CSR,WO beside long rows
};
constexpr size_t kAutoSelOffset = 32768;    // after the 1024 feature partials of 32 bytes
constexpr size_t kAutoCarryOffset = 32768 + 256;
size_t auto_workspace_bytes(int rows, int nnz);         // the least: with carries
size_t auto_meet_workspace_bytes(int rows, int nnz);    // ... with room for cut rows to meet where they may
size_t auto_slots_bytes(int rows, int nnz);             // slots for the cut rows of CSR,MP or CSR,WO
constexpr int kAutoFusedRows = 8192;        // up to here every workgroup gathers and selects for itself, no first pass
constexpr int kAutoFusedGrid = 1024;        // the product's launch selects for itself up to this many workgroups ...
constexpr int kAutoFusedMaxRows = 0;        // ... and, whatever its grid, up to this many rows (off: measured slower; the first pass
                                            // of at most kAutoFusedParts workgroups is the slower way to read row_ptr)
constexpr uint32_t kAutoFusedParts = 64;    // partials the first pass leaves for it (one per lane of the folding wave)
constexpr uint32_t kAutoWmGrid = 4096;      // combined kernel: CSR,WM loops beyond max(this, or kAutoFusedGrid if
                                            // the selection may then run inside the launch; the other schedules' grids)
struct AutoPolicy {                         // when the selection runs inside the product's launch
    int fused_rows, fused_grid, fused_max_rows;
    int select_wave;                        // 1: the selection launch is a single wave (0: a workgroup of 1024 lanes)
    uint32_t part_rows;                     // rows per workgroup of the first pass (0: the default)
    int long_all;                           // 1: long rows go apart however few entries they have
};
// heap: the flattened tree, or null if it is too deep (then the node array is walked).
// decided: null, or the record of a choice the host could make alone (shape.reachable has
// one bit): nothing is gathered then.
void launch_auto(const SpmvArgs &a, const AutoTree &tree, const AutoHeap *heap, const AutoShape &shape, bool vec,
                 const AutoPolicy &policy, const AutoSel *decided, void *workspace, void *long_workspace /* null: no
                 stage for the long rows of CSR,WO */, hipStream_t st);

// workspace: 16 bytes.  The result goes to the mailbox; count: the two counts, sum_sq (offsets) and empty (columns),
// else sum_sq: 0 if both are zero, 1 if they have to be counted
void launch_csr_check(int rows, int cols, int nnz, const int *rp, const int *ci, void *workspace, bool count,
                      FeatureRaw *mailbox_dev, uint64_t seq, hipStream_t st);
void launch_stream_copy(void *dst, const void *src, size_t n_words, hipStream_t st);
void launch_gather_sum(const int *idx, const float *val, size_t n, const float *x, void *out64, hipStream_t st);
void launch_stream_sum(const void *src, size_t n_words, void *out64, hipStream_t st);

} // namespace seer

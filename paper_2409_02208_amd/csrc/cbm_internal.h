// Internal layout shared by the host builder, the kernel launchers and the C ABI.
#pragma once

#include <cstdint>
#include <mutex>
#include <vector>

#include "cbm.h"

// One GPU work item: start from the parent's finished row, then walk `len` entries of the
// entry stream beginning at stream[start].
//   parent  >= 0: row whose result is loaded first;  -1: none (virtual null row).
//   len     low 24 bits = number of entries; high bits = CBM_TASK_* flags.
// An entry is either a delta -- a column index with the sign in bit 31 (set = Delta-): gather that
// row of X -- or a marker (CBM_ENTRY_MARK): store the running sum as row (entry & index mask) of Y
// and keep going; the next rows of the path continue from the same registers.
// A SEGMENT task has no markers: its sum goes to scratch row `row` when the entries end.
struct CbmTask {
    int32_t row;
    int32_t parent;
    uint32_t start;
    uint32_t len_flags;
};

constexpr uint32_t CBM_TASK_LEN_MASK = 0x00ffffffu;
constexpr uint32_t CBM_TASK_INTERNAL = 0x01000000u;  // some row is compressed against this one
constexpr uint32_t CBM_TASK_SEGMENT = 0x02000000u;   // `row` is a scratch slot, not a matrix row
constexpr uint32_t CBM_DELTA_MINUS = 0x80000000u;
constexpr uint32_t CBM_ENTRY_MARK = 0x40000000u;      // entry stores a row instead of gathering one
constexpr uint32_t CBM_ENTRY_INTERNAL = 0x20000000u;  // marker: another work item reads this row, keep it unscaled
constexpr uint32_t CBM_ENTRY_INDEX_MASK = 0x1fffffffu;
// Bundled paths: the rows of a path are taken in groups of CBM_BUNDLE_ROWS, and a group's deltas come in ONE ascending
// sweep over the columns, each entry saying in bits 26-28 which row of the group it belongs to; the group's markers
// follow, tagged alike, in row order.  Rows and columns are limited to 26 bits in a handle that bundles.
constexpr uint32_t CBM_BUNDLE_SLOT_SHIFT = 26;
constexpr uint32_t CBM_BUNDLE_INDEX_MASK = 0x03ffffffu;
constexpr int32_t CBM_BUNDLE_ROWS = 4;  // most rows in a bundled path (a power of two)
// Small products of flat handles (cbm_flat.hip): rows of up to so many entries have a group of lanes each, longer ones and segments a wave, and a
// product takes this way up to so many waves.
constexpr int64_t CBM_FLAT_SHORT = 32;
constexpr int64_t CBM_FLAT_MOST_WAVES = 40960;
constexpr int CBM_XCD = 8;  // accelerator complex dies of an MI355X; workgroup (linear id) b runs on XCD b mod 8

struct CbmLevel {
    // one ROUND of dependent work (the struct keeps its first name: a round of single-row paths is a tree level)
    int64_t task_begin = 0, task_count = 0;        // into tasks[]: paths headed in this round
    int64_t comb_begin = 0, comb_count = 0;        // into comb[]: split rows of this round
    int64_t deltas = 0;                            // delta entries gathered by the round's main launch
    int64_t longest = 0;                           // entries of its longest work item
    int64_t parent_reads = 0;                      // tasks in the main launch with a parent
    int64_t rows_written = 0;                      // matrix rows written by the main launch
    int64_t comb_segments = 0;                     // scratch rows read by the combine launch
    int64_t comb_parent_reads = 0;
    bool bundled = false;                          // the round's paths are emitted as bundles (see CBM_BUNDLE_SLOT_SHIFT)
    bool long_single_rows = false;                 // every path is one row (deltas, then its marker: the same entries in either
                                                   // layout), long on average, columns below 2^26: either kernel can run the round
    // work items in locality order, cut into one contiguous block per XCD (absolute indices into tasks[])
    bool by_xcd = false;
    int64_t xcd_begin[CBM_XCD] = {}, xcd_count[CBM_XCD] = {};
};

// A row block: up to CBM_BLOCK_ROWS rows whose sums come from one walk over the columns that any of them holds.
constexpr int CBM_BLOCK_TILES = 4;                       // tiles of 32 rows
constexpr int CBM_BLOCK_ROWS = 32 * CBM_BLOCK_TILES;
struct CbmBlock {
    uint32_t row0;     // first of its CBM_BLOCK_ROWS places in block_rows
    uint32_t group0;   // first of its groups
    uint32_t ngroups;  // groups of 64 columns: four steps of 16
};
constexpr uint32_t CBM_BLOCK_NO_ROW = 0xffffffffu;  // an empty place
constexpr uint32_t CBM_BLOCK_ACTIVE = 0x80000000u;  // in a column of a group, on the device (flag_active_tiles)
constexpr float CBM_BLOCK_UP = 16777216.0f;         // 2^24: rows of X are split at this size (cbm_blocks.hip says why)

// Shared sums: a work item is a column set that is summed once, or a row made of such sums and of columns of its own.
struct CbmSumItem {
    uint32_t start, len;  // its entries: CBM_SUM_BIT | set, then columns (sets with the own column of a row that does not hold it come first)
    int32_t row;          // the row it stores
    int32_t own;          // how often the row adds its own column (negative: its sets hold it more often than the row does)
};
constexpr uint32_t CBM_SUM_BIT = 0x80000000u;
constexpr uint32_t CBM_SUM_OWN = 0x80000000u;  // in len of a row: the matrix holds the row's own column
constexpr int64_t CBM_MOST_SUMS = 1 << 19;     // 32 columns of that many fill the static scratch
// Columns of X whose sums are in memory at a time: 32 MiB of them, 128 at least and 1024 at most.
inline int64_t cbm_sum_columns(int64_t num_sums) {
    const int64_t fit = ((int64_t)8 << 20) / (num_sums > 0 ? num_sums : 1) & ~(int64_t)127;
    return fit < 128 ? 128 : fit > 1024 ? 1024 : fit;
}
// Words beside a set's sums of k columns that hold the sizes of its values (cbm_sums.hip): one for each lane, a quarter of the columns at most.
inline int64_t cbm_sum_sizes(int64_t k) { return k <= 32 ? 8 : k <= 64 ? 16 : (k + 127) / 128 * 32; }
struct CbmSumScratch {  // cbm_sum_bytes of the products that one stream, or one capture on it, enqueues
    uint64_t stream = 0, capture = 0, thread = 0;
    float* sums = nullptr;
    void* done = nullptr;  // an event; `passed`: it is behind the last of these products
    bool passed = false;
};

struct cbm_handle {
    int64_t m = 0, n = 0;
    cbm_build_opts opts{};
    int32_t eff_alpha = 0, eff_max_depth = 0, eff_hub_cap = 0, eff_max_cand = 0;
    bool square_self_loops = false;

    // ---- host copy of the format -------------------------------------------------
    std::vector<int32_t> rownnz;   // nnz of each compressed row (A or A v I)
    std::vector<int32_t> parent;   // -1 = virtual null row
    std::vector<int32_t> level;    // 1 = stored in full
    std::vector<int32_t> nplus, nminus;
    std::vector<int64_t> dptr;     // m + 1
    std::vector<uint32_t> dcol;    // Delta+ then Delta- of each row, sign in bit 31 (host copy, by row)
    std::vector<uint32_t> stream;  // the same deltas in work-item order, with row markers (uploaded)
    std::vector<float> dinv;       // d_x^-1/2 (square_self_loops only)
    std::vector<float> rinv;       // 1 / nnz of each compressed row, 0 for an empty row
    std::vector<CbmTask> tasks;
    std::vector<CbmTask> comb;     // split rows: start = first scratch slot, len = number of segments
    std::vector<int32_t> internal_rows;
    std::vector<CbmLevel> levels;  // levels[0] is round 1
    int64_t num_slots = 0;         // scratch rows needed by split rows
    int64_t seg_begin[CBM_XCD] = {}, seg_count[CBM_XCD] = {};  // segment work items in tasks[], per column range
    int64_t num_segments = 0;      // all of them
    int64_t seg_deltas = 0;        // delta entries gathered by the segment launch
    int64_t seg_longest = 0;       // entries of the longest segment
    bool whole_rows = false;       // every row is stored in full: one round of single rows, and segments
    bool flat = false;             // the same with all rows in one list, longest first
    int64_t flat_long = 0;         // how many of the rows have more than CBM_FLAT_SHORT entries
    bool flat_rich = false;        // a quarter of the entries or more are theirs or segments'
    int64_t flat_most_waves = CBM_FLAT_MOST_WAVES;
    double other_us = 0;           // > 0: products run in row blocks or through shared sums, in about this time, unless the rows as they stand
                                   // (none of them split) take less: the device holds both
    bool bundled = false;          // some round's paths are emitted as bundles: delta columns are 26-bit in this handle
    cbm_stats_t stats{};

    // ---- row blocks: where they pay, the products run on these instead of the work items above ----
    std::vector<CbmBlock> row_blocks;    // empty: none
    bool hub_blocks = false;             // the blocks hold only what long rows have in common: block_rows are scratch slots, and
                                         // the sums there are parts of split rows like the segments'
    int64_t noalloc_slots = 0;           // scratch rows that cbm_spmm_noalloc goes by: those of the handle without row blocks
    std::vector<uint32_t> block_rows;    // CBM_BLOCK_ROWS matrix rows per block
    std::vector<uint32_t> block_cols;    // 64 columns per group
    std::vector<uint32_t> block_masks;   // 64 x 4 words per group: byte s of word (l, i) = columns 8 (l / 32) .. + 7 of step i
                                         // in row 32 s + l % 32
    int64_t blk_begin[CBM_XCD] = {}, blk_count[CBM_XCD] = {};  // each XCD's run of blocks

    // ---- shared sums: where they pay, the products run on these ----
    std::vector<CbmSumItem> sum_items;   // the num_sums sets (set i = item i), then the m rows
    std::vector<uint32_t> sum_entries;
    int64_t num_sums = 0;                // 0: none
    int64_t sum_begin[2][CBM_XCD] = {}, sum_count[2][CBM_XCD] = {};  // each XCD's run of sets and of rows in sum_items
    int64_t sum_longest[2] = {};         // entries of the longest set and of the longest row
    int32_t sum_most_taken_off = 0;      // how often a row that does not hold its own column takes it off its sets' sums, at most

    // ---- device arrays (owned) ---------------------------------------------------
    int device = -1;
    bool on_device = false;
    CbmTask* d_tasks = nullptr;
    CbmTask* d_comb = nullptr;
    uint32_t* d_stream = nullptr;
    float* d_dinv = nullptr;
    float* d_rinv = nullptr;
    float* d_wstream = nullptr;  // weight of every stream entry (normalised product), computed on the device at upload
    int32_t* d_internal = nullptr;
    CbmBlock* d_blocks = nullptr;
    uint32_t* d_block_rows = nullptr;
    uint32_t* d_block_cols = nullptr;
    float* d_block_w = nullptr;  // column weight (d^-1/2) times CBM_BLOCK_UP beside each of block_cols (handles built with self-loops)
    uint32_t* d_block_masks = nullptr;
    CbmSumItem* d_sum_items = nullptr;
    uint32_t* d_sum_entries = nullptr;
    float* d_sum_w = nullptr;            // d_j^-1/2 beside a column, 1 beside a sum (handles built with self-loops)
    mutable std::mutex sum_mutex;        // held while the two launches of a chunk of columns are enqueued, and for the list below
    mutable std::vector<CbmSumScratch> sum_scratch;
    mutable float* d_scratch = nullptr;  // num_slots x scratch_k floats, sized on first use
    mutable int64_t scratch_k = 0;

    // ---- column-blocked handle: the format itself lives in `inner`, built on the B m part-rows ----
    int32_t blocks = 1;
    cbm_handle* inner = nullptr;          // owned
    mutable float* d_partial = nullptr;   // B m x partial_k floats: the part-rows' sums, sized on first use
    mutable int64_t partial_k = 0;

    // ---- per-launch profiling ----------------------------------------------------
    int profiling = 0;  // as cbm_profile_enable has it: 1 segments and rows apart, 2 the launches as they are
    mutable std::vector<cbm_launch_record> prof_records;
    mutable std::vector<void*> prof_events;  // hipEvent_t pairs

    // every product is one launch over row blocks: the work items above are never launched (and stay on the host)
    bool in_row_blocks() const { return !row_blocks.empty() && !hub_blocks; }
};

// Detail text of the most recent failure on this thread (which HIP call, which error).
void cbm_set_error_detail(const char* what, const char* detail);
const char* cbm_get_error_detail();

// host builder (cbm_builder.cpp)
cbm_status cbm_build_host(int64_t m, int64_t n, const int64_t* rowptr, const int32_t* colidx, cbm_handle* h);
cbm_status cbm_decompress_host(const cbm_handle* h, int64_t* rowptr, int32_t* colidx);

// device side (cbm_kernels.hip)
enum CbmEpilogue { CBM_EPI_NONE = 0, CBM_EPI_ROWSCALE = 1, CBM_EPI_ROWSCALE_RELU = 2, CBM_EPI_MEAN = 3, CBM_EPI_SELF = 4 };
cbm_status cbm_upload(cbm_handle* h);
void cbm_release_device(cbm_handle* h);
// Candidate search of the builder on the GPU (same candidate set as the host search): for every row the
// best `keep` (<= 16) rows to compress it against, out_y / out_w = parent and distance, out_n = how many.
cbm_status cbm_device_candidates(int device, int64_t m, int64_t n, const int64_t* rowptr, const int32_t* colidx,
                                 const int64_t* tptr, const int32_t* trow, int64_t hub_cap, int64_t min_saving,
                                 int32_t keep, std::vector<int32_t>* out_n, std::vector<int32_t>* out_y,
                                 std::vector<int32_t>* out_w);
// grow the handle's split-row scratch to k columns (no-op when it is wide enough or no row is split)
cbm_status cbm_reserve_scratch(const cbm_handle* h, int32_t k);
// Delta lists (Eq. (2)) of every tree edge on the GPU: nplus / nminus / dptr / dcol exactly as the host merge writes them.
cbm_status cbm_device_deltas(int device, int64_t m, const int64_t* rowptr, const int32_t* colidx, const int32_t* parent,
                             std::vector<int32_t>* nplus, std::vector<int32_t>* nminus, std::vector<int64_t>* dptr,
                             std::vector<uint32_t>* dcol);
cbm_status cbm_launch_product(const cbm_handle* h, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy,
                              CbmEpilogue epi, float self_weight, void* stream, bool static_scratch = false, int32_t k_rule = 0);
// (k_rule: the columns of the whole product where this is one of several goes, so that all of them add in the same order)
// the product's one launch on a handle with row blocks (cbm_blocks.hip)
void cbm_launch_blocks(const cbm_handle* h, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy, int mode, const float* rw,
                       float self_w, void* stream);
// the launch before the segments on a handle with hub blocks
void cbm_launch_hub_blocks(const cbm_handle* h, const float* X, int64_t ldx, int32_t k, float* scratch, int64_t ld_scratch, bool weighted,
                           void* stream);
// Segments and / or rows of a handle whose rows are all stored in full, for products small enough to be bound by latency (cbm_flat.hip):
// lanes per group and entry, 0 if this product is not for it; the launch, false: the runtime's last error says why not.
int cbm_flat_lanes(const cbm_handle* h, int32_t k);
inline int64_t cbm_flat_waves(const cbm_handle* h, int lanes, int64_t k) {  // of such a launch, chunks of 4 lanes columns each their own
    const int64_t shorts = h->levels[0].task_count - h->flat_long;
    return ((int64_t)h->tasks.size() - shorts + (shorts * lanes + 63) / 64) * ((k + 4 * lanes - 1) / (4 * lanes));
}
bool cbm_launch_flat(const cbm_handle* h, bool segments, bool rows, int lanes, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy,
                     float* scratch, int64_t ld_scratch, int mode, const float* rw, float self_w, bool aligned, void* stream);
// Their modelled time: a launch, the longest row's batches of eight loads in each of its groups, and the gathers at L2's rate, whole cache lines of
// them (communities of 5,000 nodes, k = 128 8.1 us; 5,000 nodes of the collaboration recipe, k = 128 15.4; 1,200 nodes, k = 200 12.4).
inline double cbm_flat_us(const cbm_handle* h, int64_t k, int lanes) {
    return 4.0 + 0.25 * (double)h->levels[0].longest * lanes / 512.0 + (double)h->stats.nnz * 4.0 * (double)(k < 32 ? 32 : k) / 12.0e6;
}
// Products through shared sums (cbm_sums.hip): one of the two launches over k <= lds columns (sums at S, lds floats apart; S = nullptr: the one
// that sums each row's sets itself), and the array for the sums of a stream's products (nullptr: none to be had; the caller holds h->sum_mutex).
void cbm_launch_sum_chunk(const cbm_handle* h, bool rows, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy, int mode, const float* rw,
                          float self_w, float* S, int64_t lds, void* stream);
CbmSumScratch* cbm_sum_scratch(const cbm_handle* h, void* stream);
void cbm_sum_release_captures(const cbm_handle* h);
void cbm_sum_enqueued(const cbm_handle* h, CbmSumScratch* s, void* stream);
bool cbm_sum_guarded(const cbm_handle* h, int mode, float self_w);  // whether the product keeps the sets' sizes beside their sums
inline size_t cbm_sum_bytes(const cbm_handle* h) {
    return (size_t)h->num_sums * cbm_sum_columns(h->num_sums) * sizeof(float) / 4 * (h->sum_most_taken_off > 0 ? 5 : 4);
}
cbm_status cbm_upload_sums(cbm_handle* h);
void cbm_release_sums(cbm_handle* h);
// scratch of cbm_spmm_noalloc: one static array per GPU
constexpr int64_t CBM_STATIC_SCRATCH_FLOATS = 16 * 1024 * 1024;  // 64 MiB
inline size_t cbm_static_scratch_bytes() { return (size_t)CBM_STATIC_SCRATCH_FLOATS * sizeof(float); }
// the same through bf16 parts (cbm_gemm_split.hip) where its own rule says so: *taken
cbm_status cbm_launch_gemm_split(int64_t M, int32_t N, int32_t K, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                 int64_t ldc, void* stream, bool* taken);
// the same with B in registers, for few columns (cbm_gemm_held.hip), where its own rule says so
cbm_status cbm_launch_gemm_held(int64_t M, int32_t N, int32_t K, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                int64_t ldc, void* stream, bool* taken);
// Workgroups for each of its panels of columns, where there is work for `wanted` and `resident` run at once: all panels' together no more than that (one that
// waited would start on its equal share when others are done: with 3 x 344 and 3 x 88 of them for 1,024 and 256 that run 300000 x 32 . 32 x 144 took 52 us instead
// of 45, 2000 x 500 . 500 x 160 11.7 instead of 8.8), and several panels' a multiple of 8, so that those that read the same rows share an XCD.
inline int64_t cbm_panel_blocks(int64_t wanted, int panels, int64_t resident) {
    if (panels == 1) return wanted < resident ? wanted : resident;
    const int64_t rounded = (wanted + CBM_XCD - 1) / CBM_XCD * CBM_XCD, each = resident / panels / CBM_XCD * CBM_XCD;
    return rounded < each ? rounded : each;
}
// Whether the panel-resident fp32 kernel also takes a B that 128-bit loads cannot read (odd width or alignment): filling the panel
// element by element has to be earned by depth and by rows.  (Up to 64 columns K from 8 to 768 or more holds B in registers instead, cbm_gemm_rules.h: the lines
// there decide for K beyond 1,024, and where an environment variable asks for these kernels.)  The staged kernel has blocks of 128 rows, so it loses where M / 128 just
// exceeds the 256 compute units, and tiles of 48 columns, which suit N from 33 to 48 (microseconds, or its share of the staged kernel's time):
//  N > 64: 132534 x 64 . 64 x 130 0.61, 132534 x 32 . 32 x 65 17.8 -> 24.2, 40000 x 32 . 32 x 250 21.5 -> 25.7;
//  N <= 64, K >= 100: 34000 x 100 . 100 x 17 0.93, 32768 rows 1.23; N = 33 to 48 40000 x 100 . 100 x 47 13.3 -> 14.9, 50000 rows 0.93, and at
//    K = 256 from 40000 rows on 0.92; few rows, both kernels short of work: 9000 x 100 . 100 x 17 0.92, 12000 rows 1.08; 8192 x 100 . 100 x 50 0.84,
//    16000 rows 0.97, 18000 rows 1.15;
//  shallower: 132534 x 64 . 64 x 47 and 200000 x 48 . 48 x 47 0.90, 100000 x 64 . 64 x 47 1.06, 132534 x 32 . 32 x 47 13.2 -> 18.5.
inline bool cbm_panel_takes_unaligned(int64_t M, int32_t N, int32_t K) {
    if (N > 64) return K >= 48;
    if (K < 100) return K >= 48 && M >= 131072;
    if (N > 32 && N <= 48) return M >= (K >= 256 ? 32769 : 49152);
    return M > 32768 || M <= (N <= 32 ? 10240 : 16384);
}
// dense fp32 MFMA matmul (cbm_gemm.hip)
cbm_status cbm_launch_gemm(int64_t M, int32_t N, int32_t K, const float* A, int64_t lda, const float* B, int64_t ldb,
                           float* C, int64_t ldc, void* stream);

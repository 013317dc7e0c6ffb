// Host-side CBM builder: binary CSR -> compression tree -> delta lists -> GPU work lists.
//
// Follows Section 2 of the paper (extended Hamming-distance graph with a virtual
// null row, spanning tree rooted at the virtual vertex, delta lists per tree
// edge, Eq. (2)) and the alpha rule of Section 2.2 ("Edge Pruning"), but never
// materialises the all-pairs distance graph: an edge (y,x) can beat the virtual
// edge of x only if  w(y,x) = nnz(a_x) + nnz(a_y) - 2|a_x n a_y| < nnz(a_x),
// i.e. |a_x n a_y| > nnz(a_y)/2, so only rows sharing a column are candidates.
// The tree is grown Prim-style from the virtual vertex with a cap on depth, then
// cut into vertical paths (one GPU work item each) whose length is chosen by a
// small latency/bandwidth cost model of the kernels.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <queue>
#include <thread>

#include "cbm_block_plan.h"
#include "cbm_internal.h"
#include "cbm_sum_plan.h"

namespace {

constexpr int32_t kDefaultMaxDepth = 16;
constexpr int32_t kDefaultHubCap = 512;
constexpr int32_t kDefaultMaxCand = 8;
constexpr int64_t kLocalityMinEntries = 24;  // mean entries per work item from which a round is scheduled by locality
constexpr double kLocalityEntries = 230.0;   // such a round's bandwidth grows by 1/230 of the base per entry in a work item
constexpr int64_t kBundleMinEntries = 96;   // mean entries per work item from which a round's paths are bundled
constexpr int64_t kShareSortItems = 8192;   // work items in an XCD's share of a round up to which they run strictly longest first
constexpr long kShareBucket = 32;           // ... beyond that: by length in buckets of this many entries, locality order inside
constexpr int64_t kLongSingleRow = 64;      // mean entries of a round of single rows from which the sweep kernel may take it (narrow X)
constexpr int64_t kBundleMinItems = 256;    // ... and the work items it must have: a round of a few long paths gains nothing from sweeps in step
constexpr int64_t kDeviceSearchMinRows = 65536;  // from here on a handle bound for a GPU searches its candidates there
constexpr int64_t kSampleMinRows = 65536;  // automatic mode samples the compressibility of matrices this large first
constexpr int32_t kSplitLenDefault = 512;  // most delta entries in one segment of a split row
constexpr int32_t kSplitMinDefault = 128;  // rows with more delta entries than this are split
constexpr int32_t kPhasesDefault = 4;      // sub-ranges of an XCD's column range, for rows of >= kFineMin entries
constexpr int32_t kFineMinDefault = 1024;

// Cost model of one product (reference: k = 128, i.e. 512-byte rows).  A launch costs a fixed
// overhead plus the larger of its bandwidth time and the latency of its longest work item: a work
// item walks its entries in batches of 8 row loads, so an entry costs about one eighth of a memory
// round trip.  Measured on MI355X: ~7 us per dependent launch, ~0.2 us per entry, ~6 TB/s.
constexpr double kLaunchUs = 7.0;
constexpr double kEntryUs = 0.2;
constexpr double kBytesPerUs = 6.0e6;
constexpr double kRefRowBytes = 512.0;
// Row blocks (Builder::row_block_cost and where it is used)
constexpr double kBlockGroupUs = 0.0012;    // per group of 64 columns and slab of 32 columns of X, the chip full
constexpr double kBlockLongestUs = 0.44;    // per group of the longest block: four waves share it
constexpr double kBlockSampleMargin = 1.1;  // blocks made last find their best rows taken
constexpr double kBlockMargin = 0.7;        // the paths' model is up to 1.5 times too high where one long row decides
constexpr double kBlockLongest = 64;        // groups of the longest block: hub rows' blocks are walked by four waves while the
                                            // rest of the chip is done (R-MAT scale 14, blocks of up to 150 groups, k = 64:
                                            // 60 us against 56 on the paths)
constexpr int64_t kBlockMinRows = 512;      // four blocks
constexpr int64_t kBlockMinDegree = 16;     // mean entries of a row
constexpr int64_t kBlockColumnGroup = 256;  // blocks whose rows' columns are taken together when a block sorts its columns
// Hub blocks (Builder::hub_blocks)
constexpr int64_t kHubMinRows = 512;
// (R-MAT: at least 4 rows 0.233 ms at scale 18 and k = 47, 6 rows 0.258, 10 rows 0.280; at scale 21 and k = 128 anything from 4 to
// 10 is within 1 %)
constexpr int64_t kHubLeast = 4;          // rows of a block that hold a column, for the block to take it
constexpr double kHubEntryUs = 7e-6;      // per slab: an entry of a split row in the gather kernels,
constexpr double kHubGroupUs = 1.5e-3;    // a group of 64 columns here
constexpr double kHubMinSavedUs = 2.0;
constexpr size_t kHubPieceMin = 16, kHubPieceMax = 64;  // groups
// (R-MAT scale 21, k = 128: up to 48, 64 or 96 entries 3.97 ms, up to 128 4.10; smaller graphs do not care)
constexpr int64_t kRestWhole = 96;        // entries that hubs leave of a row, up to which they stay one segment
// Shared sums (Builder::shared_sums)
constexpr int64_t kSumMinRows = 512;
constexpr int64_t kSumSample = 256;      // rows looked at first
constexpr double kSumMargin = 0.8;       // of the paths' modelled time
constexpr double kSumBlockMargin = 1.1;  // of the row blocks' (collaboration recipe, k = 64: 10,000 nodes, models level, 22.6 -> 14.9 us; 2,500
                                         // nodes, this one 1.9 times the other, 13.7 -> 15.1)
// What row blocks and shared sums of small matrices really take of their modelled time (row blocks of 1,024 nodes 13.2 us and measured 9.1, of
// 5,000 21 and 18; shared sums of 5,000 nodes 39 and 16, of 10,000 34 and 15): the rows as they stand may take less (cbm_flat.hip)
constexpr double kFlatBlockMargin = 0.7;
constexpr double kFlatSumMargin = 0.45;
constexpr size_t kSumLongRows = 16;      // looked at for what sets would leave of them (collaboration recipe, 13,000 to 235,868 nodes with one of 300 to
                                         // 1,500 neighbours more: 0.55 to 0.99 of what the plan then leaves, never more)
constexpr size_t kSumWindow = 256;       // items that are put in order of length among themselves
constexpr int64_t kIndexShareMinRows = 16384;  // (below, all of X is in L2 anyway)
constexpr double kIndexShareMost = 0.9;        // R-MAT 1.0, citation recipe 0.7
constexpr long kIndexShareBucket = 8;          // entries: rows this much alike stay in their order in shares of many rows
constexpr int64_t kPathChoices[] = {16, 32, 64, 128, 256};

long env_or(const char* name, long dflt) {
    const char* v = std::getenv(name);
    return v ? std::atol(v) : dflt;
}
// a tuning knob from the environment, held to the range the work lists can encode
long env_clamped(const char* name, long dflt, long lo, long hi) { return std::min(hi, std::max(lo, env_or(name, dflt))); }

// fn(t) for every t < n, each in a thread of its own (n = 1: in the caller's).  What one of them throws is thrown here once all
// have ended: out of a thread it would end the process.
template <class F>
void run_threads(int n, F&& fn) {
    if (n <= 1) {
        fn(0);
        return;
    }
    std::exception_ptr error;
    std::mutex held;
    auto keep = [&] {
        std::lock_guard<std::mutex> lock(held);
        if (!error) error = std::current_exception();
    };
    std::vector<std::thread> pool;
    pool.reserve(n);
    try {
        for (int t = 0; t < n; ++t)
            pool.emplace_back([&, t] {
                try {
                    fn(t);
                } catch (...) {
                    keep();
                }
            });
    } catch (...) {  // (no more threads to be had)
        keep();
    }
    for (auto& th : pool) th.join();
    if (error) std::rethrow_exception(error);
}

template <class F>
void parallel_chunks(int nthreads, int64_t total, int64_t chunk, F&& fn) {
    if (total <= 0) return;
    std::atomic<int64_t> next{0};
    auto worker = [&](int tid) {
        for (;;) {
            int64_t b = next.fetch_add(chunk);
            if (b >= total) break;
            fn(b, std::min(total, b + chunk), tid);
        }
    };
    run_threads((int)std::max<int64_t>(1, std::min<int64_t>(nthreads, (total + chunk - 1) / chunk)), worker);
}

// Threads that may each hold a table of n 32-bit entries: at most 1 GiB of them together.
int table_threads(int nthreads, int64_t n) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(nthreads, ((int64_t)1 << 28) / std::max<int64_t>(1, n)));
}

// |a n b| for two sorted lists; binary search when one is much longer.
int64_t intersect_size(const int32_t* a, int64_t na, const int32_t* b, int64_t nb) {
    if (na > nb) {
        std::swap(a, b);
        std::swap(na, nb);
    }
    if (na == 0) return 0;
    int64_t c = 0;
    if (nb > 32 * na) {
        const int32_t* lo = b;
        const int32_t* end = b + nb;
        for (int64_t i = 0; i < na; ++i) {
            lo = std::lower_bound(lo, end, a[i]);
            if (lo == end) break;
            if (*lo == a[i]) ++c;
        }
        return c;
    }
    int64_t i = 0, j = 0;
    while (i < na && j < nb) {
        int32_t x = a[i], y = b[j];
        c += (x == y);
        i += (x <= y);
        j += (y <= x);
    }
    return c;
}

// Transpose of a CSR pattern (fewer than 2^32 entries): tptr / trow = rows holding each column, ascending inside a
// column.  A counting sort whose row blocks (equal shares of the entries, in row order) are counted and scattered by
// one thread each; a block's start inside a column is the column's start plus what the earlier blocks put there.
void transpose_pattern(int nthreads, int64_t m, int64_t n, const int64_t* rowptr, const int32_t* colidx,
                       std::vector<int64_t>& tptr, std::vector<int32_t>& trow) {
    const int64_t nz = rowptr[m];
    tptr.assign(n + 1, 0);
    trow.resize(nz);
    const int nt = nz < (1 << 20) ? 1 : table_threads(std::min(nthreads, 64), n);
    std::vector<int64_t> rb(nt + 1, m);
    rb[0] = 0;
    for (int t = 1; t < nt; ++t) rb[t] = std::lower_bound(rowptr, rowptr + m + 1, nz * t / nt) - rowptr;
    std::vector<std::vector<uint32_t>> off(nt);
    run_threads(nt, [&](int t) {
        off[t].assign(n, 0);
        for (int64_t p = rowptr[rb[t]]; p < rowptr[rb[t + 1]]; ++p) ++off[t][colidx[p]];
    });
    for (int64_t j = 0; j < n; ++j) {
        int64_t at = tptr[j];
        for (int t = 0; t < nt; ++t) {
            const uint32_t c = off[t][j];
            off[t][j] = (uint32_t)at;
            at += c;
        }
        tptr[j + 1] = at;
    }
    run_threads(nt, [&](int t) {
        for (int64_t i = rb[t]; i < rb[t + 1]; ++i)
            for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) trow[off[t][colidx[p]]++] = (int32_t)i;
    });
}

struct Cand {
    int32_t child, parent, w;
};

struct HeapEdge {
    uint64_t key;  // (w << 1) | non-virtual : draws go to the virtual edge (Section 2.2)
    int32_t x, y;  // y = -1: virtual
    bool operator>(const HeapEdge& o) const {
        if (key != o.key) return key > o.key;
        if (x != o.x) return x > o.x;
        return y > o.y;
    }
};

struct Builder {
    cbm_handle* h;
    int64_t m, n, nnz = 0;
    int nthreads;
    int32_t alpha, min_saving, max_depth, hub_cap, max_cand;
    bool auto_depth;
    const int64_t* rowptr = nullptr;  // the matrix that is compressed: A, or A v I
    const int32_t* colidx = nullptr;
    std::vector<int64_t> own_rowptr;
    std::vector<int32_t> own_colidx;
    bool verbose = false;
    std::chrono::steady_clock::time_point last;

    const int32_t* row(int64_t i) const { return colidx + rowptr[i]; }
    int64_t rlen(int64_t i) const { return h->rownnz[i]; }
    int64_t dlen(int64_t x) const { return h->dptr[x + 1] - h->dptr[x]; }
    void lap(const char* what) {
        auto now = std::chrono::steady_clock::now();
        if (verbose)
            std::fprintf(stderr, "[cbm_build] %-22s %.3f s\n", what, std::chrono::duration<double>(now - last).count());
        last = now;
    }

    cbm_status validate(const int64_t* in_rowptr, const int32_t* in_colidx);
    void self_loops(const int64_t* in_rowptr, const int32_t* in_colidx);
    void transpose_matrix();
    std::vector<int32_t> loc;  // position of every row in a breadth-first walk of the graph (square matrices)
    void locality_order();
    bool index_shares = false;  // loc is the rows' own order, for a handle whose rows are all stored in full
    bool rows_share_by_index() const;
    void index_order();
    std::vector<int64_t> optr;  // candidate edges bucketed by parent
    std::vector<int32_t> ochild, ow;
    bool device_candidates = false;  // run the candidate search on the GPU
    bool device_optional = false;    // ... and fall back to the host threads if that fails
    bool locality = false;           // rounds of long work items will be scheduled by graph locality
    bool sample_first = false;       // estimate what a tree could save from a sample of rows before the full search
    bool skip_tree = false;          // the sample said: nothing to gain, store every row in full
    cbm_status find_candidates();
    std::vector<int32_t> kept_parent, kept_level;  // the best of the grown trees while "no tree" is being priced
    std::vector<int64_t> kept_dptr;
    void prim(int64_t seeds);
    void prim(int64_t seeds, std::vector<int32_t>& parent, std::vector<int32_t>& level, std::vector<int64_t>& dptr) const;
    void arborescence();
    void all_roots();
    void delta_lists();
    // paths
    std::vector<int64_t> cptr;
    std::vector<int32_t> cidx, order, rho, cont, next, round;
    int64_t split_min = 0, split_len = 0;
    bool bundle = false;  // rounds of long work items are emitted as bundles: a path's deltas in one sweep over the columns
    int64_t bundle_min = kBundleMinEntries;  // mean entries per work item from which a round is bundled (CBM_BUNDLE_MIN)
    int64_t bundle_min_items = kBundleMinItems;  // work items a round needs before its paths are cut for bundling (CBM_BUNDLE_MIN_ITEMS)
    int64_t locality_min = kLocalityMinEntries;  // ... from which a round is scheduled by locality (CBM_LOCALITY_MIN)
    std::vector<uint8_t> cap_rows_in_round;  // rounds whose paths plan() holds to CBM_BUNDLE_ROWS rows
    void choose_bundled_rounds(int64_t path_max, int32_t* nrounds);
    bool is_split(int64_t x) const { return dlen(x) > split_min; }
    void tree_index();
    double plan(int64_t path_max, int32_t* nrounds_out);
    double last_round_us = 0.0, last_round_bytes_us = 0.0;  // of the last round: modelled time; its bandwidth term alone
    bool prune_last_round(int64_t path_max);
    double csr_cost() const;
    cbm_status emit(int32_t nrounds);
    double row_block_cost(double groups, double longest) const;
    double sampled_row_block_cost() const;
    void row_blocks();
    void hub_blocks(bool force);
    double shared_sums_cost(double gathers, double sets, double longest) const;
    void shared_sums(const std::vector<uint8_t>& holds_own);
    int64_t count_slots() const;
    // rows in hub blocks keep only the other entries for the gather kernels
    struct Rest {
        int32_t first_block = -1, blocks = 0, place = 0;  // the row's pieces and its place in them
        std::vector<uint32_t> cols;
    };
    std::vector<int32_t> rest_of;  // row -> its Rest, -1 = none; empty: no hub blocks
    std::vector<Rest> rests;
    const Rest* rest(int64_t x) const { return rest_of.empty() || rest_of[x] < 0 ? nullptr : &rests[rest_of[x]]; }
    int64_t elen(int64_t x) const { return rest(x) ? (int64_t)rest(x)->cols.size() : dlen(x); }
    const uint32_t* entries(int64_t x) const { return rest(x) ? rest(x)->cols.data() : h->dcol.data() + h->dptr[x]; }
};

cbm_status Builder::validate(const int64_t* in_rowptr, const int32_t* in_colidx) {
    if (in_rowptr[0] != 0) return CBM_ERR_INVALID_CSR;
    for (int64_t i = 0; i < m; ++i)
        if (in_rowptr[i + 1] < in_rowptr[i]) return CBM_ERR_INVALID_CSR;
    std::atomic<bool> bad{false};
    parallel_chunks(nthreads, m, 4096, [&](int64_t b, int64_t e, int) {
        for (int64_t i = b; i < e; ++i) {
            int64_t prev = -1;
            for (int64_t p = in_rowptr[i]; p < in_rowptr[i + 1]; ++p) {
                int64_t c = in_colidx[p];
                if (c <= prev || c >= n) {
                    bad = true;
                    return;
                }
                prev = c;
            }
        }
    });
    return bad ? CBM_ERR_INVALID_CSR : CBM_OK;
}

void Builder::self_loops(const int64_t* in_rowptr, const int32_t* in_colidx) {
    own_rowptr.assign(m + 1, 0);
    for (int64_t i = 0; i < m; ++i) {
        const int32_t* b = in_colidx + in_rowptr[i];
        const int32_t* e = in_colidx + in_rowptr[i + 1];
        bool has = std::binary_search(b, e, (int32_t)i);
        own_rowptr[i + 1] = own_rowptr[i] + (e - b) + (has ? 0 : 1);
    }
    own_colidx.resize(own_rowptr[m]);
    parallel_chunks(nthreads, m, 4096, [&](int64_t b0, int64_t e0, int) {
        for (int64_t i = b0; i < e0; ++i) {
            const int32_t* b = in_colidx + in_rowptr[i];
            const int32_t* e = in_colidx + in_rowptr[i + 1];
            int32_t* out = own_colidx.data() + own_rowptr[i];
            const int32_t* pos = std::lower_bound(b, e, (int32_t)i);
            out = std::copy(b, pos, out);
            if (pos == e || *pos != (int32_t)i) *out++ = (int32_t)i;
            std::copy(pos, e, out);
        }
    });
    rowptr = own_rowptr.data();
    colidx = own_colidx.data();
}

// Replace the matrix by its transpose (n x m).  Rows are scanned in order, so every new row comes out sorted.
void Builder::transpose_matrix() {
    std::vector<int64_t> tp;
    std::vector<int32_t> tc;
    transpose_pattern(nthreads, m, n, rowptr, colidx, tp, tc);
    own_rowptr.swap(tp);
    own_colidx.swap(tc);
    rowptr = own_rowptr.data();
    colidx = own_colidx.data();
    std::swap(m, n);
}

// Breadth-first order of the rows over the graph itself (row i's columns are its neighbours): rows close in this
// order have overlapping neighbourhoods, so their delta lists gather overlapping rows of X.
void Builder::locality_order() {
    loc.assign(m, -1);
    std::vector<int32_t> queue;
    queue.reserve(m);
    int32_t pos = 0;
    for (int64_t s0 = 0; s0 < m; ++s0) {
        if (loc[s0] >= 0) continue;
        loc[s0] = pos++;
        queue.clear();
        queue.push_back((int32_t)s0);
        for (size_t qh = 0; qh < queue.size(); ++qh) {
            const int32_t x = queue[qh];
            for (int64_t p = rowptr[x]; p < rowptr[x + 1]; ++p) {
                const int32_t y = colidx[p];
                if (y < m && loc[y] < 0) {
                    loc[y] = pos++;
                    queue.push_back(y);
                }
            }
        }
    }
}

// Whether rows near each other in the matrix's own order hold the same columns: how many of the eight XCDs would gather a column if each had a
// contiguous share of the rows, against shares dealt out at random.  (Counted on every few columns, over all rows.)
// Contiguous shares, an eighth of the entries each, longest rows first inside: citation recipe, 170,000 nodes, k = 128 77 -> 69 us, k = 500 314 -> 292;
// 60,000 nodes 28 -> 24.6; 19,717 nodes, k = 500 36.4 -> 30.7, k = 64 7.3 -> 6.8.  Where the order of the rows says nothing they change nothing (directed R-MAT scale 17, k = 128 97.3 /
// 97.9), and small products of long rows do better by another way (cbm_flat.hip).
bool Builder::rows_share_by_index() const {
    if (m < kIndexShareMinRows) return false;
    int64_t longs = 0, long_rows = 0;
    for (int64_t x = 0; x < m; ++x)
        if (rlen(x) > CBM_FLAT_SHORT) longs += rlen(x), ++long_rows;
    if (4 * longs >= nnz && long_rows + (m - long_rows) / 2 <= CBM_FLAT_MOST_WAVES) return false;
    const uint32_t every = (uint32_t)std::max<int64_t>(1, nnz >> 20);
    std::vector<std::atomic<uint8_t>> near((size_t)n), far((size_t)n);  // the shares that hold a column
    parallel_chunks(nthreads, m, 4096, [&](int64_t x0, int64_t x1, int) {
        for (int64_t x = x0; x < x1; ++x) {
            if (is_split(x)) continue;
            const uint8_t here = (uint8_t)(1u << (rowptr[x] * CBM_XCD / std::max<int64_t>(1, nnz)));
            const uint8_t there = (uint8_t)(1u << ((uint32_t)x * 2654435761u >> 29));
            for (int64_t p = rowptr[x]; p < rowptr[x + 1]; ++p) {
                const uint32_t c = (uint32_t)colidx[p];
                if (every > 1 && c * 0x9e3779b1u % every) continue;
                near[c].fetch_or(here, std::memory_order_relaxed);
                far[c].fetch_or(there, std::memory_order_relaxed);
            }
        }
    });
    int64_t a = 0, b = 0;
    for (int64_t c = 0; c < n; ++c) {
        a += __builtin_popcount(near[c].load(std::memory_order_relaxed));
        b += __builtin_popcount(far[c].load(std::memory_order_relaxed));
    }
    if (verbose) std::fprintf(stderr, "[cbm_build] columns on an XCD: %ld with contiguous shares of the rows, %ld with random ones\n", (long)a, (long)b);
    return a <= kIndexShareMost * b;
}
void Builder::index_order() {
    index_shares = true;
    loc.resize((size_t)m);
    for (int64_t x = 0; x < m; ++x) loc[x] = (int32_t)x;
}

void Builder::all_roots() {
    h->parent.assign(m, -1);
    h->level.assign(m, 1);
    h->dptr.assign(m + 1, 0);
    for (int64_t x = 0; x < m; ++x) h->dptr[x + 1] = h->dptr[x] + rlen(x);
}

// Candidate parents: for every row, the rows that share columns with it, ranked by exact Hamming distance.
cbm_status Builder::find_candidates() {
    // transpose: rows holding each column
    std::vector<int64_t> tptr;
    std::vector<int32_t> trow;
    transpose_pattern(nthreads, m, n, rowptr, colidx, tptr, trow);
    lap("transpose");

    // candidate parents of one row: rows sharing columns, ranked by exact Hamming distance (the best come out in sc)
    struct Scored {
        int64_t score;  // saving = nnz(a_x) - w(y,x) = 2|a_x n a_y| - nnz(a_y) (upper bound, then exact)
        int32_t y;
    };
    auto row_candidates = [&](int64_t x, std::vector<int32_t>& cnt, std::vector<int32_t>& tch, std::vector<Scored>& sc) {
        sc.clear();
        const int64_t nx = rlen(x);
        if (nx < 1) return;
        tch.clear();
        int64_t nhub = 0;
        for (const int32_t* pj = row(x); pj != row(x) + nx; ++pj) {
            int64_t deg = tptr[*pj + 1] - tptr[*pj];
            if (hub_cap >= 0 && deg > hub_cap) {  // a hub column: too many rows to expand
                ++nhub;
                continue;
            }
            for (int64_t q = tptr[*pj]; q < tptr[*pj + 1]; ++q) {
                int32_t y = trow[q];
                if (cnt[y]++ == 0) tch.push_back(y);
            }
        }
        for (int32_t y : tch) {
            int64_t ipart = cnt[y];
            cnt[y] = 0;
            if (y == x) continue;
            int64_t ny = rlen(y);
            int64_t iub = ipart + std::min<int64_t>(nhub, std::min(ny, nx) - ipart);
            int64_t ub = 2 * iub - ny;
            if (ub >= min_saving) sc.push_back({ub, y});
        }
        if (sc.empty()) return;
        auto better = [](const Scored& a, const Scored& b2) {
            return a.score != b2.score ? a.score > b2.score : a.y < b2.y;
        };
        if (nhub > 0) {
            // shared hub columns were not counted: settle the best few by exact intersection
            size_t keep = max_cand < 0 ? sc.size() : std::min<size_t>(sc.size(), 2 * (size_t)max_cand);
            if (keep < sc.size()) {
                std::nth_element(sc.begin(), sc.begin() + keep, sc.end(), better);
                sc.resize(keep);
            }
            size_t w = 0;
            for (auto& s : sc) {
                int64_t ny = rlen(s.y);
                int64_t I = intersect_size(row(x), nx, row(s.y), ny);
                s.score = 2 * I - ny;
                if (s.score >= min_saving) sc[w++] = s;
            }
            sc.resize(w);
        }
        size_t keep = max_cand < 0 ? sc.size() : std::min<size_t>(sc.size(), (size_t)max_cand);
        if (keep < sc.size()) {
            std::nth_element(sc.begin(), sc.begin() + keep, sc.end(), better);
            sc.resize(keep);
        }
    };
    std::vector<std::vector<int32_t>> counters(nthreads), touched(nthreads);

    // Automatic mode on a large matrix: look at every 64th row first.  The best candidate of a row bounds what any
    // tree can save on it; if the sample says the whole matrix would shed under 2 % of its entries, no tree can pay
    // for a dependent launch, and the full search (the bulk of the build time) is skipped.
    if (sample_first) {
        const int64_t stride = 64, nsample = (m + stride - 1) / stride;
        std::vector<int64_t> saved(nthreads, 0), seen(nthreads, 0);
        parallel_chunks(nthreads, nsample, 16, [&](int64_t b, int64_t e, int tid) {
            auto& cnt = counters[tid];
            if (cnt.empty()) cnt.assign(m, 0);
            std::vector<Scored> sc;
            for (int64_t i = b; i < e; ++i) {
                const int64_t x = i * stride;
                row_candidates(x, cnt, touched[tid], sc);
                int64_t best = 0;
                for (auto& c : sc) best = std::max(best, c.score);
                saved[tid] += best;
                seen[tid] += rlen(x);
            }
        });
        int64_t sv = 0, sn = 0;
        for (int t = 0; t < nthreads; ++t) {
            sv += saved[t];
            sn += seen[t];
        }
        if (verbose)
            std::fprintf(stderr, "[cbm_build] sample of %ld rows: at most %.2f %% of their entries can be saved\n", (long)nsample,
                         sn > 0 ? 100.0 * sv / sn : 0.0);
        lap("candidate sample");
        if (sv * 50 < sn) {
            skip_tree = true;
            return CBM_OK;
        }
    }

    std::vector<std::vector<Cand>> cand_per_thread(nthreads);
    if (device_candidates) {
        std::vector<int32_t> cn, cy, cw;
        const cbm_status st = cbm_device_candidates(h->opts.device, m, n, rowptr, colidx, tptr.data(), trow.data(), hub_cap,
                                                    min_saving, max_cand, &cn, &cy, &cw);
        if (st != CBM_OK && !device_optional) return st;
        if (st != CBM_OK) {
            if (verbose) std::fprintf(stderr, "[cbm_build] candidate search on the GPU failed (%d): host threads instead\n", (int)st);
            device_candidates = false;
        } else {
            auto& out = cand_per_thread[0];
            for (int64_t x = 0; x < m; ++x)
                for (int32_t i = 0; i < cn[x]; ++i) out.push_back({(int32_t)x, cy[x * max_cand + i], cw[x * max_cand + i]});
        }
    }
    if (!device_candidates) {
        parallel_chunks(nthreads, m, 64, [&](int64_t b, int64_t e, int tid) {
            auto& cnt = counters[tid];
            auto& out = cand_per_thread[tid];
            if (cnt.empty()) cnt.assign(m, 0);
            std::vector<Scored> sc;
            for (int64_t x = b; x < e; ++x) {
                row_candidates(x, cnt, touched[tid], sc);
                const int64_t nx = rlen(x);
                for (auto& c : sc) out.push_back({(int32_t)x, c.y, (int32_t)(nx - c.score)});
            }
        });
    }
    std::vector<int64_t>().swap(tptr);
    std::vector<int32_t>().swap(trow);
    lap("candidates");

    // bucket candidate edges by parent: Prim pushes the out-edges of each newly attached row
    optr.assign(m + 1, 0);
    for (auto& v : cand_per_thread)
        for (auto& c : v) ++optr[c.parent + 1];
    for (int64_t i = 0; i < m; ++i) optr[i + 1] += optr[i];
    ochild.resize(optr[m]);
    ow.resize(optr[m]);
    {
        std::vector<int64_t> fill(optr.begin(), optr.end() - 1);
        for (auto& v : cand_per_thread) {
            for (auto& c : v) {
                int64_t p = fill[c.parent]++;
                ochild[p] = c.child;
                ow[p] = c.w;
            }
            std::vector<Cand>().swap(v);
        }
    }
    return CBM_OK;
}

// Prim growth from the virtual vertex over the candidate edges, depth-capped.  `seeds` rows, evenly
// spread over the index range, are forced to be stored in full before anything else is attached:
// with a depth cap, growing from many seeds at once gives wider levels (more parallel work per
// dependent launch) and often fewer deltas than growing from the few cheapest rows only.
// Also leaves in dptr[] the delta count of every row (the weight of its tree edge).
void Builder::prim(int64_t seeds) { prim(seeds, h->parent, h->level, h->dptr); }

// The same into arrays of the caller's (reads the builder only: several growths can run side by side).
void Builder::prim(int64_t seeds, std::vector<int32_t>& parent, std::vector<int32_t>& level, std::vector<int64_t>& dptr) const {
    parent.assign(m, -1);
    level.assign(m, 0);
    std::vector<int32_t> wsel(m, 0);
    std::vector<HeapEdge> init;
    init.reserve(m);
    for (int64_t x = 0; x < m; ++x) init.push_back({(uint64_t)rlen(x) << 1, (int32_t)x, -1});
    if (seeds > 0 && seeds < m)
        for (int64_t i = 0; i < seeds; ++i) init[(size_t)(i * m / seeds)].key = 0;  // popped before any other edge
    std::priority_queue<HeapEdge, std::vector<HeapEdge>, std::greater<HeapEdge>> pq(std::greater<HeapEdge>(),
                                                                                    std::move(init));
    while (!pq.empty()) {
        HeapEdge e = pq.top();
        pq.pop();
        if (level[e.x] != 0) continue;
        int32_t lvl = e.y < 0 ? 1 : level[e.y] + 1;
        parent[e.x] = e.y;
        level[e.x] = lvl;
        wsel[e.x] = e.y < 0 ? (int32_t)rlen(e.x) : (int32_t)(e.key >> 1);
        if (max_depth > 0 && lvl >= max_depth) continue;  // nothing may hang below the cap
        for (int64_t p = optr[e.x]; p < optr[e.x + 1]; ++p)
            if (level[ochild[p]] == 0) pq.push({((uint64_t)ow[p] << 1) | 1u, ochild[p], e.x});
    }
    dptr.assign(m + 1, 0);
    for (int64_t x = 0; x < m; ++x) dptr[x + 1] = dptr[x] + wsel[x];
}

// Exact minimum-cost arborescence of the candidate digraph rooted at the virtual vertex (Section 2.2,
// "Edge Pruning": once edges are pruned by direction the chain of compression is an MCA).  Edmonds'
// algorithm in Tarjan's form: every vertex keeps a meldable heap (leftist, with a lazy offset) of its
// incoming edges; walking backwards along cheapest incoming edges either reaches finished ground or
// closes a cycle, which is contracted (union-find, heaps melded, the chosen edge's cost taken off every
// edge entering that vertex).  Contractions are undone in reverse order to read off the real edges.
// Cost of an edge = (m + 1) * w + [non-virtual]: total weight first, then as few real edges as possible
// (draws go to the virtual vertex).
void Builder::arborescence() {
    const int64_t V = m + 1, root = m;  // vertex m is the virtual null row
    const int64_t E = m + (int64_t)ochild.size();
    std::vector<int32_t> src(E), dst(E), lc(E, -1), rc(E, -1), rank(E, 1);
    std::vector<int64_t> key(E), lazy(E, 0);
    std::vector<int32_t> ew(E);  // Hamming weight of the edge (delta count)
    for (int64_t x = 0; x < m; ++x) {  // virtual edges
        src[x] = (int32_t)root;
        dst[x] = (int32_t)x;
        ew[x] = (int32_t)rlen(x);
        key[x] = (int64_t)rlen(x) * V;
    }
    {
        int64_t e = m;
        for (int64_t y = 0; y < m; ++y)
            for (int64_t p = optr[y]; p < optr[y + 1]; ++p, ++e) {
                src[e] = (int32_t)y;
                dst[e] = ochild[p];
                ew[e] = ow[p];
                key[e] = (int64_t)ow[p] * V + 1;
            }
    }
    auto push_down = [&](int32_t a) {
        if (lazy[a] == 0) return;
        for (int32_t c : {lc[a], rc[a]})
            if (c >= 0) {
                key[c] += lazy[a];
                lazy[c] += lazy[a];
            }
        lazy[a] = 0;
    };
    std::function<int32_t(int32_t, int32_t)> meld = [&](int32_t a, int32_t b) -> int32_t {
        if (a < 0) return b;
        if (b < 0) return a;
        if (key[b] < key[a] || (key[b] == key[a] && b < a)) std::swap(a, b);
        push_down(a);
        rc[a] = meld(rc[a], b);
        if (lc[a] < 0 || rank[lc[a]] < rank[rc[a]]) std::swap(lc[a], rc[a]);
        rank[a] = rc[a] < 0 ? 1 : rank[rc[a]] + 1;
        return a;
    };
    std::vector<int32_t> heap(V, -1);
    for (int64_t e = 0; e < E; ++e) heap[dst[e]] = meld(heap[dst[e]], (int32_t)e);

    // union-find with rollback (union by size, no path compression)
    std::vector<int32_t> up(V), sz(V, 1);
    for (int64_t v = 0; v < V; ++v) up[v] = (int32_t)v;
    std::vector<std::pair<int32_t, int32_t>> log;  // (child root, parent root) of every union
    auto find = [&](int32_t v) {
        while (up[v] != v) v = up[v];
        return v;
    };
    auto unite = [&](int32_t a, int32_t b) {  // a, b are roots; returns the new root
        if (sz[a] < sz[b]) std::swap(a, b);
        up[b] = a;
        sz[a] += sz[b];
        log.push_back({b, a});
        return a;
    };
    struct Cycle {
        size_t log_size;                                     // union-find state before the contraction
        std::vector<std::pair<int32_t, int32_t>> members;    // (component at that time, its chosen in-edge)
        int32_t merged;                                      // component after the contraction
    };
    std::vector<Cycle> cycles;
    std::vector<int32_t> chosen(V, -1);  // chosen in-edge of a live component
    std::vector<int32_t> state(V, 0);    // 0 = untouched, 1 = on the current walk, 2 = finished
    state[root] = 2;
    std::vector<int32_t> walk;
    for (int64_t s = 0; s < m; ++s) {
        int32_t u = find((int32_t)s);
        if (state[u] != 0) continue;
        walk.clear();
        for (;;) {
            if (state[u] == 2) break;  // reached finished ground
            if (state[u] == 1) {
                // u closes a cycle with the top of the walk: contract everything above u on the walk, and u
                Cycle c;
                c.log_size = log.size();
                int32_t merged = u, h2 = -1;
                for (;;) {
                    const int32_t w = walk.back();
                    walk.pop_back();
                    c.members.push_back({w, chosen[w]});
                    h2 = meld(h2, heap[w]);
                    if (w == u) break;
                }
                for (auto& mw : c.members)
                    if (mw.first != merged) merged = unite(find(merged), find(mw.first));
                merged = find(merged);
                heap[merged] = h2;
                state[merged] = 0;
                chosen[merged] = -1;
                c.merged = merged;
                cycles.push_back(std::move(c));
                u = merged;
                continue;
            }
            state[u] = 1;
            walk.push_back(u);
            // cheapest edge entering u from outside u
            int32_t e = heap[u];
            while (e >= 0 && find(src[e]) == u) {
                push_down(e);
                e = heap[u] = meld(lc[e], rc[e]);
            }
            // every vertex has its virtual edge, so a heap never runs dry before the root is reached
            push_down(e);
            heap[u] = meld(lc[e], rc[e]);
            lc[e] = rc[e] = -1;
            chosen[u] = e;
            if (heap[u] >= 0) {  // reduced costs for the other edges entering u
                key[heap[u]] -= key[e];
                lazy[heap[u]] -= key[e];
            }
            u = find(src[e]);
        }
        for (int32_t w : walk) state[w] = 2;
    }
    // undo the contractions, newest first: inside a cycle every member keeps its chosen edge except the
    // member that the cycle's own in-edge really enters
    for (size_t i = cycles.size(); i-- > 0;) {
        Cycle& c = cycles[i];
        const int32_t e_in = chosen[c.merged];
        while (log.size() > c.log_size) {
            auto [child, parent] = log.back();
            log.pop_back();
            up[child] = child;
            sz[parent] -= sz[child];
        }
        for (auto& mw : c.members) chosen[mw.first] = mw.second;
        chosen[find(dst[e_in])] = e_in;
    }
    h->parent.assign(m, -1);
    h->level.assign(m, 0);
    h->dptr.assign(m + 1, 0);
    for (int64_t x = 0; x < m; ++x) {
        const int32_t e = chosen[x];
        h->parent[x] = src[e] == root ? -1 : src[e];
        h->dptr[x + 1] = h->dptr[x] + ew[e];
    }
    // levels by walking down from the rows stored in full
    std::vector<int64_t> cp(m + 1, 0);
    for (int64_t x = 0; x < m; ++x)
        if (h->parent[x] >= 0) ++cp[h->parent[x] + 1];
    for (int64_t x = 0; x < m; ++x) cp[x + 1] += cp[x];
    std::vector<int32_t> ch(cp[m]);
    {
        std::vector<int64_t> fill(cp.begin(), cp.end() - 1);
        for (int64_t x = 0; x < m; ++x)
            if (h->parent[x] >= 0) ch[fill[h->parent[x]]++] = (int32_t)x;
    }
    std::vector<int32_t> frontier;
    for (int64_t x = 0; x < m; ++x)
        if (h->parent[x] < 0) {
            h->level[x] = 1;
            frontier.push_back((int32_t)x);
        }
    for (size_t i = 0; i < frontier.size(); ++i) {
        const int32_t x = frontier[i];
        for (int64_t q = cp[x]; q < cp[x + 1]; ++q) {
            h->level[ch[q]] = h->level[x] + 1;
            frontier.push_back(ch[q]);
        }
    }
}

// Delta lists (Eq. (2)) of every tree edge by list merge -- or, for a handle that searched its candidates on the GPU,
// by the GPU's kernel, which writes the same lists in the same order (the host merge is the fallback).
void Builder::delta_lists() {
    bool any_parent = false;  // with every row stored in full the lists are the rows themselves: nothing to send anywhere
    for (int64_t x = 0; x < m && !any_parent; ++x) any_parent = h->parent[x] >= 0;
    if (device_candidates && any_parent) {
        const cbm_status st = cbm_device_deltas(h->opts.device, m, rowptr, colidx, h->parent.data(), &h->nplus, &h->nminus,
                                                &h->dptr, &h->dcol);
        if (st == CBM_OK) {
            lap("delta lists (GPU)");
            return;
        }
        if (verbose) std::fprintf(stderr, "[cbm_build] delta lists on the GPU failed (%d): host threads instead\n", (int)st);
    }
    h->nplus.assign(m, 0);
    h->nminus.assign(m, 0);
    parallel_chunks(nthreads, m, 1024, [&](int64_t b, int64_t e, int) {
        for (int64_t x = b; x < e; ++x) {
            int32_t y = h->parent[x];
            if (y < 0) {
                h->nplus[x] = (int32_t)rlen(x);
                continue;
            }
            int64_t I = intersect_size(row(x), rlen(x), row(y), rlen(y));
            h->nplus[x] = (int32_t)(rlen(x) - I);
            h->nminus[x] = (int32_t)(rlen(y) - I);
        }
    });
    h->dptr.assign(m + 1, 0);
    for (int64_t x = 0; x < m; ++x) h->dptr[x + 1] = h->dptr[x] + h->nplus[x] + h->nminus[x];
    h->dcol.resize(h->dptr[m]);
    parallel_chunks(nthreads, m, 1024, [&](int64_t b, int64_t e, int) {
        for (int64_t x = b; x < e; ++x) {
            uint32_t* plus = h->dcol.data() + h->dptr[x];
            int32_t y = h->parent[x];
            if (y < 0) {
                for (int64_t i = 0; i < rlen(x); ++i) plus[i] = (uint32_t)row(x)[i];
                continue;
            }
            uint32_t* minus = plus + h->nplus[x];
            const int32_t *a = row(x), *ae = a + rlen(x), *c = row(y), *ce = c + rlen(y);
            while (a != ae && c != ce) {
                if (*a == *c) {
                    ++a;
                    ++c;
                } else if (*a < *c) {
                    *plus++ = (uint32_t)*a++;
                } else {
                    *minus++ = (uint32_t)*c++ | CBM_DELTA_MINUS;
                }
            }
            while (a != ae) *plus++ = (uint32_t)*a++;
            while (c != ce) *minus++ = (uint32_t)*c++ | CBM_DELTA_MINUS;
        }
    });
    lap("delta lists");
}

// Children lists, level order, and for every row the child that should continue its path: the
// non-split child whose subtree needs the most rounds (a Strahler-number rule, so the number of
// dependent rounds is as small as the tree allows).
void Builder::tree_index() {
    int32_t depth = 0;
    for (int64_t x = 0; x < m; ++x) depth = std::max(depth, h->level[x]);
    cptr.assign(m + 1, 0);
    for (int64_t x = 0; x < m; ++x)
        if (h->parent[x] >= 0) ++cptr[h->parent[x] + 1];
    for (int64_t x = 0; x < m; ++x) cptr[x + 1] += cptr[x];
    cidx.resize(cptr[m]);
    {
        std::vector<int64_t> fill(cptr.begin(), cptr.end() - 1);
        for (int64_t x = 0; x < m; ++x)
            if (h->parent[x] >= 0) cidx[fill[h->parent[x]]++] = (int32_t)x;
    }
    order.resize(m);  // rows by level: parents before children
    {
        std::vector<int64_t> lpos(depth + 2, 0);
        for (int64_t x = 0; x < m; ++x) ++lpos[h->level[x] + 1];
        for (int l = 0; l <= depth; ++l) lpos[l + 1] += lpos[l];
        for (int64_t x = 0; x < m; ++x) order[lpos[h->level[x]]++] = (int32_t)x;
    }
    rho.assign(m, 1);
    cont.assign(m, -1);
    for (int64_t i = m - 1; i >= 0; --i) {
        const int32_t x = order[i];
        int32_t best = -1, need = 1;
        if (!is_split(x))
            for (int64_t q = cptr[x]; q < cptr[x + 1]; ++q) {
                const int32_t c = cidx[q];
                if (!is_split(c) && (best < 0 || rho[c] > rho[best])) best = c;
            }
        for (int64_t q = cptr[x]; q < cptr[x + 1]; ++q) {
            const int32_t c = cidx[q];
            need = std::max(need, c == best ? rho[c] : rho[c] + 1);
        }
        rho[x] = need;
        cont[x] = best;
    }
}

// Cut the tree into paths of at most path_max entries (deltas + one marker per row); fills next[]
// and round[] and returns the modelled time of one product in microseconds.
double Builder::plan(int64_t path_max, int32_t* nrounds_out) {
    next = cont;
    round.assign(m, 0);
    std::vector<int64_t> run(m, 0);  // entries of the path up to and including x
    std::vector<int32_t> prow(m, 0);  // rows of the path up to and including x
    int32_t nrounds = 0;
    for (int64_t i = 0; i < m; ++i) {
        const int32_t x = order[i];
        const int32_t y = h->parent[x];
        const bool continues = y >= 0 && next[y] == x;
        if (continues) {
            round[x] = round[y];
            run[x] = run[y] + dlen(x) + 1;
            prow[x] = prow[y] + 1;
        } else {
            round[x] = y < 0 ? 1 : round[y] + 1;
            run[x] = dlen(x) + 1;
            prow[x] = 1;
        }
        if (next[x] >= 0 && run[x] + dlen(next[x]) + 1 > path_max) next[x] = -1;  // cut: the child heads a new path
        // a round that is going to be bundled holds paths of at most CBM_BUNDLE_ROWS rows
        if (next[x] >= 0 && (size_t)round[x] < cap_rows_in_round.size() && cap_rows_in_round[round[x]] && prow[x] >= CBM_BUNDLE_ROWS)
            next[x] = -1;
        nrounds = std::max(nrounds, round[x]);
    }
    *nrounds_out = nrounds;
    // cost: per round, entries gathered and the longest path; split rows add one segment launch and combines
    std::vector<int64_t> entries(nrounds + 1, 0), rows(nrounds + 1, 0), longest(nrounds + 1, 0), comb(nrounds + 1, 0);
    std::vector<int64_t> heads(nrounds + 1, 0), written(nrounds + 1, 0);
    int64_t seg_entries = 0;
    bool fixup = false;
    for (int64_t i = 0; i < m; ++i) {
        const int32_t x = order[i];
        const int r = round[x];
        const int64_t nc = cptr[x + 1] - cptr[x];
        fixup = fixup || nc > 1 || (nc == 1 && next[x] < 0);
        if (is_split(x)) {
            seg_entries += dlen(x);
            comb[r] += (dlen(x) + split_len - 1) / split_len + CBM_XCD;
            continue;
        }
        entries[r] += dlen(x);
        const bool head = h->parent[x] < 0 || next[h->parent[x]] != x;
        rows[r] += 1 + (h->parent[x] >= 0 && head);  // Y write (+ parent read for a head)
        heads[r] += head;
        ++written[r];
        if (next[x] < 0) longest[r] = std::max(longest[r], run[x]);
    }
    double us = 0.0;
    if (seg_entries > 0)
        us += kLaunchUs + std::max((double)split_len * kEntryUs, seg_entries * kRefRowBytes / (2.0 * kBytesPerUs));
    for (int r = 1; r <= nrounds; ++r) {
        double round_us = 0.0, bytes_us = 0.0;
        if (entries[r] + rows[r] > 0) {
            // a round of long work items is scheduled by graph locality (see emit): more of its gathers hit in L2
            const bool local = locality && heads[r] >= 64 * CBM_XCD && entries[r] + written[r] >= locality_min * heads[r];
            // measured on the protein recipe: 1.25x the base rate at 68 entries per work item, 1.6x at 130, 2.4x at 320
            const double per_item = heads[r] > 0 ? (double)(entries[r] + written[r]) / (double)heads[r] : 0.0;
            // ... and less when there are too few long items to fill the chip (2,500 of them: 0.6 of the rate of 12,000)
            const double fill = (double)heads[r] / ((double)heads[r] + 2048.0);
            const double rate = local ? kBytesPerUs * (1.0 + std::min(1.5, per_item / kLocalityEntries)) * fill / 0.85 : kBytesPerUs;
            bytes_us = (entries[r] + rows[r]) * kRefRowBytes / rate;
            round_us += kLaunchUs + std::max(longest[r] * kEntryUs, bytes_us);
        }
        if (comb[r] > 0) {
            round_us += kLaunchUs + comb[r] * kRefRowBytes / kBytesPerUs;
            bytes_us += comb[r] * kRefRowBytes / kBytesPerUs;
        }
        us += round_us;
        last_round_us = round_us;
        last_round_bytes_us = bytes_us;
    }
    if (fixup && h->square_self_loops) us += kLaunchUs;
    return us;
}

// Rounds whose work items are long (kBundleMinEntries entries on average) and hold more than one row are going to be
// bundled; their paths are then cut again so that none has more than CBM_BUNDLE_ROWS rows.  (The rows cut off head new
// paths one round later; emit() bundles a round only if every path in it obeys the limit, so a round that the second
// cut changes in an unforeseen way simply stays in the plain layout.)  The limit is given up if it would lengthen the
// product by more than an eighth of its rounds.
void Builder::choose_bundled_rounds(int64_t path_max, int32_t* nrounds) {
    std::vector<int64_t> ent(*nrounds + 1, 0), items(*nrounds + 1, 0);
    std::vector<uint8_t> multi(*nrounds + 1, 0);
    for (int64_t x = 0; x < m; ++x) {
        if (is_split(x)) continue;
        const int32_t y = h->parent[x];
        const bool head = y < 0 || next[y] != x;
        ent[round[x]] += dlen(x) + 1;
        items[round[x]] += head;
        multi[round[x]] |= !head;
    }
    cap_rows_in_round.assign(*nrounds + 2, 0);
    bool any = false;
    for (int r = 1; r <= *nrounds; ++r)
        if (multi[r] && items[r] >= bundle_min_items && ent[r] >= bundle_min * items[r]) cap_rows_in_round[r] = 1, any = true;
    if (!any) return;
    const int32_t before = *nrounds;
    plan(path_max, nrounds);  // (the limits stay in force for every later plan() of this build)
    if (*nrounds > before + std::max(1, before / 8)) {
        // a very deep tree: the row limit would add dependent launches, which cost more than the sweeps save
        cap_rows_in_round.clear();
        plan(path_max, nrounds);
    }
}

// The paper prunes compression opportunities that do not pay for their overhead (Section 2.2, "Edge
// Pruning").  Here the overhead that matters is a whole dependent launch: if storing the heads of the LAST
// round in full costs less (a few more gathered rows in round 1) than that round's launch and latency, do
// so; the round disappears.  The round's gathered rows do not: its paths move to round 1 with their
// entries, so what is saved is the launch, the latency of its longest path where that exceeds the
// bandwidth term, and one parent-row read per head.  Returns true if the tree changed.
bool Builder::prune_last_round(int64_t path_max) {
    int32_t nr = 0;
    plan(path_max, &nr);
    if (nr <= 1) return false;
    int64_t extra = 0;
    std::vector<int32_t> heads;
    for (int64_t x = 0; x < m; ++x) {
        if (round[x] != nr) continue;
        const int32_t y = h->parent[x];
        if (y >= 0 && next[y] == x) continue;  // continues a path of this round: moves with its head
        heads.push_back((int32_t)x);
        extra += rlen(x) - dlen(x);
    }
    const double saved = last_round_us - last_round_bytes_us + heads.size() * kRefRowBytes / kBytesPerUs;
    if (saved <= extra * kRefRowBytes / kBytesPerUs) return false;
    if (verbose)
        std::fprintf(stderr, "[cbm_build] round %d (%zu heads, saves %.1f us) dropped: heads stored in full, +%ld deltas\n", nr,
                     heads.size(), saved, (long)extra);
    std::vector<int64_t> len(m);
    for (int64_t x = 0; x < m; ++x) len[x] = dlen(x);
    for (int32_t x : heads) {
        h->parent[x] = -1;
        len[x] = rlen(x);
    }
    for (int64_t x = 0; x < m; ++x) h->dptr[x + 1] = h->dptr[x] + len[x];
    for (int64_t i = 0; i < m; ++i) {  // the old level order is still parents-first
        const int32_t x = order[i];
        h->level[x] = h->parent[x] < 0 ? 1 : h->level[h->parent[x]] + 1;
    }
    tree_index();
    return true;
}

// Modelled time of one product with every row stored in full (plain CSR on the same kernels).
double Builder::csr_cost() const {
    int64_t seg = 0, ent = 0, longest = 0;
    for (int64_t x = 0; x < m; ++x) {
        if (rlen(x) > split_min) {
            seg += rlen(x);
        } else {
            ent += rlen(x) + 1;
            longest = std::max(longest, rlen(x) + 1);
        }
    }
    double us = kLaunchUs + std::max(longest * kEntryUs, ent * kRefRowBytes / kBytesPerUs);
    if (seg > 0)
        us += 2 * kLaunchUs + std::max((double)split_len * kEntryUs, seg * kRefRowBytes / (2.0 * kBytesPerUs));
    return us;
}

// Write the entry stream and the work-item lists for the paths chosen by plan().
cbm_status Builder::emit(int32_t nrounds) {
    const int phases = (int)env_clamped("CBM_PHASES", kPhasesDefault, 1, 64);
    const int64_t fine_min = env_clamped("CBM_FINE_MIN", kFineMinDefault, 1, (long)CBM_TASK_LEN_MASK);
    const int64_t rest_whole = env_clamped("CBM_REST_WHOLE", kRestWhole, 0, 1 << 20);
    // rows that a row of ANOTHER work item is compressed against keep their unscaled sum in Y
    std::vector<uint8_t> internal(m, 0);
    h->internal_rows.clear();
    for (int64_t x = 0; x < m; ++x) {
        const int64_t nc = cptr[x + 1] - cptr[x];
        internal[x] = nc > 1 || (nc == 1 && next[x] < 0);
        if (internal[x]) h->internal_rows.push_back((int32_t)x);
    }
    h->levels.assign(nrounds, CbmLevel{});
    h->tasks.clear();
    h->comb.clear();
    h->stream.clear();
    h->num_slots = 0;
    h->num_segments = 0;
    h->seg_deltas = 0;
    h->seg_longest = 0;
    int64_t split_rows = 0;
    std::vector<std::vector<CbmTask>> rtasks(nrounds + 1), rcomb(nrounds + 1);
    std::vector<std::vector<int32_t>> rrows(nrounds + 1);  // rows of each path, beside rtasks
    std::vector<std::vector<CbmTask>> seg_tasks((size_t)CBM_XCD * (phases + 1));  // [xcd][phase]; last = unphased
    // Pass 1, in order: where every work item's entries go in the stream (heads of paths and split rows only).
    struct Piece {
        int32_t x;
        int64_t base;  // first entry in the stream
    };
    std::vector<Piece> paths, splits;
    int64_t at = 0;
    for (int64_t i = 0; i < m; ++i) {
        const int32_t x = order[i];
        const int32_t y = h->parent[x];
        if (y >= 0 && next[y] == x) continue;  // not a head
        CbmLevel& R = h->levels[round[x] - 1];
        if (is_split(x)) {
            splits.push_back({x, at});
            at += elen(x);
            continue;
        }
        const int64_t start = at;
        int32_t path_rows = 0;
        for (int32_t v = x; v >= 0; v = next[v]) {
            at += dlen(v) + 1;
            R.deltas += dlen(v);
            ++R.rows_written;
            ++path_rows;
        }
        // the entry count shares a word with the work item's flags
        if (at - start > (int64_t)CBM_TASK_LEN_MASK) return CBM_ERR_UNSUPPORTED;
        paths.push_back({x, start});
        rtasks[round[x]].push_back({x, y, (uint32_t)start, (uint32_t)(at - start)});
        rrows[round[x]].push_back(path_rows);
        R.parent_reads += y >= 0;
        R.longest = std::max(R.longest, at - start);
    }
    if (at >= (int64_t)UINT32_MAX) return CBM_ERR_UNSUPPORTED;
    // Which rounds are bundled: those of long work items with more than one row.  (Measured on the protein graph: rounds
    // averaging 134 to 165 entries per work item run 11 to 21 % faster bundled, rounds averaging 105 to 120 run 5 to 10 %
    // slower -- fewer loads in flight per work item than the row-by-row kernel keeps; rounds of short items, as on the
    // collaboration graph, 8 % slower.)
    std::vector<uint8_t> round_bundled(nrounds + 1, 0);
    h->bundled = false;
    for (int r = 1; r <= nrounds && bundle; ++r) {
        int64_t ent = 0;
        int32_t most = 1;
        for (size_t i = 0; i < rtasks[r].size(); ++i) {
            ent += rtasks[r][i].len_flags & CBM_TASK_LEN_MASK;
            most = std::max(most, rrows[r][i]);
        }
        if (verbose)
            std::fprintf(stderr, "[cbm_build] round %d: %zu work items, %.1f entries each (%ld at most), at most %d rows in a path\n", r,
                         rtasks[r].size(), rtasks[r].empty() ? 0.0 : (double)ent / (double)rtasks[r].size(),
                         (long)h->levels[r - 1].longest, (int)most);
        // (a round of long single rows has the same entries in either layout: the launch picks the kernel by the width of X)
        h->levels[r - 1].long_single_rows = most == 1 && !rtasks[r].empty() && ent >= kLongSingleRow * (int64_t)rtasks[r].size();
        if (most > 1 && most <= CBM_BUNDLE_ROWS && ent >= bundle_min * (int64_t)rtasks[r].size()) {
            round_bundled[r] = 1;
            h->levels[r - 1].bundled = true;
            h->bundled = true;
        }
    }
    h->stream.resize((size_t)at);
    // A row's deltas go into the stream in ONE ascending sweep over the columns (Delta+ and Delta- merged; the sign
    // travels with the entry).  Work items that run at the same time then move through X in step, low rows first,
    // and find each other's rows in L2: 4 to 6 % off the protein product against "Delta+ then Delta-".
    const bool merge_sort = std::getenv("CBM_NO_MERGE_SORT") == nullptr;
    // Pass 2, on all threads: the entries themselves.  A path is its rows' deltas, each followed by the row's marker;
    // a split row is its deltas re-sorted by column.
    parallel_chunks(nthreads, (int64_t)paths.size(), 256, [&](int64_t b, int64_t e, int) {
        for (int64_t i = b; i < e; ++i) {
            uint32_t* out = h->stream.data() + paths[i].base;
            if (round_bundled[round[paths[i].x]]) {
                // every delta of the path (at most CBM_BUNDLE_ROWS rows), tagged with its row's place in the path, in one
                // ascending sweep; then the rows' markers, in row order
                uint32_t* first = out;
                uint32_t slot = 0;
                for (int32_t v = paths[i].x; v >= 0; v = next[v], ++slot)
                    for (int64_t q = h->dptr[v]; q < h->dptr[v + 1]; ++q) *out++ = h->dcol[q] | (slot << CBM_BUNDLE_SLOT_SHIFT);
                std::sort(first, out, [](uint32_t a, uint32_t b2) { return (a & CBM_BUNDLE_INDEX_MASK) < (b2 & CBM_BUNDLE_INDEX_MASK); });
                for (int32_t v = paths[i].x; v >= 0; v = next[v])
                    *out++ = (uint32_t)v | CBM_ENTRY_MARK | (internal[v] ? CBM_ENTRY_INTERNAL : 0u);
                continue;
            }
            for (int32_t v = paths[i].x; v >= 0; v = next[v]) {
                uint32_t* first = out;
                out = std::copy(h->dcol.begin() + h->dptr[v], h->dcol.begin() + h->dptr[v + 1], out);
                if (merge_sort && h->nminus[v] > 0)
                    std::sort(first, out, [](uint32_t a, uint32_t b2) { return (a & CBM_ENTRY_INDEX_MASK) < (b2 & CBM_ENTRY_INDEX_MASK); });
                *out++ = (uint32_t)v | CBM_ENTRY_MARK | (internal[v] ? CBM_ENTRY_INTERNAL : 0u);
            }
        }
    });
    parallel_chunks(nthreads, (int64_t)splits.size(), 4, [&](int64_t b, int64_t e, int) {
        for (int64_t i = b; i < e; ++i) {
            const int32_t x = splits[i].x;
            uint32_t* out = h->stream.data() + splits[i].base;
            std::copy(entries(x), entries(x) + elen(x), out);
            if (h->nminus[x] > 0)  // Delta+ alone is already in column order
                std::sort(out, out + elen(x), [](uint32_t a, uint32_t b2) {
                    return (a & CBM_ENTRY_INDEX_MASK) < (b2 & CBM_ENTRY_INDEX_MASK);
                });
        }
    });
    // Pass 3, in order: a long row is cut into segments that depend on nothing.  Its entries, sorted by column,
    // are cut at the CBM_XCD column-range boundaries first: all segments of one column range run on one XCD
    // (workgroup id mod 8), so the popular rows of X in that range stay in that XCD's L2.  Very long rows are cut
    // finer still: each XCD's range is walked in `phases` sub-ranges, one after the other, so that at any time an
    // XCD gathers from 1/(8 phases) of X.
    // The boundaries give every range an equal share of the split rows' entries (equal widths would overload one XCD
    // on a matrix whose popular columns sit together in the index range); cut[f] = first column of fine piece f.
    std::vector<uint32_t> cut((size_t)CBM_XCD * phases + 1, 0);
    {
        const int P = CBM_XCD * phases;
        std::vector<int64_t> upto((size_t)n + 1, 0);  // entries of split rows in columns < c
        for (const Piece& sp : splits)
            for (int64_t i = 0; i < elen(sp.x); ++i) ++upto[(h->stream[sp.base + i] & CBM_ENTRY_INDEX_MASK) + 1];
        for (int64_t c2 = 0; c2 < n; ++c2) upto[c2 + 1] += upto[c2];
        const int64_t total = upto[n];
        for (int f = 1; f < P; ++f)
            cut[f] = total > 0 ? (uint32_t)(std::lower_bound(upto.begin(), upto.end(), (total * f + P - 1) / P) - upto.begin())
                               : (uint32_t)((int64_t)f * n / P);
        cut[P] = (uint32_t)n;
        for (int f = 1; f <= P; ++f) cut[f] = std::min<uint32_t>((uint32_t)n, std::max(cut[f], cut[f - 1]));
    }
    for (const Piece& sp : splits) {
        const int32_t x = sp.x;
        const int32_t y = h->parent[x];
        CbmLevel& R = h->levels[round[x] - 1];
        ++split_rows;
        const int64_t len = elen(x);
        const int64_t base = sp.base;
        const uint32_t* ent = h->stream.data() + base;
        const int64_t slot0 = h->num_slots;
        const int fine = len >= fine_min ? phases : 1;  // pieces per XCD range
        if (const Rest* r = rest(x)) {
            for (int32_t b = 0; b < r->blocks; ++b)
                h->block_rows[(size_t)(r->first_block + b) * CBM_BLOCK_ROWS + r->place] = (uint32_t)h->num_slots++;
            if (len > 0 && len <= rest_whole) {  // what the hubs leave of a row is seldom worth a piece in every range
                seg_tasks[(size_t)(sp.x % CBM_XCD) * (phases + 1) + phases].push_back(
                    {(int32_t)h->num_slots, -1, (uint32_t)base, (uint32_t)len | CBM_TASK_SEGMENT});
                ++h->num_slots;
                h->seg_longest = std::max(h->seg_longest, len);
            }
        }
        const int npieces = rest(x) && len <= rest_whole ? 0 : CBM_XCD * fine;
        int64_t pos = 0;
        for (int f = 0; f < npieces; ++f) {
            const uint32_t hi = cut[(size_t)(f + 1) * (phases / fine)];  // columns < hi
            const int64_t end = std::partition_point(ent + pos, ent + len, [&](uint32_t e2) { return (e2 & CBM_ENTRY_INDEX_MASK) < hi; }) - ent;
            auto& list = seg_tasks[(size_t)(f / fine) * (phases + 1) + (fine > 1 ? f % fine : phases)];
            for (int64_t b = pos; b < end; b += split_len) {
                const int64_t e = std::min(end, b + split_len);
                list.push_back({(int32_t)h->num_slots, -1, (uint32_t)(base + b), (uint32_t)(e - b) | CBM_TASK_SEGMENT});
                ++h->num_slots;
                h->seg_longest = std::max(h->seg_longest, e - b);
            }
            pos = end;
        }
        const int64_t nseg = h->num_slots - slot0;
        h->seg_deltas += len;
        rcomb[round[x]].push_back({x, y, (uint32_t)slot0, (uint32_t)nseg | (internal[x] ? CBM_TASK_INTERNAL : 0u)});
        R.comb_segments += nseg;
        R.comb_parent_reads += y >= 0;
    }
    if ((int64_t)h->stream.size() >= (int64_t)UINT32_MAX) return CBM_ERR_UNSUPPORTED;
    // longest first: wave-mates get similar lengths and the tail of a launch is short
    auto longest_first = [](const CbmTask& a, const CbmTask& b2) {
        return (a.len_flags & CBM_TASK_LEN_MASK) > (b2.len_flags & CBM_TASK_LEN_MASK);
    };
    for (int j = 0; j < CBM_XCD; ++j) {  // segment work items first: one block per XCD, phases in order
        h->seg_begin[j] = (int64_t)h->tasks.size();
        for (int ph = 0; ph <= phases; ++ph) {
            auto& list = seg_tasks[(size_t)j * (phases + 1) + ph];
            std::stable_sort(list.begin(), list.end(), longest_first);
            h->tasks.insert(h->tasks.end(), list.begin(), list.end());
        }
        h->seg_count[j] = (int64_t)h->tasks.size() - h->seg_begin[j];
        h->num_segments += h->seg_count[j];
    }
    const bool by_locality = !loc.empty();
    for (int r = 1; r <= nrounds; ++r) {
        CbmLevel& R = h->levels[r - 1];
        auto& lt = rtasks[r];
        R.task_begin = (int64_t)h->tasks.size();
        R.task_count = (int64_t)lt.size();
        int64_t round_entries = 0;
        for (auto& t : lt) round_entries += (t.len_flags & CBM_TASK_LEN_MASK);
        // worth it for rounds of long work items (protein: 8 % faster); rounds of short ones lose more to the
        // ragged tail of each XCD's block than they gain (and a graph without a tree has no such order at all)
        if (by_locality && (int64_t)lt.size() >= 64 * CBM_XCD && (index_shares || round_entries >= locality_min * (int64_t)lt.size())) {
            // neighbours in the graph next to each other, one contiguous share of the entries per XCD: what the
            // work items running on an XCD at one time gather overlaps, and stays in that XCD's L2
            std::stable_sort(lt.begin(), lt.end(), [&](const CbmTask& a, const CbmTask& b2) { return loc[a.row] < loc[b2.row]; });
            const int64_t total = round_entries;
            R.by_xcd = true;
            size_t i = 0;
            int64_t seen = 0;
            for (int j = 0; j < CBM_XCD; ++j) {
                R.xcd_begin[j] = R.task_begin + (int64_t)i;
                const int64_t want = total * (j + 1) / CBM_XCD;
                while (i < lt.size() && (j == CBM_XCD - 1 || seen < want)) seen += (lt[i++].len_flags & CBM_TASK_LEN_MASK);
                R.xcd_count[j] = R.task_begin + (int64_t)i - R.xcd_begin[j];
            }
            // Inside a share the longest work items go first: which XCD gathers what is what the locality is about, and
            // a long item that starts last is the tail of the whole launch (protein product: 1.05 -> 0.80 ms; only the
            // longer half first gains half of that).  A share of very many short items has no tail to speak of and lives
            // on neighbours running side by side instead (collaboration graph with every row stored in full: 0.44 ms in
            // locality order, 0.54 ms longest-first): there the order is by length only in buckets of 32 entries,
            // locality order inside a bucket.  CBM_SHARE_SORT: 0 = locality order, 1 = longest first, n = buckets of n.
            const long share_mode = env_clamped("CBM_SHARE_SORT", -1, -1, 1 << 20);
            for (int j = 0; j < CBM_XCD; ++j) {
                auto b = lt.begin() + (R.xcd_begin[j] - R.task_begin);
                const long mode = share_mode >= 0 ? share_mode : (R.xcd_count[j] <= kShareSortItems ? 1 : index_shares ? kIndexShareBucket : kShareBucket);
                if (mode == 1)
                    std::stable_sort(b, b + R.xcd_count[j], longest_first);
                else if (mode > 1)
                    std::stable_sort(b, b + R.xcd_count[j], [&](const CbmTask& x, const CbmTask& y) {
                        return (x.len_flags & CBM_TASK_LEN_MASK) / mode > (y.len_flags & CBM_TASK_LEN_MASK) / mode;
                    });
            }
        } else {
            std::stable_sort(lt.begin(), lt.end(), longest_first);
        }
        h->tasks.insert(h->tasks.end(), lt.begin(), lt.end());
        R.comb_begin = (int64_t)h->comb.size();
        R.comb_count = (int64_t)rcomb[r].size();
        h->comb.insert(h->comb.end(), rcomb[r].begin(), rcomb[r].end());
    }
    h->stats.num_split_rows = split_rows;
    h->whole_rows = nrounds == 1 && !h->levels[0].bundled && std::all_of(h->parent.begin(), h->parent.end(), [](int32_t y) { return y < 0; });
    h->flat = h->whole_rows && !h->levels[0].by_xcd;
    h->flat_long = 0;
    h->flat_rich = false;
    h->flat_most_waves = env_clamped("CBM_FLAT_WAVES", CBM_FLAT_MOST_WAVES, 0, 1 << 30);
    if (h->flat) {
        const CbmLevel& R = h->levels[0];
        int64_t longs = h->seg_deltas;
        for (int64_t i = 0; i < R.task_count; ++i) {
            const int64_t len = (int64_t)(h->tasks[R.task_begin + i].len_flags & CBM_TASK_LEN_MASK) - 1;  // (less the marker)
            if (len <= CBM_FLAT_SHORT) break;
            ++h->flat_long;
            longs += len;
        }
        h->flat_rich = longs > 0 && 4 * longs >= h->seg_deltas + R.deltas;
    }
    if (!h->hub_blocks) h->noalloc_slots = h->num_slots;
    return CBM_OK;
}

// Scratch rows that the split rows would take if every one were cut at the column ranges (pass 3 of emit, counted only).
int64_t Builder::count_slots() const {
    const int phases = (int)env_clamped("CBM_PHASES", kPhasesDefault, 1, 64);
    const int64_t fine_min = env_clamped("CBM_FINE_MIN", kFineMinDefault, 1, (long)CBM_TASK_LEN_MASK);
    const int P = CBM_XCD * phases;
    std::vector<std::vector<int32_t>> part((size_t)table_threads(nthreads, n));
    parallel_chunks((int)part.size(), m, 4096, [&](int64_t b, int64_t e, int th) {
        if (part[th].empty()) part[th].assign((size_t)n, 0);
        for (int64_t x = b; x < e; ++x)
            if (is_split(x))
                for (int64_t i = h->dptr[x]; i < h->dptr[x + 1]; ++i) ++part[th][h->dcol[i] & CBM_ENTRY_INDEX_MASK];
    });
    std::vector<int64_t> upto((size_t)n + 1, 0);
    parallel_chunks(nthreads, n, 16384, [&](int64_t b, int64_t e, int) {
        for (const auto& p : part)
            if (!p.empty())
                for (int64_t c = b; c < e; ++c) upto[c + 1] += p[c];
    });
    for (int64_t c = 0; c < n; ++c) upto[c + 1] += upto[c];
    std::vector<uint32_t> cut((size_t)P + 1, 0);
    const int64_t total = upto[n];
    for (int f = 1; f < P; ++f)
        cut[f] = total > 0 ? (uint32_t)(std::lower_bound(upto.begin(), upto.end(), (total * f + P - 1) / P) - upto.begin()) : (uint32_t)((int64_t)f * n / P);
    cut[P] = (uint32_t)n;
    for (int f = 1; f <= P; ++f) cut[f] = std::min<uint32_t>((uint32_t)n, std::max(cut[f], cut[f - 1]));
    std::atomic<int64_t> slots{0};
    parallel_chunks(nthreads, m, 4096, [&](int64_t b, int64_t e, int) {
        int64_t mine = 0;
        for (int64_t x = b; x < e; ++x) {
            if (!is_split(x)) continue;
            const uint32_t *ent = h->dcol.data() + h->dptr[x], *end = ent + dlen(x);
            const int fine = dlen(x) >= fine_min ? phases : 1;
            for (int f = 0; f < CBM_XCD * fine; ++f) {
                const uint32_t* to = std::lower_bound(ent, end, cut[(size_t)(f + 1) * (phases / fine)]);
                mine += (to - ent + split_len - 1) / split_len;
                ent = to;
            }
        }
        slots += mine;
    });
    return slots;
}

// Hub blocks: where no tree pays, long rows still share the popular columns.  The split rows, longest first, are cut into blocks
// of CBM_BLOCK_ROWS; a column that at least `least` of a block's rows hold goes into the block (one row of X gathered for
// all of them, on the matrix cores), the rest of a row stays with the gather kernels.  A block is walked in pieces of bounded
// length, each of which writes one partial sum per row into the scratch rows that the combine launch adds up anyway.
// Measured (with / without): R-MAT scale 21, k = 128 3.97 / 4.42 ms (43 M of the split rows' 104 M entries in 77,000 groups;
// what is left hits L2 less), scale 20, k = 128 1.69 / 2.02, scale 18, k = 47 0.235 / 0.330, scale 15, k = 64 0.065 / 0.078.
void Builder::hub_blocks(bool force) {
    std::vector<int32_t> rows;
    for (int64_t x = 0; x < m; ++x)
        if (is_split(x)) rows.push_back((int32_t)x);
    if (rows.empty() || ((int64_t)rows.size() < kHubMinRows && !force)) return;
    std::stable_sort(rows.begin(), rows.end(), [&](int32_t a, int32_t c) { return dlen(a) > dlen(c); });
    constexpr int64_t per = CBM_BLOCK_ROWS;
    constexpr int T = CBM_BLOCK_TILES;
    const int least = (int)env_clamped("CBM_HUB_LEAST", kHubLeast, 2, CBM_BLOCK_ROWS);
    const int64_t nb = ((int64_t)rows.size() + per - 1) / per;
    // how often each column is held: blocks take their columns most popular first, so that those running at one time are at
    // the same rows of X
    std::vector<int32_t> held((size_t)n, 0);
    {
        std::vector<std::vector<int32_t>> part((size_t)table_threads(nthreads, n));
        parallel_chunks((int)part.size(), (int64_t)rows.size(), 256, [&](int64_t b, int64_t e, int th) {
            if (part[th].empty()) part[th].assign((size_t)n, 0);
            for (int64_t r = b; r < e; ++r)
                for (int64_t i = h->dptr[rows[r]]; i < h->dptr[rows[r] + 1]; ++i) ++part[th][h->dcol[i]];
        });
        parallel_chunks(nthreads, n, 16384, [&](int64_t b, int64_t e, int) {
            for (const auto& p : part)
                if (!p.empty())
                    for (int64_t c = b; c < e; ++c) held[c] += p[c];
        });
    }
    struct Built {
        std::vector<uint32_t> cols, masks;
    };
    std::vector<Built> built((size_t)nb);
    rests.resize(rows.size());
    std::vector<std::vector<int32_t>> local((size_t)table_threads(nthreads, n));
    std::atomic<int64_t> taken{0};
    parallel_chunks((int)local.size(), nb, 1, [&](int64_t b0, int64_t b1, int th) {
        std::vector<int32_t>& count = local[th];  // column -> how many rows of the block hold it, then its place (negative)
        if (count.empty()) count.assign((size_t)n, 0);
        std::vector<uint32_t> cols;
        for (int64_t b = b0; b < b1; ++b) {
            const int64_t r0 = b * per, r1 = std::min<int64_t>((int64_t)rows.size(), r0 + per);
            cols.clear();
            for (int64_t r = r0; r < r1; ++r)
                for (int64_t i = h->dptr[rows[r]]; i < h->dptr[rows[r] + 1]; ++i)
                    if (++count[h->dcol[i]] == least) cols.push_back(h->dcol[i]);
            std::sort(cols.begin(), cols.end(), [&](uint32_t a, uint32_t c) { return held[a] != held[c] ? held[a] > held[c] : a < c; });
            cols.resize(cols.size() / 64 * 64);  // whole groups
            for (int64_t r = r0; r < r1; ++r)
                for (int64_t i = h->dptr[rows[r]]; i < h->dptr[rows[r] + 1]; ++i) count[h->dcol[i]] = 0;
            for (size_t i = 0; i < cols.size(); ++i) count[cols[i]] = -(int32_t)i - 1;
            Built& out = built[b];
            out.cols = cols;
            out.masks.assign(cols.size() * 4, 0u);
            int64_t mine = 0;
            for (int64_t r = r0; r < r1; ++r) {
                const int32_t x = rows[r], at = (int32_t)(r - r0);
                std::vector<uint32_t>& left = rests[r].cols;
                left.reserve((size_t)dlen(x));
                for (int64_t q = h->dptr[x]; q < h->dptr[x + 1]; ++q) {
                    const int32_t place = -count[h->dcol[q]] - 1;
                    if (place < 0) {
                        left.push_back(h->dcol[q]);
                        continue;
                    }
                    const size_t i = (size_t)place;
                    out.masks[i / 64 * 256 + 4 * (at % 32 + 32 * (i % 16 / 8)) + i % 64 / 16] |= 1u << (8 * (at / 32) + i % 8);
                    ++mine;
                }
            }
            for (uint32_t c : cols) count[c] = 0;
            taken += mine;
        }
    });
    std::vector<std::vector<int32_t>>().swap(local);
    static_assert(T == 4, "a mask word has a byte per tile");
    size_t groups = 0;
    for (const Built& x : built) groups += x.cols.size() / 64;
    // worth it?  per slab of 32 columns of X: 1.5 ns a group, 7 ns a thousand entries gathered from L2
    const double saved = (double)taken * kHubEntryUs - (double)groups * kHubGroupUs;
    if (verbose)
        std::fprintf(stderr, "[cbm_build] hub blocks: %ld rows, %zu groups of 64 columns hold %ld of their entries, saving %.1f us a slab\n",
                     (long)rows.size(), groups, (long)taken.load(), saved);
    // pieces: enough to fill the chip, long enough that the partial sums they add are few
    const long forced_piece = env_or("CBM_HUB_PIECE", 0);
    const size_t most = forced_piece > 0 ? (size_t)forced_piece : std::min<size_t>(kHubPieceMax, std::max<size_t>(kHubPieceMin, groups / 768));
    size_t pieces = 0;
    for (const Built& x : built) pieces += (x.cols.size() / 64 + most - 1) / most;
    if (groups == 0 || (saved < kHubMinSavedUs && !force)) {
        rests.clear();
        return;
    }
    const int64_t slots_without = count_slots();
    rest_of.assign((size_t)m, -1);
    for (size_t r = 0; r < rows.size(); ++r) rest_of[rows[r]] = (int32_t)r;
    h->block_cols.clear();
    h->block_masks.clear();
    h->block_rows.assign(pieces * per, CBM_BLOCK_NO_ROW);
    std::vector<CbmBlock> all;
    for (int64_t b = 0; b < nb; ++b) {
        const size_t ng = built[b].cols.size() / 64;
        const int32_t first = (int32_t)all.size();
        for (size_t g = 0; g < ng; g += most)
            all.push_back({(uint32_t)(all.size() * per), (uint32_t)(h->block_cols.size() / 64 + g), (uint32_t)std::min(most, ng - g)});
        for (int64_t r = b * per; r < std::min<int64_t>((int64_t)rows.size(), (b + 1) * per); ++r) {
            rests[r].first_block = first;
            rests[r].blocks = (int32_t)all.size() - first;
            rests[r].place = (int32_t)(r - b * per);
        }
        h->block_cols.insert(h->block_cols.end(), built[b].cols.begin(), built[b].cols.end());
        h->block_masks.insert(h->block_masks.end(), built[b].masks.begin(), built[b].masks.end());
        built[b] = Built{};
    }
    // longest pieces first, dealt over the XCDs
    std::vector<int32_t> by(all.size());
    for (size_t i = 0; i < by.size(); ++i) by[i] = (int32_t)i;
    std::stable_sort(by.begin(), by.end(), [&](int32_t a, int32_t c) { return all[a].ngroups > all[c].ngroups; });
    h->row_blocks.clear();
    for (int j = 0; j < CBM_XCD; ++j) {
        h->blk_begin[j] = (int64_t)h->row_blocks.size();
        for (size_t i = j; i < by.size(); i += CBM_XCD) h->row_blocks.push_back(all[by[i]]);
        h->blk_count[j] = (int64_t)h->row_blocks.size() - h->blk_begin[j];
    }
    h->hub_blocks = true;
    h->noalloc_slots = slots_without;
    lap("hub blocks");
}

// Modelled time of the row-block launch over `groups` groups of 64 columns (k = 128: four column slabs).  Measured: 1.2 ns a
// group and slab with the chip full (protein recipe, 34,700 groups: 0.18 ms at k = 128, 0.32 to 0.39 ms at k = 256 with the clock); with few blocks
// the launch lasts as long as its longest block (6,000 nodes, 60 neighbours: blocks of 13 groups, 11.4 us a product against
// 18.3 us on the paths; 300 neighbours: 26 groups, 18 against 29 us).
double Builder::row_block_cost(double groups, double longest) const {
    if (longest > kBlockLongest) return 1e300;
    return kLaunchUs + std::max(groups * 4 * kBlockGroupUs, longest * kBlockLongestUs);
}

// What row blocks would cost, from the blocks that a few evenly spread rows and the rows nearest to them would make: the
// number of columns a block needs decides, and a matrix whose neighbouring rows have little in common shows it at once.
double Builder::sampled_row_block_cost() const {
    std::vector<int32_t> mark((size_t)n, -1), members;
    std::vector<uint8_t> in((size_t)m, 0);
    constexpr int kSeeds = 32;
    double columns = 0, most = 0;
    int seen = 0;
    for (int q = 0; q < kSeeds; ++q) {
        const int32_t s = (int32_t)(m * q / kSeeds);
        if (rlen(s) == 0) continue;
        members.assign(1, s);
        in[s] = 1;
        nearest_rows(s, rowptr, colidx, [&](int32_t y) { return y < m && !in[y]; }, mark, [&](int32_t y) {
            if ((int64_t)members.size() < CBM_BLOCK_ROWS) {
                in[y] = 1;
                members.push_back(y);
            }
        });
        for (size_t i = 1; i < members.size() && (int64_t)members.size() < CBM_BLOCK_ROWS; ++i)  // too few neighbours: theirs
            for (int64_t p = rowptr[members[i]]; p < rowptr[members[i] + 1] && (int64_t)members.size() < CBM_BLOCK_ROWS; ++p)
                if (colidx[p] < m && !in[colidx[p]]) {
                    in[colidx[p]] = 1;
                    members.push_back(colidx[p]);
                }
        int64_t distinct = 0;
        for (int32_t x : members)
            for (int64_t p = rowptr[x]; p < rowptr[x + 1]; ++p)
                if (mark[colidx[p]] != (int32_t)m + q) {
                    mark[colidx[p]] = (int32_t)m + q;
                    ++distinct;
                }
        for (int32_t x : members) in[x] = 0;
        columns += (double)distinct / (double)members.size();
        most = std::max(most, (double)distinct);
        ++seen;
    }
    if (!seen) return 1e300;
    return row_block_cost(kBlockSampleMargin * columns / seen * (double)m / 64.0, most / 64.0);
}

// Row blocks (cbm_blocks.hip): rows in an order of much the same columns, cut every CBM_BLOCK_ROWS rows; a block's columns
// sorted by where their own rows lie in that order, coarsely, so that blocks that run side by side ask for the same rows of X
// at about the same time (L2 misses 59 -> 42 % of requests on the protein recipe), and then by which of the block's tiles hold
// them, so that a step of 16 columns touches as few tiles as it can (2.6 -> 2.1 of 4 with the rows sorted into tiles).
void Builder::row_blocks() {
    constexpr int64_t per = CBM_BLOCK_ROWS;
    constexpr int T = CBM_BLOCK_TILES;
    const std::vector<int32_t> rows = block_order(m, rowptr, colidx, per);
    const int64_t nb = (m + per - 1) / per;
    std::vector<int32_t> pos((size_t)m);
    for (int64_t i = 0; i < m; ++i) pos[rows[i]] = (int32_t)i;
    struct Built {
        std::vector<uint32_t> cols, masks;
    };
    std::vector<Built> built((size_t)nb);
    h->block_rows.assign((size_t)nb * per, CBM_BLOCK_NO_ROW);
    std::vector<std::vector<int32_t>> local((size_t)table_threads(nthreads, n));
    parallel_chunks((int)local.size(), nb, 4, [&](int64_t b0, int64_t b1, int th) {
        std::vector<int32_t>& place = local[th];  // column -> its place among the block's columns
        if (place.empty()) place.assign((size_t)n, -1);
        std::vector<int32_t> cols, by;
        std::vector<uint32_t> bits;  // T words per column: the rows of each tile that hold it
        std::vector<uint64_t> keys, alike;
        for (int64_t b = b0; b < b1; ++b) {
            cols.clear();
            bits.clear();
            uint32_t* mine = h->block_rows.data() + (size_t)(b * per);
            const int count = (int)(std::min(m, (b + 1) * per) - b * per);
            for (int i = 0; i < count; ++i) mine[i] = (uint32_t)rows[b * per + i];
            tiles_of_alike_rows(mine, count, 32, rowptr, colidx, place, alike);
            for (int i = 0; i < count; ++i)
                for (int64_t p = rowptr[mine[i]]; p < rowptr[mine[i] + 1]; ++p) {
                    int32_t& at = place[colidx[p]];
                    if (at < 0) {
                        at = (int32_t)cols.size();
                        cols.push_back(colidx[p]);
                        bits.insert(bits.end(), T, 0u);
                    }
                    bits[(size_t)at * T + i / 32] |= 1u << (i % 32);
                }
            keys.resize(cols.size());
            by.resize(cols.size());
            for (size_t i = 0; i < cols.size(); ++i) {
                place[cols[i]] = -1;
                by[i] = (int32_t)i;
                uint64_t none = 0;  // the tiles without this column
                for (int s = 0; s < T; ++s) none |= (uint64_t)(bits[i * T + s] == 0) << s;
                keys[i] = (uint64_t)(pos[cols[i]] / (per * kBlockColumnGroup)) << 36 | none << 32 | (uint32_t)pos[cols[i]];
            }
            std::sort(by.begin(), by.end(), [&](int32_t i, int32_t j) { return keys[i] < keys[j]; });
            const size_t groups = (by.size() + 63) / 64;
            Built& out = built[b];
            out.cols.resize(groups * 64);
            out.masks.assign(groups * 256, 0u);
            for (size_t i = 0; i < groups * 64; ++i) {
                const int32_t j = by[std::min(i, by.size() - 1)];
                out.cols[i] = (uint32_t)cols[j];  // (places past the last column repeat it, with no bits)
                if (i >= by.size()) continue;
                uint32_t* words = out.masks.data() + i / 64 * 256 + (i % 16 / 8) * 128 + i % 64 / 16;
                for (int s = 0; s < T; ++s)
                    for (uint32_t w = bits[(size_t)j * T + s]; w; w &= w - 1) words[4 * __builtin_ctz(w)] |= 1u << (8 * s + i % 8);
            }
        }
    });
    h->row_blocks.resize((size_t)nb);
    size_t at = 0;
    for (int64_t b = 0; b < nb; ++b) {
        h->row_blocks[b] = {(uint32_t)(b * per), (uint32_t)at, (uint32_t)(built[b].cols.size() / 64)};
        at += built[b].cols.size() / 64;
    }
    h->block_cols.resize(at * 64);
    h->block_masks.resize(at * 256);
    parallel_chunks(nthreads, nb, 4, [&](int64_t b0, int64_t b1, int) {
        for (int64_t b = b0; b < b1; ++b) {
            std::copy(built[b].cols.begin(), built[b].cols.end(), h->block_cols.begin() + (size_t)h->row_blocks[b].group0 * 64);
            std::copy(built[b].masks.begin(), built[b].masks.end(), h->block_masks.begin() + (size_t)h->row_blocks[b].group0 * 256);
        }
    });
    // One contiguous share of equal work per XCD, in the order of the rows (neighbours run side by side and share rows of X
    // in that XCD's L2) except that the smallest quarter comes last: the launch then ends on short blocks (k = 32: 58 -> 54 us,
    // nothing lost at k = 256, where longest-first throughout costs 2 %).
    size_t i = 0;
    for (int j = 0; j < CBM_XCD; ++j) {
        h->blk_begin[j] = (int64_t)i;
        const size_t want = at * (j + 1) / CBM_XCD;
        while (i < (size_t)nb && (j == CBM_XCD - 1 || h->row_blocks[i].group0 + h->row_blocks[i].ngroups / 2 < want)) ++i;
        h->blk_count[j] = (int64_t)i - h->blk_begin[j];
        const auto first = h->row_blocks.begin() + h->blk_begin[j], end = h->row_blocks.begin() + i;
        std::vector<uint32_t> sizes;
        for (auto it = first; it != end; ++it) sizes.push_back(it->ngroups);
        if (sizes.empty()) continue;
        std::nth_element(sizes.begin(), sizes.begin() + sizes.size() / 4, sizes.end());
        const uint32_t few = sizes[sizes.size() / 4];
        std::stable_partition(first, end, [&](const CbmBlock& c) { return c.ngroups > few; });
    }
    if (verbose)
        std::fprintf(stderr, "[cbm_build] row blocks: %ld of %ld rows, %zu groups of 64 columns (%.1f columns a row)\n", (long)nb, (long)per,
                     at, 64.0 * at / m);
}

// Modelled time of one product through shared sums: two dependent launches of gathers.
double Builder::shared_sums_cost(double gathers, double sets, double longest) const {
    return 2 * kLaunchUs + std::max(longest * kEntryUs, (gathers + sets + (double)m) * kRefRowBytes / kBytesPerUs);
}

// Sets and rows as work items.  Rows of the same largest set come one after the other, on one XCD: its sum is then read from that XCD's L2.
// Inside stretches of kSumWindow items the longest come first, so that the items of a wave are of one length.
void Builder::shared_sums(const std::vector<uint8_t>& holds_own) {
    const SharedSums S = SharedSumFinder(m, rowptr, colidx, holds_own.data()).find([&](int64_t total, auto&& fn) {
        parallel_chunks(nthreads, total, 16, [&](int64_t b, int64_t e, int) { fn(b, e); });
    });
    const int64_t ns = S.num_sets();
    if (ns == 0 || ns > CBM_MOST_SUMS) return;
    auto set_len = [&](int64_t g) { return S.set_ptr[g + 1] - S.set_ptr[g]; };
    auto by_window = [&](std::vector<int32_t>& order, auto&& len) {
        for (size_t b = 0; b < order.size(); b += kSumWindow)
            std::stable_sort(order.begin() + b, order.begin() + std::min(order.size(), b + kSumWindow), [&](int32_t x, int32_t y) { return len(x) > len(y); });
    };
    std::vector<int32_t> sets((size_t)ns), at((size_t)ns), rows((size_t)m), largest((size_t)m, (int32_t)ns);
    for (int64_t g = 0; g < ns; ++g) sets[g] = (int32_t)g;
    by_window(sets, set_len);
    for (int64_t i = 0; i < ns; ++i) at[sets[i]] = (int32_t)i;
    std::vector<int32_t> len((size_t)m);
    parallel_chunks(nthreads, m, 1024, [&](int64_t x0, int64_t x1, int) {
        for (int64_t x = x0; x < x1; ++x) {
            rows[x] = (int32_t)x;
            int64_t most = 0;
            for (int64_t q = S.row_ptr[x]; q < S.row_ptr[x + 1]; ++q)
                if (set_len(S.row_sets[q]) > most) most = set_len(S.row_sets[q]), largest[x] = S.row_sets[q];
            int64_t single = -(int64_t)holds_own[x];  // (the own column is never covered)
            for (int64_t p = rowptr[x]; p < rowptr[x + 1]; ++p) single += !S.covered[p];
            len[x] = (int32_t)(S.row_ptr[x + 1] - S.row_ptr[x] + single);
        }
    });
    std::stable_sort(rows.begin(), rows.end(), [&](int32_t x, int32_t y) { return largest[x] < largest[y]; });
    by_window(rows, [&](int32_t x) { return len[x]; });
    h->num_sums = ns;
    h->sum_items.resize((size_t)(ns + m));
    uint32_t end = 0;
    for (int64_t i = 0; i < ns; ++i) {
        h->sum_items[i] = {end, (uint32_t)set_len(sets[i]), 0, 0};
        end += (uint32_t)set_len(sets[i]);
    }
    for (int64_t i = 0; i < m; ++i) {
        const int32_t x = rows[i];
        h->sum_items[ns + i] = {end, (uint32_t)len[x] | (holds_own[x] ? CBM_SUM_OWN : 0u), x, S.own[x]};
        if (!holds_own[x]) h->sum_most_taken_off = std::max(h->sum_most_taken_off, -S.own[x]);
        end += (uint32_t)len[x];
    }
    h->sum_entries.resize(end);
    parallel_chunks(nthreads, ns + m, 1024, [&](int64_t i0, int64_t i1, int) {
        for (int64_t i = i0; i < i1; ++i) {
            uint32_t* e = h->sum_entries.data() + h->sum_items[i].start;
            if (i < ns) {
                std::copy(S.set_cols.begin() + S.set_ptr[sets[i]], S.set_cols.begin() + S.set_ptr[sets[i] + 1], e);
                continue;
            }
            const int32_t x = rows[i - ns];
            auto add_sets = [&](bool with_own) {
                for (int64_t q = S.row_ptr[x]; q < S.row_ptr[x + 1]; ++q) {
                    const int32_t *b = S.set_cols.data() + S.set_ptr[S.row_sets[q]], *t = S.set_cols.data() + S.set_ptr[S.row_sets[q] + 1];
                    if (holds_own[x] ? with_own : std::binary_search(b, t, x) == with_own) *e++ = CBM_SUM_BIT | (uint32_t)at[S.row_sets[q]];
                }
            };
            add_sets(true);  // (of a row that does not hold its own column: the sets that do come first, -own of them)
            add_sets(false);
            for (int64_t p = rowptr[x]; p < rowptr[x + 1]; ++p)
                if (colidx[p] != x && !S.covered[p]) *e++ = (uint32_t)colidx[p];
        }
    });
    for (int half = 0; half < 2; ++half) {  // equal shares of the entries, and an item costs about as much as two of them
        const int64_t first = half ? ns : 0, last = half ? ns + m : ns;
        auto cost = [&](int64_t i) { return (int64_t)(h->sum_items[i].len & ~CBM_SUM_OWN) + 2; };
        int64_t total = 0, sum = 0, i = first;
        for (int64_t j = first; j < last; ++j) {
            total += cost(j);
            h->sum_longest[half] = std::max(h->sum_longest[half], cost(j) - 2);
        }
        for (int j = 0; j < CBM_XCD; ++j) {
            h->sum_begin[half][j] = i;
            while (i < last && (j == CBM_XCD - 1 || sum + cost(i) / 2 < total * (j + 1) / CBM_XCD)) sum += cost(i++);
            h->sum_count[half][j] = i - h->sum_begin[half][j];
        }
    }
    if (verbose)
        std::fprintf(stderr, "[cbm_build] shared sums: %ld sets of %ld columns, %ld entries in their rows (%ld before)\n", (long)ns, (long)S.set_cols.size(),
                     (long)(h->sum_entries.size() - S.set_cols.size()), (long)nnz);
}

}  // namespace

// Column-blocked CBM: the columns are cut into B equal ranges and the part of every row inside a range becomes a row
// of its own; the B m part-rows, stacked block after block (part-row b m + i = row i inside range b), are compressed
// as ONE matrix by the builder above -- its candidate search only ever pairs rows that share columns, so trees form
// inside ranges -- and a product is the sum of the B partial rows of every row.  The format lives in h->inner.
static cbm_status cbm_build_blocked(int64_t m, int64_t n, const int64_t* in_rowptr, const int32_t* in_colidx, cbm_handle* h) {
    auto t0 = std::chrono::steady_clock::now();
    const cbm_build_opts& o = h->opts;
    const int64_t B = o.column_blocks;
    if (o.flags & CBM_FLAG_TRANSPOSE) return CBM_ERR_INVALID_ARG;
    if (o.add_self_loops && m != n) return CBM_ERR_INVALID_ARG;
    if (B > 64 || B * m > (int64_t)CBM_ENTRY_INDEX_MASK || n > (int64_t)CBM_ENTRY_INDEX_MASK) return CBM_ERR_UNSUPPORTED;
    Builder P;  // borrowed for its CSR checks and the A v I step
    P.h = h;
    P.m = m;
    P.n = n;
    P.nthreads = o.num_threads > 0 ? o.num_threads : (int)std::max(1u, std::thread::hardware_concurrency());
    cbm_status st = P.validate(in_rowptr, in_colidx);
    if (st != CBM_OK) return st;
    P.rowptr = in_rowptr;
    P.colidx = in_colidx;
    if (o.add_self_loops) P.self_loops(in_rowptr, in_colidx);
    const int64_t nnz = P.rowptr[m];
    if (nnz >= (int64_t)UINT32_MAX) return CBM_ERR_UNSUPPORTED;
    h->m = m;
    h->n = n;
    h->blocks = (int32_t)B;
    h->square_self_loops = o.add_self_loops != 0;
    // the part-rows, block after block
    std::vector<int64_t> srp((size_t)(B * m) + 1, 0);
    std::vector<int32_t> sci((size_t)nnz);
    auto lo_of = [&](int64_t b) { return (int32_t)((b * n + B - 1) / B); };  // block b = columns [lo_of(b), lo_of(b + 1))
    parallel_chunks(P.nthreads, m, 4096, [&](int64_t r0, int64_t r1, int) {
        for (int64_t i = r0; i < r1; ++i) {
            const int32_t* row = P.colidx + P.rowptr[i];
            const int32_t* end = P.colidx + P.rowptr[i + 1];
            for (int64_t b = 0; b < B; ++b) {
                const int32_t* lo = std::lower_bound(row, end, lo_of(b));
                const int32_t* hi = std::lower_bound(lo, end, lo_of(b + 1));
                srp[(size_t)(b * m + i) + 1] = hi - lo;
            }
        }
    });
    for (int64_t v = 0; v < B * m; ++v) srp[v + 1] += srp[v];
    parallel_chunks(P.nthreads, m, 4096, [&](int64_t r0, int64_t r1, int) {
        for (int64_t i = r0; i < r1; ++i) {
            const int32_t* row = P.colidx + P.rowptr[i];
            const int32_t* end = P.colidx + P.rowptr[i + 1];
            for (int64_t b = 0; b < B; ++b) {
                const int32_t* lo = std::lower_bound(row, end, lo_of(b));
                const int32_t* hi = std::lower_bound(lo, end, lo_of(b + 1));
                std::copy(lo, hi, sci.begin() + srp[(size_t)(b * m + i)]);
            }
        }
    });
    cbm_handle* in = new cbm_handle();
    h->inner = in;  // owned from here on: freed with the outer handle, also on failure
    in->opts = o;
    in->opts.column_blocks = 0;
    in->opts.add_self_loops = 0;
    st = cbm_build_host(B * m, n, srp.data(), sci.data(), in);
    if (st != CBM_OK) return st;
    // weights by index: an entry's index is a column (< n) or a part-row b m + i, whose weights are those of row i
    std::vector<float> dinv, rinv(m);
    for (int64_t i = 0; i < m; ++i) {
        const int64_t len = P.rowptr[i + 1] - P.rowptr[i];
        rinv[i] = len > 0 ? (float)(1.0 / (double)len) : 0.0f;
    }
    in->rinv.resize((size_t)(B * m));
    for (int64_t v = 0; v < B * m; ++v) in->rinv[v] = rinv[v % m];
    if (h->square_self_loops) {  // D = row sums of A v I
        in->square_self_loops = true;
        in->dinv.resize((size_t)(B * m));
        for (int64_t v = 0; v < B * m; ++v) {
            const int64_t i = v % m;
            in->dinv[v] = (float)(1.0 / std::sqrt((double)(P.rowptr[i + 1] - P.rowptr[i])));
        }
        in->stats.bytes_cbm += 4 * (int64_t)in->dinv.size();
    }
    h->rownnz.resize(m);
    for (int64_t i = 0; i < m; ++i) h->rownnz[i] = (int32_t)(P.rowptr[i + 1] - P.rowptr[i]);
    cbm_stats_t& s = h->stats;
    s = in->stats;
    s.m = m;
    s.n = n;
    s.nnz = nnz;
    s.scalar_ops += (B - 1) * m;  // the additions of the block sum
    s.bytes_csr = 8 * (m + 1) + 4 * in_rowptr[m];
    s.add_self_loops = o.add_self_loops != 0;
    s.column_blocks = (int32_t)B;
    s.build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return CBM_OK;
}

cbm_status cbm_build_host(int64_t m, int64_t n, const int64_t* in_rowptr, const int32_t* in_colidx, cbm_handle* h) {
    auto t0 = std::chrono::steady_clock::now();
    const cbm_build_opts& o = h->opts;
    if (o.alpha < 0 || o.max_depth < -1 || o.hub_cap < -1 || o.max_candidates < -1 || o.seed_roots < -1 ||
        o.num_threads < 0 || o.column_blocks < 0)
        return CBM_ERR_INVALID_ARG;
    if (o.column_blocks > 1) return cbm_build_blocked(m, n, in_rowptr, in_colidx, h);
    if (m > (int64_t)CBM_ENTRY_INDEX_MASK || n > (int64_t)CBM_ENTRY_INDEX_MASK) return CBM_ERR_UNSUPPORTED;
    if (o.add_self_loops && m != n) return CBM_ERR_INVALID_ARG;
    Builder B;
    B.h = h;
    B.m = m;
    B.n = n;
    B.nthreads = o.num_threads > 0 ? o.num_threads : (int)std::max(1u, std::thread::hardware_concurrency());
    B.alpha = o.alpha;
    B.min_saving = std::max(o.alpha, 1);  // strict gain at alpha = 0: draws go to the virtual edge
    B.auto_depth = o.max_depth == 0;
    B.max_depth = o.max_depth == 0 ? kDefaultMaxDepth : o.max_depth;  // -1 = unlimited
    B.hub_cap = o.hub_cap == 0 ? kDefaultHubCap : o.hub_cap;
    B.max_cand = o.max_candidates == 0 ? kDefaultMaxCand : o.max_candidates;
    B.verbose = std::getenv("CBM_VERBOSE") != nullptr;
    B.last = t0;
    // segments and unsplit rows both have to fit the 24-bit entry count of a work item
    B.split_len = env_clamped("CBM_SPLIT_LEN", kSplitLenDefault, 1, 1 << 20);
    B.split_min = env_clamped("CBM_SPLIT_MIN", kSplitMinDefault, 1, 1 << 20);
    h->m = m;
    h->n = n;
    h->eff_alpha = B.alpha;
    h->eff_max_depth = B.max_depth;
    h->eff_hub_cap = B.hub_cap;
    h->eff_max_cand = B.max_cand;
    h->square_self_loops = o.add_self_loops != 0;

    cbm_status st = B.validate(in_rowptr, in_colidx);
    if (st != CBM_OK) return st;
    B.rowptr = in_rowptr;
    B.colidx = in_colidx;
    if (o.add_self_loops) B.self_loops(in_rowptr, in_colidx);
    B.nnz = B.rowptr[m];
    if (B.nnz >= (int64_t)UINT32_MAX) return CBM_ERR_UNSUPPORTED;
    if (h->square_self_loops) {  // D^-1/2 of A v I: D is the row sums of the matrix as given, transposed or not
        h->dinv.resize(m);
        for (int64_t i = 0; i < m; ++i) h->dinv[i] = (float)(1.0 / std::sqrt((double)(B.rowptr[i + 1] - B.rowptr[i])));
    }
    if (o.flags & CBM_FLAG_TRANSPOSE) {
        B.transpose_matrix();
        m = B.m;
        n = B.n;
        h->m = m;
        h->n = n;
    }
    h->rownnz.resize(m);
    for (int64_t i = 0; i < m; ++i) h->rownnz[i] = (int32_t)(B.rowptr[i + 1] - B.rowptr[i]);
    B.lap("validate + A v I");

    h->rinv.resize(m);  // 1/nnz per row: the mean aggregator's row weight
    for (int64_t i = 0; i < m; ++i) h->rinv[i] = B.rlen(i) > 0 ? (float)(1.0 / (double)B.rlen(i)) : 0.0f;

    // ---- tree, paths, rounds ---------------------------------------------------------------------
    // The tree is cut into vertical paths.  A path is ONE work item: its running sum stays in
    // registers from row to row (c_x = c_y + deltas, Eq. (5)), so only the head of a path waits for
    // another work item, the one that produced its parent's row.  Paths whose head hangs off a row of
    // a round-r path run in round r + 1, and every round is one kernel launch.  Longer paths mean fewer
    // rounds but a longer chain of dependent batches inside one work item.  The number of seeded roots
    // and the path length cap are the pair the cost model likes best; with the default depth option the
    // model may also find that no tree pays for its extra launches (small graphs): then every row is
    // stored in full.  A depth cap of 1 means exactly that and needs no candidate search.
    int32_t nrounds = 0;
    double chosen_us = 1e300;  // modelled time of the plan that is kept
    int64_t best_len = kPathChoices[0], best_split = B.split_min;
    // rows longer than the split threshold are cut into per-XCD segments: worth a launch or two of their own on
    // graphs with many long rows, a loss where only a handful exist
    std::vector<int64_t> split_choices = {kSplitMinDefault, kSplitLenDefault};
    if (std::getenv("CBM_SPLIT_MIN")) split_choices = {B.split_min};
    bool tree = B.max_depth != 1 && m > 1;
    B.locality = m == n && !std::getenv("CBM_NO_LOCALITY");
    B.bundle = tree && n <= (int64_t)CBM_BUNDLE_INDEX_MASK && !std::getenv("CBM_NO_BUNDLE");
    B.bundle_min = env_clamped("CBM_BUNDLE_MIN", kBundleMinEntries, 1, 1 << 20);
    B.bundle_min_items = env_clamped("CBM_BUNDLE_MIN_ITEMS", kBundleMinItems, 1, 1 << 30);
    B.locality_min = env_clamped("CBM_LOCALITY_MIN", kLocalityMinEntries, 1, 1 << 20);
    const bool exact_tree = (o.flags & CBM_FLAG_EXACT_TREE) != 0;
    if (o.flags & CBM_FLAG_DEVICE_BUILD) {  // asked for: an error if it cannot be had
        if ((o.flags & (CBM_FLAG_HOST_ONLY | CBM_FLAG_HOST_SEARCH)) || B.max_cand < 1 || B.max_cand > 16) return CBM_ERR_INVALID_ARG;
        B.device_candidates = true;
    } else if (!(o.flags & (CBM_FLAG_HOST_ONLY | CBM_FLAG_HOST_SEARCH)) && m >= kDeviceSearchMinRows && B.max_cand >= 1 &&
               B.max_cand <= 16) {
        // not asked for: a handle that is going to a GPU anyway searches there too when the matrix is large, and
        // falls back to the host threads if the GPU cannot take it (memory); both give the same candidates
        B.device_candidates = true;
        B.device_optional = true;
    }
    if (tree && exact_tree) {
        if ((st = B.find_candidates()) != CBM_OK) return st;
        B.arborescence();
        B.tree_index();
        double best_us = 1e300;
        for (int64_t cap : kPathChoices) {
            int32_t nr = 0;
            const double us = B.plan(cap, &nr);
            if (us < best_us) {
                best_us = us;
                best_len = cap;
            }
        }
        B.lap("exact arborescence");
    } else if (tree) {
        B.sample_first = B.auto_depth && m >= kSampleMinRows && !std::getenv("CBM_NO_SAMPLE");
        if ((st = B.find_candidates()) != CBM_OK) return st;
    }
    if (tree && !exact_tree && B.skip_tree) tree = false;
    if (tree && !exact_tree) {
        const int64_t forced_len = env_clamped("CBM_PATH_MAX", 0, 0, 1 << 20);
        const int64_t forced_seeds = o.seed_roots > 0 ? o.seed_roots : o.seed_roots < 0 ? 0 : env_or("CBM_SEED_ROOTS", -1);
        double best_us = 1e300;
        // the trees grown from 0, m/128, m/32, m/8 seeded roots, side by side (or the one the caller asked for)
        struct Grown {
            int64_t seeds;
            std::vector<int32_t> parent, level;
            std::vector<int64_t> dptr;
        };
        std::vector<Grown> grown;
        for (int64_t seeds : {(int64_t)0, m / 128, m / 32, m / 8}) {
            grown.push_back({forced_seeds >= 0 ? forced_seeds : seeds, {}, {}, {}});
            if (forced_seeds >= 0 || m < 1024) break;
        }
        auto grow = [&](size_t i) { B.prim(grown[i].seeds, grown[i].parent, grown[i].level, grown[i].dptr); };
        if (B.nthreads > 1)
            run_threads((int)grown.size(), [&](int i) { grow((size_t)i); });
        else
            for (size_t i = 0; i < grown.size(); ++i) grow(i);
        size_t best_tree = 0;
        for (size_t gi = 0; gi < grown.size(); ++gi) {
            const int64_t seeds = grown[gi].seeds;
            h->parent.swap(grown[gi].parent);
            h->level.swap(grown[gi].level);
            h->dptr.swap(grown[gi].dptr);
            for (int64_t split : split_choices) {
                B.split_min = split;
                B.tree_index();
                for (int64_t cap : kPathChoices) {
                    if (forced_len > 0) cap = forced_len;
                    int32_t nr = 0;
                    const double us = B.plan(cap, &nr);
                    if (B.verbose)
                        std::fprintf(stderr,
                                     "[cbm_build] seeds %7ld split above %3ld path cap %4ld: %3d rounds, %ld deltas, model %.1f us\n",
                                     (long)seeds, (long)split, (long)cap, nr, (long)h->dptr[m], us);
                    if (us < best_us) {
                        best_us = us;
                        best_len = cap;
                        best_split = split;
                        best_tree = gi;
                    }
                    if (forced_len > 0) break;
                }
            }
            h->parent.swap(grown[gi].parent);
            h->level.swap(grown[gi].level);
            h->dptr.swap(grown[gi].dptr);
        }
        B.kept_parent.swap(grown[best_tree].parent);  // the winner, for after the comparison with "no tree"
        B.kept_level.swap(grown[best_tree].level);
        B.kept_dptr.swap(grown[best_tree].dptr);
        grown.clear();
        if (B.auto_depth && forced_len <= 0) {
            B.all_roots();
            for (int64_t split : split_choices) {
                B.split_min = split;
                const double csr_us = B.csr_cost();
                if (B.verbose)
                    std::fprintf(stderr, "[cbm_build] all rows in full, split above %ld: model %.1f us (best tree: %.1f us)\n",
                                 (long)split, csr_us, best_us);
                if (csr_us <= best_us) {
                    best_us = csr_us;
                    best_split = split;
                    tree = false;
                }
            }
        }
        chosen_us = best_us;
        B.lap("tree + path model");
    } else if (!tree) {
        B.all_roots();
        double best_us = 1e300;
        for (int64_t split : split_choices) {
            B.split_min = split;
            const double us = B.csr_cost();
            if (us < best_us) {
                best_us = us;
                best_split = split;
            }
        }
        chosen_us = best_us;
    }
    const double product_us = chosen_us;
    B.split_min = best_split;
    if (tree && exact_tree) {
        // keep the arborescence as found
        if (B.bundle) {
            int32_t nr = 0;
            B.plan(best_len, &nr);
            B.choose_bundled_rounds(best_len, &nr);
        }
    } else if (tree) {
        h->parent.swap(B.kept_parent);
        h->level.swap(B.kept_level);
        h->dptr.swap(B.kept_dptr);
        B.tree_index();
        if (B.bundle) {  // before the last round is priced: the row limit of bundled rounds moves some rows one round down
            int32_t nr = 0;
            B.plan(best_len, &nr);
            B.choose_bundled_rounds(best_len, &nr);
        }
        while (B.auto_depth && B.prune_last_round(best_len)) {  // part of the automatic policy only
        }
    } else {
        B.all_roots();
    }
    std::vector<int64_t>().swap(B.optr);
    std::vector<int32_t>().swap(B.ochild);
    std::vector<int32_t>().swap(B.ow);
    if (!tree) B.bundle = false;  // every row stored in full: nothing to bundle
    B.delta_lists();
    B.tree_index();
    B.plan(best_len, &nrounds);
    if (tree && B.locality) B.locality_order();
    else if (!tree && B.locality && B.rows_share_by_index()) B.index_order();
    cbm_stats_t& s = h->stats;
    std::memset(&s, 0, sizeof(s));
    // (CBM_HUB_BLOCKS: 0 = never, 2 = whatever they save, on host-only handles too, 3 = as by default, on host-only handles too)
    const long want_hubs = env_clamped("CBM_HUB_BLOCKS", 1, 0, 3);
    if (!tree && B.auto_depth && !exact_tree && (want_hubs >= 2 || (want_hubs == 1 && !(o.flags & CBM_FLAG_HOST_ONLY)))) B.hub_blocks(want_hubs == 2);
    st = B.emit(nrounds);
    // cbm_spmm_noalloc takes a product's columns in as many goes as its scratch needs, at least four columns at a time
    const int64_t all_slots = (int64_t)(cbm_static_scratch_bytes() / 16);
    const int64_t most_slots = env_clamped("CBM_MOST_SLOTS", all_slots, 0, all_slots);
    if (st == CBM_OK && h->hub_blocks && h->num_slots > most_slots && h->noalloc_slots <= most_slots) {
        B.rest_of.clear();
        h->hub_blocks = false;
        std::vector<CbmBlock>().swap(h->row_blocks);
        std::vector<uint32_t>().swap(h->block_rows);
        std::vector<uint32_t>().swap(h->block_cols);
        std::vector<uint32_t>().swap(h->block_masks);
        st = B.emit(nrounds);
    }
    if (st != CBM_OK) return st;
    B.lap("paths + work lists");
    // ---- row blocks ------------------------------------------------------------------------------
    // Part of the automatic policy: the tree and its counters are what they are, but where one walk over the columns of 128
    // alike rows on the matrix cores is modelled cheaper than the rounds of paths, the products run that way.
    // (CBM_ROW_BLOCKS: 0 = never, 1 = whenever the matrix is square and the policy automatic, 2 = as by default, on host-only handles too.)
    const long want_blocks = env_clamped("CBM_ROW_BLOCKS", -1, -1, 2);
    double blocks_us = 0, sums_us = 0;
    if (B.auto_depth && !exact_tree && !h->hub_blocks && want_blocks != 0 && m == n && m > 0 && (want_blocks >= 1 || !(o.flags & CBM_FLAG_HOST_ONLY))) {
        const double limit = kBlockMargin * product_us;
        const int32_t most = *std::max_element(h->rownnz.begin(), h->rownnz.end());  // a block needs its longest row's columns
        const bool worth = want_blocks == 1 || (m >= kBlockMinRows && B.nnz >= kBlockMinDegree * m && most <= 64 * kBlockLongest &&
                                                B.sampled_row_block_cost() < limit);
        if (worth) {
            B.row_blocks();
            double longest = 0;
            for (const CbmBlock& b : h->row_blocks) longest = std::max(longest, (double)b.ngroups);
            const double us = B.row_block_cost((double)h->block_cols.size() / 64.0, longest);
            blocks_us = us;
            if (B.verbose) std::fprintf(stderr, "[cbm_build] row blocks: model %.1f us (paths: %.1f us)\n", us, product_us);
            if (want_blocks != 1 && us >= limit) {
                std::vector<CbmBlock>().swap(h->row_blocks);
                std::vector<uint32_t>().swap(h->block_rows);
                std::vector<uint32_t>().swap(h->block_cols);
                std::vector<uint32_t>().swap(h->block_masks);
            }
        }
        B.lap("row blocks");
    }

    // ---- shared sums -----------------------------------------------------------------------------
    // Part of the automatic policy too: column sets that many rows hold in full (the cliques of a collaboration network) are summed
    // once and the rows made of the sums.  The paths (or row blocks) stay, for handles that cannot be given the memory.
    // (CBM_SHARED_SUMS: 0 = never, 1 = whenever there are any, 2 = as by default, on host-only handles too.)
    const long want_sums = env_clamped("CBM_SHARED_SUMS", -1, -1, 2);
    if (B.verbose && h->hub_blocks) std::fprintf(stderr, "[cbm_build] shared sums: products do without\n");
    if (B.auto_depth && !exact_tree && !h->hub_blocks && want_sums != 0 && m == n && m > 0 && (want_sums == 1 || want_blocks != 1) &&
        (want_sums >= 1 || !(o.flags & CBM_FLAG_HOST_ONLY))) {
        const double limit = std::min(kSumMargin * product_us, h->row_blocks.empty() ? 1e300 : kSumBlockMargin * blocks_us);
        std::vector<uint8_t> holds_own((size_t)m, 1);
        if (!h->square_self_loops)
            parallel_chunks(B.nthreads, m, 4096, [&](int64_t x0, int64_t x1, int) {
                for (int64_t x = x0; x < x1; ++x) holds_own[x] = std::binary_search(B.row(x), B.row(x) + B.rlen(x), (int32_t)x);
            });
        auto parallel = [&](int64_t total, auto&& fn) { parallel_chunks(B.nthreads, total, 1, [&](int64_t b, int64_t e, int) { fn(b, e); }); };
        auto promising = [&] {  // the plan takes a while to make: the least it could cost, and what a few rows say of it, come first
            if (m < kSumMinRows || B.shared_sums_cost(0, 0, 0) >= limit) return false;
            SharedSumFinder finder(m, B.rowptr, B.colidx, holds_own.data());
            const double gathers = finder.sample(kSumSample, parallel) * (double)B.nnz;
            if (B.shared_sums_cost(gathers, 0, 0) >= limit) return false;
            std::vector<int32_t> longest;  // those long enough to matter, which is not many of them
            for (int64_t x = 0; x < m; ++x)
                if (B.shared_sums_cost(0, 0, (double)B.rlen(x)) >= limit) longest.push_back((int32_t)x);
            const size_t most = std::min(longest.size(), kSumLongRows);
            std::partial_sort(longest.begin(), longest.begin() + most, longest.end(), [&](int32_t x, int32_t y) { return B.rlen(x) != B.rlen(y) ? B.rlen(x) > B.rlen(y) : x < y; });
            longest.resize(most);
            return B.shared_sums_cost(gathers, 0, (double)finder.longest_left(longest, parallel)) < limit;
        };
        const bool worth = want_sums == 1 || promising();
        if (worth) {
            B.shared_sums(holds_own);
            double gathers = (double)h->sum_entries.size();
            for (const CbmSumItem& it : h->sum_items) gathers += it.own != 0;
            const double us = B.shared_sums_cost(gathers, (double)h->num_sums, (double)(h->sum_longest[0] + h->sum_longest[1]));
            sums_us = us;
            if (B.verbose) std::fprintf(stderr, "[cbm_build] shared sums: model %.1f us (paths: %.1f us)\n", us, product_us);
            if (want_sums != 1 && us >= limit) {
                h->num_sums = 0;
                std::vector<CbmSumItem>().swap(h->sum_items);
                std::vector<uint32_t>().swap(h->sum_entries);
            }
        }
        if (B.verbose) std::fprintf(stderr, "[cbm_build] shared sums: products %s\n", h->num_sums > 0 ? "take them" : "do without");
        B.lap("shared sums");
    }

    s.nnz = B.nnz;
    // (the narrowest product is where the rows as they stand do best)
    if (B.auto_depth && !exact_tree && h->flat_rich && h->num_slots == 0 && want_blocks != 1 && want_sums != 1 && (h->in_row_blocks() || h->num_sums > 0)) {
        const double us = h->num_sums > 0 ? kFlatSumMargin * sums_us : kFlatBlockMargin * blocks_us;
        if (cbm_flat_waves(h, 8, 32) <= CBM_FLAT_MOST_WAVES && cbm_flat_us(h, 32, 8) < us) h->other_us = us;
    }

    // ---- counters (Properties 1 and 2) -----------------------------------------------------------
    s.m = m;
    s.n = n;
    int32_t depth = 0;
    for (int64_t x = 0; x < m; ++x) {
        depth = std::max(depth, h->level[x]);
        s.num_delta_plus += h->nplus[x];
        s.num_delta_minus += h->nminus[x];
        if (h->parent[x] < 0) {
            ++s.num_roots;
            s.scalar_ops += B.rlen(x);
        } else {
            s.scalar_ops += 1 + h->nplus[x] + h->nminus[x];
        }
    }
    s.num_internal = (int64_t)h->internal_rows.size();
    s.num_tasks = (int64_t)h->tasks.size();
    s.bytes_csr = 8 * (m + 1) + 4 * in_rowptr[m];
    // (a host-only handle counts its work lists; row blocks are all that a device handle with them uploads)
    const int64_t block_bytes = 4 * (int64_t)(h->block_rows.size() + h->block_cols.size() + h->block_masks.size()) +
                                (int64_t)sizeof(CbmBlock) * (int64_t)h->row_blocks.size();
    const bool blocks_only = h->in_row_blocks() && h->other_us == 0 && !(o.flags & CBM_FLAG_HOST_ONLY);
    s.bytes_cbm = 4 * (int64_t)h->dinv.size() + (blocks_only || h->hub_blocks ? block_bytes : 0);
    if (!blocks_only)
        s.bytes_cbm += 4 * (int64_t)(h->stream.size() + h->internal_rows.size()) + (int64_t)sizeof(CbmTask) * (int64_t)(h->tasks.size() + h->comb.size());
    if (!(o.flags & CBM_FLAG_HOST_ONLY)) s.bytes_cbm += 4 * (int64_t)h->sum_entries.size() + (int64_t)sizeof(CbmSumItem) * (int64_t)h->sum_items.size();
    s.depth = depth;
    s.rounds = nrounds;
    s.alpha = B.alpha;
    s.add_self_loops = o.add_self_loops != 0;
    s.column_blocks = 1;
    for (const CbmLevel& L : h->levels) s.bundled_rounds += L.bundled;
    s.build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return CBM_OK;
}

cbm_status cbm_decompress_host(const cbm_handle* h, int64_t* rowptr, int32_t* colidx) {
    if (h->blocks > 1) {  // rebuild the part-rows from the inner format, then put every row's parts back together
        const cbm_handle* in = h->inner;
        const int64_t m = h->m, B = h->blocks;
        std::vector<int64_t> srp((size_t)(B * m) + 1);
        std::vector<int32_t> sci((size_t)std::max<int64_t>(1, in->stats.nnz));
        const cbm_status st = cbm_decompress_host(in, srp.data(), sci.data());
        if (st != CBM_OK) return st;
        rowptr[0] = 0;
        for (int64_t i = 0; i < m; ++i) {
            int32_t* out = colidx + rowptr[i];
            for (int64_t b = 0; b < B; ++b)  // ranges ascend, so the parts in block order are the sorted row
                out = std::copy(sci.begin() + srp[(size_t)(b * m + i)], sci.begin() + srp[(size_t)(b * m + i) + 1], out);
            rowptr[i + 1] = out - colidx;
        }
        return CBM_OK;
    }
    const int64_t m = h->m;
    rowptr[0] = 0;
    for (int64_t x = 0; x < m; ++x) rowptr[x + 1] = rowptr[x] + h->rownnz[x];
    // parents before children: visit rows by level; a row is rebuilt from its parent's rebuilt
    // list and its own two delta lists only (Eq. (2))
    std::vector<int32_t> order(m);
    for (int64_t x = 0; x < m; ++x) order[x] = (int32_t)x;
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return h->level[a] < h->level[b]; });
    for (int32_t x : order) {
        const uint32_t* plus = h->dcol.data() + h->dptr[x];
        const uint32_t* pe = plus + h->nplus[x];
        const uint32_t* minus = pe;
        const uint32_t* me = minus + h->nminus[x];
        int32_t* out = colidx + rowptr[x];
        int32_t* oe = colidx + rowptr[x + 1];
        int32_t y = h->parent[x];
        const int32_t* a = y >= 0 ? colidx + rowptr[y] : nullptr;
        const int32_t* ae = y >= 0 ? colidx + rowptr[y + 1] : nullptr;
        // (a_y \ Delta-) merged with Delta+
        while (a != ae || plus != pe) {
            if (a != ae && minus != me && (uint32_t)*a == (*minus & ~CBM_DELTA_MINUS)) {
                ++a;
                ++minus;
                continue;
            }
            int32_t v;
            if (plus == pe || (a != ae && (uint32_t)*a < *plus))
                v = *a++;
            else
                v = (int32_t)*plus++;
            if (out == oe) return CBM_ERR_STATE;
            *out++ = v;
        }
        if (out != oe || minus != me) return CBM_ERR_STATE;
    }
    return CBM_OK;
}

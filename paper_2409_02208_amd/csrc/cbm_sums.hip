// Products through shared sums: column sets that many rows hold in full are summed once, rows are made of those sums.
//
// Two launches a product (or for as many columns at a time as there is memory for sums).  The first writes the sum of every set's rows of X (times their column
// weights) to scratch memory; the second makes each row of Y from its sets' sums, the columns no set brings and, where the sets hold the
// row's own column more or less often than the row does, its own row of X as often as that takes.  Both are gathers like those of the
// paths, bound by the memory behind L2; what they gain is that there are fewer of them (collaboration recipe, 235,868 nodes: 1.8 million
// rows read or written a product instead of 5.0 million, and no round waits for another but the second for the first: k = 128 334 -> 136 us,
// 48 for the sets at 6.1 TB/s behind L2 and 84 for the rows at 6.5; GIN, k = 64 191 -> 73; 20,000 nodes, k = 64 37 -> 18).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <functional>
#include <thread>

#include "cbm_internal.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// The four columns of a lane in the block's 4 LANES.  RAGGED = false: 4 sl .. 4 sl + 3, one 128-bit access; true: sl, sl + LANES, ..., 32-bit
// accesses.
// Lanes beyond the last column load one that exists and store nothing.
template <bool RAGGED, int LANES>
struct Columns {
    uint32_t at[RAGGED ? 4 : 1];
    bool on[RAGGED ? 4 : 1];
    __device__ __forceinline__ Columns(int sl, int k) {
        const int first = blockIdx.y * (4 * LANES);
#pragma unroll
        for (int c = 0; c < (RAGGED ? 4 : 1); ++c) {
            const int col = first + (RAGGED ? sl + c * LANES : 4 * sl);
            on[c] = col < k;
            at[c] = on[c] ? (uint32_t)col : 0u;
        }
    }
    __device__ __forceinline__ f4 load(const float* row) const {
        if constexpr (!RAGGED) return *reinterpret_cast<const f4*>(row + at[0]);
        f4 r;
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = row[at[RAGGED ? c : 0]];
        return r;
    }
    template <bool KEEP>  // rows of Y are not read again by the launch, sums are by the next one
    __device__ __forceinline__ void store(float* row, f4 v) const {
        if constexpr (!RAGGED) {
            if (!on[0]) return;
            if (KEEP) *reinterpret_cast<f4*>(row + at[0]) = v;
            else __builtin_nontemporal_store(v, reinterpret_cast<f4*>(row + at[0]));
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (on[c]) {
                    if (KEEP) row[at[c]] = v[c];
                    else __builtin_nontemporal_store(v[c], row + at[c]);
                }
        }
    }
};

struct SumMap {
    uint32_t begin[CBM_XCD], count[CBM_XCD];
};

// acc += sum over the entries of (weight times) the row of X, or the set's sum, that each names.  Entries come LANES at a time, the
// next ones while these are worked on, and are broadcast inside the group; U rows are in flight at a time.
template <bool RAGGED, int LANES, bool WEIGHTED, bool SETS, int U>
__device__ __forceinline__ void walk(f4& acc, const uint32_t* __restrict__ es, const float* __restrict__ ws, uint32_t len, int sl, const float* X,
                                     uint32_t ldx, const float* S, uint32_t lds, const Columns<RAGGED, LANES>& cols) {
    uint32_t e = (uint32_t)sl < len ? __builtin_nontemporal_load(es + sl) : 0u;
    float w = WEIGHTED && (uint32_t)sl < len ? __builtin_nontemporal_load(ws + sl) : 0.0f;
    for (uint32_t at = 0; at < len; at += LANES) {
        uint32_t e1 = 0u;
        float w1 = 0.0f;
        if (at + LANES + sl < len) {
            e1 = __builtin_nontemporal_load(es + at + LANES + sl);
            if (WEIGHTED) w1 = __builtin_nontemporal_load(ws + at + LANES + sl);
        }
        const int n = (int)min((uint32_t)LANES, len - at);
        for (int b = 0; b < n; b += U) {
            f4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t eu = (uint32_t)__shfl((int)e, b + u, LANES);
                x[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                if (b + u < n) {
                    const bool sum = SETS && (eu & CBM_SUM_BIT);
                    x[u] = cols.load((sum ? S : X) + (uint64_t)(eu & ~CBM_SUM_BIT) * (sum ? lds : ldx));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (WEIGHTED) {
                    const float wu = __shfl(w, b + u, LANES);  // (0 past the last entry)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = fmaf(wu, x[u][c], acc[c]);
                } else {
                    acc += x[u];
                }
            }
        }
        e = e1;
        w = w1;
    }
}

template <int LANES>
__device__ __forceinline__ int64_t item_of(const SumMap& map) {  // workgroup b runs on XCD b mod 8 and takes its items from that XCD's run
    constexpr int G = 64 / LANES;
    const int xcd = blockIdx.x % CBM_XCD;
    const uint32_t i = ((uint32_t)(blockIdx.x / CBM_XCD) * 4 + (threadIdx.x >> 6)) * G + (threadIdx.x & 63) / LANES;
    return i < map.count[xcd] ? (int64_t)map.begin[xcd] + i : -1;
}

template <bool RAGGED, int LANES, bool WEIGHTED, int U>
__global__ __launch_bounds__(256, 4) void cbm_sum_sets_kernel(const CbmSumItem* __restrict__ items, const SumMap map,
                                                              const uint32_t* __restrict__ entries, const float* __restrict__ ws,
                                                              const float* __restrict__ X, uint32_t ldx, float* __restrict__ S, uint32_t lds, int k) {
    const int64_t t = item_of<LANES>(map);
    if (t < 0) return;
    const uint32_t start = items[t].start, len = items[t].len;
    const int sl = threadIdx.x % LANES;
    const Columns<RAGGED, LANES> cols(sl, k);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    walk<RAGGED, LANES, WEIGHTED, false, U>(acc, entries + start, WEIGHTED ? ws + start : nullptr, len, sl, X, ldx, nullptr, 0, cols);
    cols.template store<true>(S + (uint64_t)t * lds, acc);
}

// MODE as for the paths: 0 M X, 1 D^-1/2 M D^-1/2 X, 2 = 1 then max(., 0), 3 D^-1 M X, 4 M X + s X.
template <bool RAGGED, int LANES, int MODE, int U>
__global__ __launch_bounds__(256, 4) void cbm_sum_rows_kernel(const CbmSumItem* __restrict__ items, const SumMap map,
                                                              const uint32_t* __restrict__ entries, const float* __restrict__ ws,
                                                              const float* __restrict__ X, uint32_t ldx, const float* __restrict__ S, uint32_t lds,
                                                              float* __restrict__ Y, uint32_t ldy, const float* __restrict__ rw, float self_w, int k) {
    constexpr bool WEIGHTED = MODE == 1 || MODE == 2;
    const int64_t t = item_of<LANES>(map);
    if (t < 0) return;
    const CbmSumItem it = items[t];
    const uint32_t len = it.len & ~CBM_SUM_OWN;
    const int sl = threadIdx.x % LANES;
    const Columns<RAGGED, LANES> cols(sl, k);
    const float w = MODE == 0 || MODE == 4 ? 1.0f : rw[it.row];
    const float* mine = X + (uint64_t)(uint32_t)it.row * ldx;
    const bool add_own = MODE == 4 || it.own != 0;
    f4 own = {0.0f, 0.0f, 0.0f, 0.0f};
    if (add_own) own = cols.load(mine);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    walk<RAGGED, LANES, WEIGHTED, true, U>(acc, entries + it.start, WEIGHTED ? ws + it.start : nullptr, len, sl, X, ldx, S, lds, cols);
    const float times = ((float)it.own + (MODE == 4 ? self_w : 0.0f)) * (WEIGHTED ? w : 1.0f);
    if (add_own)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(times, own[c], acc[c]);
    if (it.own < 0) {
        // The row's own column was summed more often than the row holds it and taken off again: right for finite sums only (an infinity
        // less itself is NaN).  Where a sum is not finite the row is put together from its sets' columns, each once.
        bool bad = false;
#pragma unroll
        for (int c = 0; c < 4; ++c) bad = bad || !(fabsf(acc[c]) < INFINITY);
        const uint64_t group = (LANES == 64 ? ~0ull : ((1ull << LANES) - 1)) << ((threadIdx.x & 63) / LANES * LANES);
        if (__ballot(bad) & group) {
            f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
            auto add = [&](uint32_t entry, uint32_t place) {
                const f4 x = cols.load(X + (uint64_t)entry * ldx);
                const float v = WEIGHTED ? ws[place] : 1.0f;
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[c] = fmaf(v, x[c], sum[c]);
            };
            for (uint32_t i = it.start; i < it.start + len; ++i) {
                const uint32_t e = entries[i];
                if (e & CBM_SUM_BIT) {
                    const CbmSumItem set = items[e & ~CBM_SUM_BIT];
                    for (uint32_t j = set.start; j < set.start + set.len; ++j)
                        if (entries[j] != (uint32_t)it.row) add(entries[j], j);
                } else {
                    add(e, i);
                }
            }
            const float once = ((it.len & CBM_SUM_OWN ? 1.0f : 0.0f) + (MODE == 4 ? self_w : 0.0f)) * (WEIGHTED ? w : 1.0f);
            const f4 x = cols.load(mine);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (MODE == 4 || (it.len & CBM_SUM_OWN)) sum[c] = fmaf(once, x[c], sum[c]);
                if (!(fabsf(acc[c]) < INFINITY)) acc[c] = sum[c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (MODE >= 1 && MODE <= 3) acc[c] *= w;
        if (MODE == 2) acc[c] = fmaxf(acc[c], 0.0f);
    }
    cols.template store<false>(Y + (uint64_t)(uint32_t)it.row * ldy, acc);
}

struct Args {
    const cbm_handle* h;
    const float* X;
    uint32_t ldx;
    float* S;
    uint32_t lds;
    float* Y;
    uint32_t ldy;
    const float* rw;
    float self_w;
    int k;
    hipStream_t stream;
};

template <bool RAGGED, int LANES, int MODE>
void launch(const Args& a, bool rows) {
    constexpr int G = 64 / LANES;
    constexpr int U = 8;  // 4 waves a SIMD; 4 rows at 8 waves: 30,000 nodes, k = 64 26 us instead of 22, 235,868 nodes the same; 2 rows 31
    SumMap map;
    uint32_t most = 0;
    for (int j = 0; j < CBM_XCD; ++j) {
        map.begin[j] = (uint32_t)a.h->sum_begin[rows][j];
        map.count[j] = (uint32_t)a.h->sum_count[rows][j];
        most = std::max(most, map.count[j]);
    }
    const dim3 grid(CBM_XCD * ((most + 4 * G - 1) / (4 * G)), (a.k + 4 * LANES - 1) / (4 * LANES));
    if (rows)
        hipLaunchKernelGGL((cbm_sum_rows_kernel<RAGGED, LANES, MODE, U>), grid, dim3(256), 0, a.stream, a.h->d_sum_items, map, a.h->d_sum_entries,
                           a.h->d_sum_w, a.X, a.ldx, a.S, a.lds, a.Y, a.ldy, a.rw, a.self_w, a.k);
    else
        hipLaunchKernelGGL((cbm_sum_sets_kernel<RAGGED, LANES, MODE == 1, U>), grid, dim3(256), 0, a.stream, a.h->d_sum_items, map, a.h->d_sum_entries,
                           a.h->d_sum_w, a.X, a.ldx, a.S, a.lds, a.k);
}
template <bool RAGGED, int LANES>
void launch_mode(const Args& a, int mode, bool rows) {
    if (!rows) return mode == 1 || mode == 2 ? launch<RAGGED, LANES, 1>(a, false) : launch<RAGGED, LANES, 0>(a, false);
    switch (mode) {
        case 0: return launch<RAGGED, LANES, 0>(a, true);
        case 1: return launch<RAGGED, LANES, 1>(a, true);
        case 2: return launch<RAGGED, LANES, 2>(a, true);
        case 3: return launch<RAGGED, LANES, 3>(a, true);
        default: return launch<RAGGED, LANES, 4>(a, true);
    }
}
template <bool RAGGED>
void launch_lanes(const Args& a, int mode, bool rows) {
    if (a.k <= 32) launch_mode<RAGGED, 8>(a, mode, rows);
    else if (a.k <= 64) launch_mode<RAGGED, 16>(a, mode, rows);
    else launch_mode<RAGGED, 32>(a, mode, rows);
}

constexpr size_t kMostScratch = 8;  // arrays of sums a handle keeps: one each for so many streams and captures
constexpr uint64_t kNobody = ~0ull;

}  // namespace

void cbm_launch_sum_chunk(const cbm_handle* h, bool rows, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy, int mode, const float* rw,
                          float self_w, float* S, int64_t lds, void* stream) {
    const Args a{h, X, (uint32_t)ldx, S, (uint32_t)lds, Y, (uint32_t)ldy, rw, self_w, (int)k, (hipStream_t)stream};
    const bool aligned = k % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && ((uintptr_t)X & 15) == 0 && ((uintptr_t)Y & 15) == 0;
    if (aligned) launch_lanes<false>(a, mode, rows);
    else launch_lanes<true>(a, mode, rows);
}

// The array for the sums of products on this stream; nullptr if there is none and none can be had.  Products of different streams may
// run at the same time, so each has its own; so has every capture, whose graph may be replayed beside anything.  The caller holds
// h->sum_mutex.  (The first is allocated with the handle; the allocation here is one that a capture under way does not mind.)
float* cbm_sum_scratch(const cbm_handle* h, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    CbmSumScratch key{(uint64_t)(uintptr_t)stream, 0, 0, nullptr};
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(stream, &status, &id) != hipSuccess) (void)hipGetLastError();
    else if (status == hipStreamCaptureStatusActive) key.capture = id + 1;
    if (stream == hipStreamPerThread) key.thread = (uint64_t)std::hash<std::thread::id>{}(std::this_thread::get_id());
    for (CbmSumScratch& s : h->sum_scratch)
        if (s.stream == key.stream && s.capture == key.capture && s.thread == key.thread) return s.sums;
    if (key.capture == 0)
        for (CbmSumScratch& s : h->sum_scratch)
            if (s.stream == kNobody) {
                key.sums = s.sums;
                s = key;
                return s.sums;
            }
    if (h->sum_scratch.size() >= kMostScratch) return nullptr;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    const hipError_t err = hipMalloc((void**)&key.sums, (size_t)h->num_sums * cbm_sum_columns(h->num_sums) * sizeof(float));
    if (err != hipSuccess) (void)hipGetLastError();
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (err != hipSuccess) return nullptr;
    h->sum_scratch.push_back(key);
    return key.sums;
}

cbm_status cbm_upload_sums(cbm_handle* h) {
    if (h->num_sums == 0) return CBM_OK;
    auto up = [&](auto** dptr, const void* src, size_t bytes) {
        if (hipMalloc((void**)dptr, bytes + 16) != hipSuccess) return false;
        return hipMemcpy(*dptr, src, bytes, hipMemcpyHostToDevice) == hipSuccess;
    };
    bool ok = up(&h->d_sum_items, h->sum_items.data(), h->sum_items.size() * sizeof(CbmSumItem)) &&
              up(&h->d_sum_entries, h->sum_entries.data(), h->sum_entries.size() * sizeof(uint32_t));
    if (ok && h->square_self_loops) {
        std::vector<float> w(h->sum_entries.size());
        for (size_t i = 0; i < w.size(); ++i) w[i] = h->sum_entries[i] & CBM_SUM_BIT ? 1.0f : h->dinv[h->sum_entries[i]];
        ok = up(&h->d_sum_w, w.data(), w.size() * sizeof(float));
    }
    CbmSumScratch first{kNobody, 0, 0, nullptr};
    if (ok) ok = hipMalloc((void**)&first.sums, (size_t)h->num_sums * cbm_sum_columns(h->num_sums) * sizeof(float)) == hipSuccess;
    if (!ok) {  // the paths do without
        (void)hipGetLastError();
        cbm_release_sums(h);
        h->num_sums = 0;
        return CBM_OK;
    }
    h->sum_scratch.reserve(kMostScratch);
    h->sum_scratch.push_back(first);
    return CBM_OK;
}

void cbm_release_sums(cbm_handle* h) {
    for (CbmSumScratch& s : h->sum_scratch) hipFree(s.sums);
    h->sum_scratch.clear();
    if (h->d_sum_items) hipFree(h->d_sum_items);
    if (h->d_sum_entries) hipFree(h->d_sum_entries);
    if (h->d_sum_w) hipFree(h->d_sum_w);
    h->d_sum_items = nullptr;
    h->d_sum_entries = nullptr;
    h->d_sum_w = nullptr;
}

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
#include <cmath>
#include <functional>
#include <thread>
#include <type_traits>

#include "cbm_internal.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// Rows that do not hold their own column (A without self-loops) are made of sums that do, and what rounding takes from these is relative to the
// row's own value, which the row's sum may be far below: own value 1e5, others near 1, 2e-4 of the sum; the type's lowest value, 0 instead of the sum.
// So the sets' launch also writes the exponent of each set's second largest value in every column (a byte beside four), and a row whose own value, as
// often as it is taken off, is more than kGuard times the largest of the others (or half as much: the exponent is all that is known of it) is put
// together without it.  What is let through is off by 32 x 2^-24 = 2e-6 of the row's terms for each addition that took as much from it: 5e-6 is the worst
// of 1,080 products of random matrices with values of random size.  Rows put together again are waited for, and
// sets have as few as four columns: with 16 the rows' launch takes 113 us instead of 83 on Gaussian features (235,868 nodes, k = 128), with 32 and 128
// the same (79 where no row is looked at); of features with every other value zero 92, with 128 86.  Both launches 132 us instead of 127; 30,000 nodes,
// k = 64 25 instead of 23.  (Rows that hold their own column are off by as much of a sum that it is part of.)
constexpr float kGuard = 32.0f;

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

// What a row's others amount to, for rows that do not hold their own column (kGuard above): in the sets' launch the largest and the second largest value
// of each column, in the rows' launch the largest of the single ones and of the sums without the row's own value and, as packed exponents, of the
// sets' second largest.  (Zero is zero: a value that is alone in its set is that set's sum.)
struct Sizes {
    f4 first = {0.0f, 0.0f, 0.0f, 0.0f}, second = {0.0f, 0.0f, 0.0f, 0.0f};
    ushort2v even = {0, 0}, odd = {0, 0};
    __device__ __forceinline__ void add_to_set(const f4& x) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            second[c] = __builtin_amdgcn_fmed3f(first[c], second[c], fabsf(x[c]));
            first[c] = fmaxf(first[c], fabsf(x[c]));
        }
    }
    // exponents of the second largest ones, a byte for each column: 0 for zero, 1 for all others below 2^-125
    __device__ __forceinline__ uint32_t packed() const {
        uint32_t r = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) r |= (second[c] != 0.0f ? max(__float_as_uint(second[c]) >> 23 & 255u, 1u) : 0u) << (8 * c);
        return r;
    }
    // `mine`: x is the sum of a set that holds the row's own value, of which only the others are asked for
    __device__ __forceinline__ void add_to_row(const f4& x, bool mine, uint32_t exponents) {
#pragma unroll
        for (int c = 0; c < 4; ++c) first[c] = fmaxf(first[c], fabsf(mine ? 0.0f : x[c]));
        even = __builtin_elementwise_max(even, __builtin_bit_cast(ushort2v, exponents & 0x00ff00ffu));
        odd = __builtin_elementwise_max(odd, __builtin_bit_cast(ushort2v, exponents >> 8 & 0x00ff00ffu));
    }
    __device__ __forceinline__ float others(int c) const {  // no more than the largest of them, no less than half of it
        const uint32_t exponent = c % 2 ? odd[c / 2] : even[c / 2];
        return fmaxf(first[c], __uint_as_float(exponent == 1 ? 1u : exponent << 23));
    }
};

struct Rows {  // where the rows of X and the sums are
    const float* X;
    uint32_t ldx;
    const float* S;
    uint32_t lds;
    const uint32_t* sizes;  // of the sets, this lane's
    uint32_t ld_sizes;
};

// acc += sum over the entries of (weight times) the row of X, or the set's sum, that each names.  Entries come LANES at a time, the
// next ones while these are worked on, and are broadcast inside the group; U rows are in flight at a time.  SIZED: the entries are a set's, whose
// sizes are wanted.  SKIP: entry `skip` is left out.
template <bool RAGGED, int LANES, bool WEIGHTED, bool SETS, bool SIZED, bool SKIP, int U>
__device__ __forceinline__ void walk(f4& acc, Sizes& sizes, const uint32_t* __restrict__ es, const float* __restrict__ ws, uint32_t len, int sl,
                                     const Rows& r, uint32_t skip, const Columns<RAGGED, LANES>& cols) {
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
                if (b + u < n && !(SKIP && eu == skip)) {
                    const bool sum = SETS && (eu & CBM_SUM_BIT);
                    x[u] = cols.load((sum ? r.S : r.X) + (uint64_t)(eu & ~CBM_SUM_BIT) * (sum ? r.lds : r.ldx));
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
                if (SIZED) sizes.add_to_set(x[u]);
            }
        }
        e = e1;
        w = w1;
    }
}

// The same for a row whose others' sizes are wanted too.  These cost a batch of entries twice its instructions where sets are among them (30,000 nodes,
// k = 64: 6 us more, waiting for the longest rows); sets come first, and batches without any do without.  The first `mine` hold the row's own column.
template <bool RAGGED, int LANES, int U0>
__device__ __forceinline__ void walk_sized(f4& acc, Sizes& sizes, const uint32_t* __restrict__ es, uint32_t len, int mine, int sl, const Rows& r,
                                           const Columns<RAGGED, LANES>& cols) {
    uint32_t e = (uint32_t)sl < len ? __builtin_nontemporal_load(es + sl) : 0u;
    for (uint32_t at = 0; at < len; at += LANES) {
        const uint32_t e1 = at + LANES + sl < len ? __builtin_nontemporal_load(es + at + LANES + sl) : 0u;
        const int n = (int)min((uint32_t)LANES, len - at);
        const uint64_t group = ((1ull << LANES) - 1) << ((threadIdx.x & 63) / LANES * LANES);
        const int sets = __popcll(__ballot(e & CBM_SUM_BIT) & group);
        auto batch = [&](int b, auto mixed) {
            constexpr bool MIXED = decltype(mixed)::value;
            constexpr int U = MIXED ? U0 / 2 : U0;
            f4 x[U];
            uint32_t size[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t eu = (uint32_t)__shfl((int)e, b + u, LANES);
                x[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                size[u] = 0u;
                if (b + u < n) {
                    const bool sum = MIXED && (eu & CBM_SUM_BIT);
                    x[u] = cols.load((sum ? r.S : r.X) + (uint64_t)(eu & ~CBM_SUM_BIT) * (sum ? r.lds : r.ldx));
                    if (MIXED) size[u] = r.sizes[(uint64_t)(sum ? eu & ~CBM_SUM_BIT : 0u) * r.ld_sizes];  // (a column: any set's)
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                acc += x[u];
                sizes.add_to_row(x[u], MIXED && (int)at + b + u < mine, b + u < sets ? size[u] : 0u);
            }
        };
        int b = 0;
        for (; b < sets; b += U0 / 2) batch(b, std::true_type{});
        for (; b < n; b += U0) batch(b, std::false_type{});
        e = e1;
    }
}

template <int LANES>
__device__ __forceinline__ int64_t item_of(const SumMap& map) {  // workgroup b runs on XCD b mod 8 and takes its items from that XCD's run
    constexpr int G = 64 / LANES;
    const int xcd = blockIdx.x % CBM_XCD;
    const uint32_t i = ((uint32_t)(blockIdx.x / CBM_XCD) * 4 + (threadIdx.x >> 6)) * G + (threadIdx.x & 63) / LANES;
    return i < map.count[xcd] ? (int64_t)map.begin[xcd] + i : -1;
}

template <bool RAGGED, int LANES, bool WEIGHTED, bool GUARD, int U>
__global__ __launch_bounds__(256, 4) void cbm_sum_sets_kernel(const CbmSumItem* __restrict__ items, const SumMap map,
                                                              const uint32_t* __restrict__ entries, const float* __restrict__ ws,
                                                              const float* __restrict__ X, uint32_t ldx, float* __restrict__ S, uint32_t lds,
                                                              uint32_t* __restrict__ set_sizes, uint32_t ld_sizes, int k) {
    const int64_t t = item_of<LANES>(map);
    if (t < 0) return;
    const uint32_t start = items[t].start, len = items[t].len;
    const int sl = threadIdx.x % LANES;
    const Columns<RAGGED, LANES> cols(sl, k);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    Sizes sizes;
    walk<RAGGED, LANES, WEIGHTED, false, GUARD, false, U>(acc, sizes, entries + start, WEIGHTED ? ws + start : nullptr, len, sl,
                                                          Rows{X, ldx, nullptr, 0, nullptr, 0}, 0, cols);
    cols.template store<true>(S + (uint64_t)t * lds, acc);
    if (GUARD) set_sizes[(uint64_t)t * ld_sizes + blockIdx.y * LANES + sl] = sizes.packed();
}

// The sum over a row's entries with its sets' columns one by one, its own left out of them.
template <bool RAGGED, int LANES, bool WEIGHTED>
__device__ __forceinline__ f4 apart(const CbmSumItem* __restrict__ items, const uint32_t* __restrict__ entries, const float* __restrict__ ws,
                                    uint32_t start, uint32_t len, uint32_t row, int sl, const Rows& r, const Columns<RAGGED, LANES>& cols) {
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    Sizes none;
    uint32_t i = start;
    for (; i < start + len; ++i) {  // sets come first
        const uint32_t e = entries[i];
        if (!(e & CBM_SUM_BIT)) break;
        const uint32_t first = items[e & ~CBM_SUM_BIT].start, n = items[e & ~CBM_SUM_BIT].len;
        walk<RAGGED, LANES, WEIGHTED, false, false, true, 4>(acc, none, entries + first, WEIGHTED ? ws + first : nullptr, n, sl, r, row, cols);
    }
    walk<RAGGED, LANES, WEIGHTED, false, false, false, 4>(acc, none, entries + i, WEIGHTED ? ws + i : nullptr, start + len - i, sl, r, 0, cols);
    return acc;
}

// The sum over a row's entries with its sets summed here and now, in the order in which the two launches do it: the same bits without the memory.
template <bool RAGGED, int LANES, bool WEIGHTED, bool GUARD, int U>
__device__ __forceinline__ void in_place(f4& acc, Sizes& sizes, const CbmSumItem* __restrict__ items, const uint32_t* __restrict__ entries,
                                         const float* __restrict__ ws, uint32_t start, uint32_t len, int mine, int sl, const Rows& r,
                                         const Columns<RAGGED, LANES>& cols) {
    uint32_t i = start;
    for (; i < start + len; ++i) {  // sets come first
        const uint32_t e = entries[i];
        if (!(e & CBM_SUM_BIT)) break;
        const uint32_t first = items[e & ~CBM_SUM_BIT].start, n = items[e & ~CBM_SUM_BIT].len;
        f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
        Sizes set;
        walk<RAGGED, LANES, WEIGHTED, false, GUARD, false, U>(sum, set, entries + first, WEIGHTED ? ws + first : nullptr, n, sl, r, 0, cols);
        acc += sum;
        if (GUARD) sizes.add_to_row(sum, (int)(i - start) < mine, set.packed());
    }
    if constexpr (GUARD) walk_sized<RAGGED, LANES, U>(acc, sizes, entries + i, start + len - i, 0, sl, r, cols);
    else walk<RAGGED, LANES, WEIGHTED, false, false, false, U>(acc, sizes, entries + i, WEIGHTED ? ws + i : nullptr, start + len - i, sl, r, 0, cols);
}

// MODE as for the paths: 0 M X, 1 D^-1/2 M D^-1/2 X, 2 = 1 then max(., 0), 3 D^-1 M X, 4 M X + s X.  DIRECT: no sums in memory.
template <bool RAGGED, int LANES, int MODE, bool GUARD, bool DIRECT, int U>
__global__ __launch_bounds__(256, 4) void cbm_sum_rows_kernel(const CbmSumItem* __restrict__ items, const SumMap map,
                                                              const uint32_t* __restrict__ entries, const float* __restrict__ ws,
                                                              const float* __restrict__ X, uint32_t ldx, const float* __restrict__ S, uint32_t lds,
                                                              const uint32_t* __restrict__ set_sizes, uint32_t ld_sizes, float* __restrict__ Y,
                                                              uint32_t ldy, const float* __restrict__ rw, float self_w, int k) {
    constexpr bool WEIGHTED = MODE == 1 || MODE == 2;
    const int64_t t = item_of<LANES>(map);
    if (t < 0) return;
    const CbmSumItem it = items[t];
    const uint32_t len = it.len & ~CBM_SUM_OWN;
    const bool holds_own = it.len & CBM_SUM_OWN;
    const int sl = threadIdx.x % LANES;
    const Columns<RAGGED, LANES> cols(sl, k);
    const float w = MODE == 0 || MODE == 4 ? 1.0f : rw[it.row];
    const float* mine = X + (uint64_t)(uint32_t)it.row * ldx;
    const bool add_own = MODE == 4 || it.own != 0;
    f4 own = {0.0f, 0.0f, 0.0f, 0.0f};
    if (add_own && !GUARD) own = cols.load(mine);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    Sizes sizes;
    const Rows from{X, ldx, S, lds, GUARD && !DIRECT ? set_sizes + blockIdx.y * LANES + sl : nullptr, ld_sizes};
    if constexpr (DIRECT) in_place<RAGGED, LANES, WEIGHTED, GUARD, U>(acc, sizes, items, entries, ws, it.start, len, -it.own, sl, from, cols);
    else if constexpr (GUARD) walk_sized<RAGGED, LANES, U>(acc, sizes, entries + it.start, len, -it.own, sl, from, cols);
    else walk<RAGGED, LANES, WEIGHTED, true, false, false, U>(acc, sizes, entries + it.start, WEIGHTED ? ws + it.start : nullptr, len, sl, from, 0, cols);
    if (add_own && GUARD) own = cols.load(mine);  // (here, 7 waves a SIMD; asked for before the walk, 6)
    const float times = ((float)it.own + (MODE == 4 ? self_w : 0.0f)) * (WEIGHTED ? w : 1.0f);
    if (add_own)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(times, own[c], acc[c]);
    if (it.own < 0) {
        // The row's own column was summed more often than the row holds it and taken off again.  That is right for finite sums only (an
        // infinity less itself is NaN), and where the row does not hold its own column at all, what rounding leaves of it has to be small beside
        // what the row does hold (kGuard).  Otherwise the row is put together from its sets' columns, each once.
        bool again[4], any = false;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            again[c] = !(fabsf(acc[c]) < INFINITY);
            if (GUARD && !holds_own && !again[c]) {
                const float kept = MODE == 4 ? fabsf(self_w * own[c]) : 0.0f;
                if (-(float)it.own * fabsf(own[c]) > kGuard * fmaxf(sizes.others(c), kept)) {
                    if (sizes.others(c) == 0.0f) acc[c] = MODE == 4 ? self_w * own[c] : 0.0f;  // all others are zero
                    else again[c] = true;
                }
            }
            any = any || again[c];
        }
        const uint64_t group = (LANES == 64 ? ~0ull : ((1ull << LANES) - 1)) << ((threadIdx.x & 63) / LANES * LANES);
        if (__ballot(any) & group) {
            // (its place among the entries is read once more: two registers less beside the walk, 7 waves a SIMD where there would be 6: 139 -> 136 us at k = 128)
            const volatile CbmSumItem* me = items + item_of<LANES>(map);
            const f4 sum = apart<RAGGED, LANES, WEIGHTED>(items, entries, ws, me->start, me->len & ~CBM_SUM_OWN, (uint32_t)it.row, sl, from, cols);
            const float once = ((holds_own ? 1.0f : 0.0f) + (MODE == 4 ? self_w : 0.0f)) * (WEIGHTED ? w : 1.0f);
            const f4 x = cols.load(mine);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (again[c]) acc[c] = MODE == 4 || holds_own ? fmaf(once, x[c], sum[c]) : sum[c];
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
    uint32_t* sizes;
    float* Y;
    uint32_t ldy;
    const float* rw;
    float self_w;
    int k;
    hipStream_t stream;
};

// The two launches of a product, and the one that does without memory for sums.
enum Part { SETS, ROWS, DIRECT };

template <bool RAGGED, int LANES, int MODE, bool GUARD>
void launch(const Args& a, Part part) {
    constexpr int G = 64 / LANES;
    constexpr int U = 8;  // 4 waves a SIMD; 4 rows at 8 waves: 30,000 nodes, k = 64 26 us instead of 22, 235,868 nodes the same; 2 rows 31
    SumMap map;
    uint32_t most = 0;
    for (int j = 0; j < CBM_XCD; ++j) {
        map.begin[j] = (uint32_t)a.h->sum_begin[part != SETS][j];
        map.count[j] = (uint32_t)a.h->sum_count[part != SETS][j];
        most = std::max(most, map.count[j]);
    }
    const dim3 grid(CBM_XCD * ((most + 4 * G - 1) / (4 * G)), (a.k + 4 * LANES - 1) / (4 * LANES));
    const uint32_t ld_sizes = (uint32_t)cbm_sum_sizes(a.k);
    auto rows = [&](auto direct) {
        hipLaunchKernelGGL((cbm_sum_rows_kernel<RAGGED, LANES, MODE, GUARD, decltype(direct)::value, U>), grid, dim3(256), 0, a.stream, a.h->d_sum_items, map,
                           a.h->d_sum_entries, a.h->d_sum_w, a.X, a.ldx, a.S, a.lds, a.sizes, ld_sizes, a.Y, a.ldy, a.rw, a.self_w, a.k);
    };
    if (part == ROWS) rows(std::false_type{});
    else if (part == DIRECT) rows(std::true_type{});
    else if constexpr (MODE <= 1)
        hipLaunchKernelGGL((cbm_sum_sets_kernel<RAGGED, LANES, MODE == 1, GUARD, U>), grid, dim3(256), 0, a.stream, a.h->d_sum_items, map,
                           a.h->d_sum_entries, a.h->d_sum_w, a.X, a.ldx, a.S, a.lds, a.sizes, ld_sizes, a.k);
}
template <bool RAGGED, int LANES>
void launch_mode(const Args& a, int mode, bool guard, Part part) {
    if (part == SETS) mode = mode == 1 || mode == 2 ? 1 : 0;  // (weighted or not)
    switch (mode) {
        case 0: return guard ? launch<RAGGED, LANES, 0, true>(a, part) : launch<RAGGED, LANES, 0, false>(a, part);
        case 1: return launch<RAGGED, LANES, 1, false>(a, part);
        case 2: return launch<RAGGED, LANES, 2, false>(a, part);
        case 3: return guard ? launch<RAGGED, LANES, 3, true>(a, part) : launch<RAGGED, LANES, 3, false>(a, part);
        default: return guard ? launch<RAGGED, LANES, 4, true>(a, part) : launch<RAGGED, LANES, 4, false>(a, part);
    }
}
template <bool RAGGED>
void launch_lanes(const Args& a, int mode, bool guard, Part part) {
    if (a.k <= 32) launch_mode<RAGGED, 8>(a, mode, guard, part);
    else if (a.k <= 64) launch_mode<RAGGED, 16>(a, mode, guard, part);
    else launch_mode<RAGGED, 32>(a, mode, guard, part);
}

constexpr size_t kMostScratch = 16;  // arrays of sums a handle keeps: one each for so many streams and captures
constexpr size_t kForStreams = 2;    // of these, never given to captures
constexpr size_t kQuietStreams = 4;
constexpr uint64_t kNobody = ~0ull;

}  // namespace

void cbm_launch_sum_chunk(const cbm_handle* h, bool rows, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy, int mode, const float* rw,
                          float self_w, float* S, int64_t lds, void* stream) {
    const bool guard = cbm_sum_guarded(h, mode, self_w);
    uint32_t* sizes = guard && S ? reinterpret_cast<uint32_t*>(S + h->num_sums * lds) : nullptr;
    const Args a{h, X, (uint32_t)ldx, S, (uint32_t)lds, sizes, Y, (uint32_t)ldy, rw, self_w, (int)k, (hipStream_t)stream};
    const bool aligned = k % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && ((uintptr_t)X & 15) == 0 && ((uintptr_t)Y & 15) == 0;
    const Part part = !S ? DIRECT : rows ? ROWS : SETS;
    if (aligned) launch_lanes<false>(a, mode, guard, part);
    else launch_lanes<true>(a, mode, guard, part);
}

bool cbm_sum_guarded(const cbm_handle* h, int mode, float self_w) {  // (the sum that a GIN layer makes holds 1 + eps times the row's own value)
    return (mode == 0 || mode == 3 || mode == 4) && (float)h->sum_most_taken_off > (mode == 4 ? kGuard * std::fabs(self_w) : 0.0f);
}

// The array for the sums of products on this stream; nullptr if there is none and none can be had.  Products of different streams may
// run at the same time, so each has its own; so has every capture, whose graph may be replayed beside anything.  A stream's array is another's that asks
// for one when the event behind the last product on its own stream, where there is one, has passed.  A capture's is kept until the caller says that no graph
// is left (cbm_release_captures): the graph's end does not say so, for hipGraphExecUpdate has an instance of another graph go on with what this one
// used.  The caller holds h->sum_mutex and calls cbm_sum_enqueued when the product is enqueued.  (The first array is allocated with the handle; the
// allocation and the questions here are ones that a capture under way does not mind.)
CbmSumScratch* cbm_sum_scratch(const cbm_handle* h, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    const uint64_t me = (uint64_t)(uintptr_t)stream;
    uint64_t capture = 0, thread = 0;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(stream, &status, &id) != hipSuccess) (void)hipGetLastError();
    else if (status == hipStreamCaptureStatusActive) capture = id + 1;
    if (stream == hipStreamPerThread) thread = (uint64_t)std::hash<std::thread::id>{}(std::this_thread::get_id());
    auto& all = h->sum_scratch;
    for (CbmSumScratch& s : all)
        if (s.stream == me && s.capture == capture && s.thread == thread) {
            s.passed = false;
            return &s;
        }
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    size_t captured = 0;
    for (const CbmSumScratch& s : all) captured += s.capture != 0;
    CbmSumScratch* mine = nullptr;
    for (CbmSumScratch& s : all)
        if (!mine && s.stream == kNobody && (capture == 0 || captured + 1 < all.size())) mine = &s;
    if (capture == 0)
        for (CbmSumScratch& s : all)
            if (!mine && s.capture == 0 && s.passed) {
                if (hipEventQuery((hipEvent_t)s.done) == hipSuccess) mine = &s;
                else (void)hipGetLastError();
            }
    if (!mine && all.size() < kMostScratch && (capture == 0 || captured + kForStreams < kMostScratch)) {
        float* sums = nullptr;
        if (hipMalloc((void**)&sums, cbm_sum_bytes(h)) == hipSuccess) {
            all.emplace_back();
            mine = &all.back();
            mine->sums = sums;
        } else {
            (void)hipGetLastError();
        }
    }
    if (mine) {
        mine->stream = me;
        mine->capture = capture;
        mine->thread = thread;
        mine->passed = false;
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return mine;
}

// (The event takes 2.8 us of the stream's time, 18.5 us a product on 20,000 nodes: up to kQuietStreams streams keep what they have without.)
void cbm_sum_enqueued(const cbm_handle* h, CbmSumScratch* s, void* stream) {
    if (s->capture != 0) return;
    size_t streams = 0;
    for (const CbmSumScratch& o : h->sum_scratch) streams += o.capture == 0 && o.stream != kNobody;
    if (streams <= kQuietStreams) return;
    if (!s->done && hipEventCreateWithFlags((hipEvent_t*)&s->done, hipEventDisableTiming) != hipSuccess) s->done = nullptr;
    s->passed = s->done && hipEventRecord((hipEvent_t)s->done, (hipStream_t)stream) == hipSuccess;
    if (!s->passed) (void)hipGetLastError();
}

void cbm_sum_release_captures(const cbm_handle* h) {
    std::lock_guard<std::mutex> lock(h->sum_mutex);
    for (CbmSumScratch& s : h->sum_scratch)
        if (s.capture != 0) {
            s.stream = kNobody;
            s.capture = 0;
        }
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
    CbmSumScratch first;
    first.stream = kNobody;
    if (ok) ok = hipMalloc((void**)&first.sums, cbm_sum_bytes(h)) == hipSuccess;
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
    for (CbmSumScratch& s : h->sum_scratch) {
        hipFree(s.sums);
        if (s.done) hipEventDestroy((hipEvent_t)s.done);
    }
    h->sum_scratch.clear();
    if (h->d_sum_items) hipFree(h->d_sum_items);
    if (h->d_sum_entries) hipFree(h->d_sum_entries);
    if (h->d_sum_w) hipFree(h->d_sum_w);
    h->d_sum_items = nullptr;
    h->d_sum_entries = nullptr;
    h->d_sum_w = nullptr;
}

// Products of small handles whose rows are all stored in full: segments and rows in one launch, a wave for each.
//
// Such a product is bound by latency: a row of a hundred entries walked by one group of eight lanes is thirteen batches of loads, one
// after the other (communities of 300 nodes, k = 16: 18.6 us for a launch of ten workgroups), and the segments of split rows wait for nobody,
// yet ran in a launch of their own before the rows.  Here the 64 / LANES groups of a wave take an item's entries in turn, 64 at a time, and
// add their sums across the wave at the end; rows of up to CBM_FLAT_SHORT entries have a group each.  The columns of X beyond 4 LANES are other
// workgroups' (blockIdx.y).
// Measured (us, before -> here): communities of 300, 1,024 and 5,000 nodes, k = 32 18.9 -> 5.6, 16.7 -> 6.1 (in row blocks 9.1), 17.9 -> 5.6; directed R-MAT
// scale 14, k = 64 37 -> 16, scale 16 68 -> 45; R-MAT scale 14, 32 edges a node, k = 64 46 -> 24.
// Which launches (CBM_FLAT_MOST_WAVES and the builder's flat_rich): what has more waves keeps the chip busy as it is, and sharing rows out costs it
// (R-MAT scale 15, k = 200, 54,000 waves 85 -> 99; scale 16, k = 100, 54,000 77 -> 86; directed scale 17, k = 128, 90,000 97 -> 130;
// below 43,000 everything gained: scale 16, k = 64 62 -> 57).  Now that segments share the rows' launch (cbm_kernels.hip) some below the line would be
// faster there (scale 16, k = 64 56 / 50, scale 14, k = 200 49 / 39), but less precise (2.3e-8 / 2.6e-8).  Nor do rows that are nearly all short gain (citation recipe, 19,717 nodes, k = 128 12 -> 16).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cbm_internal.h"
#include "cbm_rows.h"

namespace {

struct FlatArgs {
    const CbmTask* tasks;
    CbmSegMap segments;
    uint32_t segment_blocks, long_blocks;  // workgroups of segments, a multiple of 8, then of long rows; those of short rows follow
    int64_t row_begin, row_long, row_end;  // the rows, longest first; from row_long on they are short
    const uint32_t* stream;
    const float* ws;
    const float* rw;
    const float* X;
    int64_t ldx;
    float* Y;
    int64_t ldy;
    float* scratch;
    int64_t ld_scratch;
    float self_w;
    int k;
};

// One item by S neighbouring groups of LANES lanes, which take its entries in turn (entry i is group i mod S's).
template <bool RAGGED, int LANES, int MODE, int S>
__device__ __forceinline__ void flat_item(const FlatArgs& a, const CbmTask tk) {
    using M = Mode<MODE>;
    constexpr int W = LANES * S;  // lanes of the item: its entries come W at a time
    constexpr int U = 8;          // rows a group loads per batch
    static_assert(LANES % U == 0 && W <= 64, "a chunk of entries is whole batches");
    constexpr uint32_t BPC = LANES / U;  // batches per chunk
    const int lane = threadIdx.x % W, group = lane / LANES, sl = lane % LANES;
    const bool segment = tk.len_flags & CBM_TASK_SEGMENT;
    const uint32_t len = (tk.len_flags & CBM_TASK_LEN_MASK) - (segment ? 0 : 1);  // (a row's last entry is its marker)
    const int c0 = first_column<RAGGED, LANES>(blockIdx.y, sl);
    const bool colok = c0 < a.k;
    const float* X = a.X;
    const uint32_t* es = a.stream + tk.start;
    const float* wes = a.ws + tk.start;
    auto load_e = [&](uint32_t at) { return at + lane < len ? __builtin_nontemporal_load(es + at + lane) : 0u; };
    auto load_w = [&](uint32_t at) { return M::wcol && at + lane < len ? __builtin_nontemporal_load(wes + at + lane) : 0.0f; };
    uint32_t e0 = load_e(0), e1 = load_e(W);
    float w0 = load_w(0), w1 = load_w(W), wprev = 0.0f;
    uint32_t cur = 0;
    // what storing the row takes, while its entries are on their way
    float w = 1.0f;
    Vec4 own;
#pragma unroll
    for (int c = 0; c < 4; ++c) own.v[c] = 0.0f;
    if (!segment) {
        if (M::wrow) w = a.rw[tk.row];
        if (M::self && colok) own = ld_row<RAGGED, LANES>(X + (int64_t)tk.row * a.ldx, c0, a.k);
    }

    constexpr int P4 = 4;  // sums that take a group's entries in turn
    Vec4 part[P4];
#pragma unroll
    for (int p = 0; p < P4; ++p)
#pragma unroll
        for (int c = 0; c < 4; ++c) part[p].v[c] = 0.0f;
    struct Batch {
        Vec4 x[U];
    };
    const uint32_t nb = (len + U * S - 1) / (U * S);
    auto fetch = [&](Batch& B, uint32_t b) {
        if (b > 0 && b % BPC == 0) {
            e0 = e1;
            wprev = w0;
            w0 = w1;
            cur = b / BPC;
            e1 = load_e((cur + 1) * W);
            w1 = load_w((cur + 1) * W);
        }
        const int off = (int)(b % BPC) * U * S + group;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = (uint32_t)__shfl((int)e0, off + u * S, W);
            if (b * U * S + u * S + group < len && colok) {
                B.x[u] = ld_row<RAGGED, LANES>(X + (int64_t)(e & CBM_ENTRY_INDEX_MASK) * a.ldx, c0, a.k);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) B.x[u].v[c] = 0.0f;
            }
        }
    };
    auto consume = [&](const Batch& B, uint32_t b) {
        const float wsrc = b / BPC == cur ? w0 : wprev;
        const int off = (int)(b % BPC) * U * S + group;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float v = M::wcol ? __shfl(wsrc, off + u * S, W) : 1.0f;  // (0 past the last entry)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float& sum = part[u % P4].v[c];
                sum = M::wcol ? fmaf(v, B.x[u].v[c], sum) : sum + B.x[u].v[c];
            }
        }
    };
    Batch P, Q;
    if (nb > 0) fetch(P, 0);
    for (uint32_t b = 0; b < nb; b += 2) {
        if (b + 1 < nb) fetch(Q, b + 1);
        consume(P, b);
        if (b + 2 < nb) fetch(P, b + 2);
        if (b + 1 < nb) consume(Q, b + 1);
    }
    // The sums, and beside them what rounding takes from each of these additions (exactly, by Knuth's TwoSum: a sum's error is a value of its own),
    // added at the end: the result is then nearer to the sum than the matrix cores of row blocks come (communities of 1,024 nodes, k = 16, error against 64
    // bits 5.6e-8, in row blocks 7.3e-8; with one sum a group and no errors 7.9e-8).  Of a sum that is not finite the errors say nothing.
    Vec4 acc = part[0], lost;
#pragma unroll
    for (int c = 0; c < 4; ++c) lost.v[c] = 0.0f;
    auto add = [&](int c, float y) {
        const float x = acc.v[c], sum = x + y, more = sum - x;
        lost.v[c] += (x - (sum - more)) + (y - more);
        acc.v[c] = sum;
    };
#pragma unroll
    for (int p = 1; p < P4; ++p)
#pragma unroll
        for (int c = 0; c < 4; ++c) add(c, part[p].v[c]);
#pragma unroll
    for (int d = LANES; d < W; d *= 2)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float other = __shfl_xor(lost.v[c], d, 64);
            add(c, __shfl_xor(acc.v[c], d, 64));
            lost.v[c] += other;
        }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (fabsf(acc.v[c]) < INFINITY) acc.v[c] += lost.v[c];
    if (group != 0 || !colok) return;
    if (segment) st_row<RAGGED, LANES>(a.scratch + (int64_t)tk.row * a.ld_scratch, c0, a.k, acc);
    else store_row<RAGGED, LANES, MODE>(a.Y + (int64_t)tk.row * a.ldy, c0, a.k, acc, true, w, own, a.self_w);
}

template <bool RAGGED, int LANES, int MODE>
__global__ __launch_bounds__(256, 3) void cbm_flat_kernel(const FlatArgs a) {
    constexpr int G = 64 / LANES;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x >= a.segment_blocks + a.long_blocks) {  // short rows: a group each
        const int64_t t = a.row_long + ((int64_t)(blockIdx.x - a.segment_blocks - a.long_blocks) * 4 + wave) * G + (threadIdx.x & 63) / LANES;
        if (t < a.row_end) flat_item<RAGGED, LANES, MODE, 1>(a, a.tasks[t]);
        return;
    }
    int64_t t;
    if (blockIdx.x < a.segment_blocks) {
        const int xcd = blockIdx.x % CBM_XCD;
        const int64_t i = (int64_t)(blockIdx.x / CBM_XCD) * 4 + wave;
        if (i >= a.segments.count[xcd]) return;
        t = a.segments.begin[xcd] + i;
    } else {
        t = a.row_begin + (int64_t)(blockIdx.x - a.segment_blocks) * 4 + wave;
        if (t >= a.row_long) return;
    }
    flat_item<RAGGED, LANES, MODE, G>(a, a.tasks[t]);
}

template <bool RAGGED, int LANES>
const void* kernel(int mode) {
    switch (mode) {
        case 0: return (const void*)cbm_flat_kernel<RAGGED, LANES, 0>;
        case 1: return (const void*)cbm_flat_kernel<RAGGED, LANES, 1>;
        case 2: return (const void*)cbm_flat_kernel<RAGGED, LANES, 2>;
        case 3: return (const void*)cbm_flat_kernel<RAGGED, LANES, 3>;
        default: return (const void*)cbm_flat_kernel<RAGGED, LANES, 4>;
    }
}
template <bool RAGGED>
const void* kernel_lanes(int lanes, int mode) {
    switch (lanes) {
        case 8: return kernel<RAGGED, 8>(mode);
        case 16: return kernel<RAGGED, 16>(mode);
        default: return kernel<RAGGED, 32>(mode);
    }
}

// Launches of so few waves take slabs of 32 columns (16, ...) as long as they stay that few: more loads in flight for each row (communities of
// 1,024 nodes, k = 128 7.9 -> 6.1 us; with 8,192 waves 5,000 nodes would go from 8.1 to 9.0).
constexpr int64_t kFlatNarrowWaves = 2048;

}  // namespace

int cbm_flat_lanes(const cbm_handle* h, int32_t k) {
    int lanes = 8;
    while (lanes < 32 && 4 * (int64_t)lanes < k) lanes *= 2;
    while (lanes > 8 && cbm_flat_waves(h, lanes / 2, k) <= kFlatNarrowWaves) lanes /= 2;
    return cbm_flat_waves(h, lanes, k) <= h->flat_most_waves ? lanes : 0;
}

bool cbm_launch_flat(const cbm_handle* h, bool segments, bool rows, int lanes, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy,
                     float* scratch, int64_t ld_scratch, int mode, const float* rw, float self_w, bool aligned, void* stream) {
    FlatArgs a{h->d_tasks, {}, 0, 0, 0, 0, 0, h->d_stream, h->d_wstream, rw, X, ldx, Y, ldy, scratch, ld_scratch, self_w, (int)k};
    int64_t blocks = 0;
    if (segments) {
        int64_t most = 0;
        for (int j = 0; j < CBM_XCD; ++j) {
            a.segments.begin[j] = h->seg_begin[j];
            a.segments.count[j] = h->seg_count[j];
            most = std::max(most, h->seg_count[j]);
        }
        a.segments.use = 1;
        a.segment_blocks = (uint32_t)(CBM_XCD * ((most + 3) / 4));
        blocks = a.segment_blocks;
    }
    if (rows) {
        a.row_begin = h->levels[0].task_begin;
        a.row_long = a.row_begin + h->flat_long;
        a.row_end = a.row_begin + h->levels[0].task_count;
        a.long_blocks = (uint32_t)((h->flat_long + 3) / 4);
        const int64_t per = 4 * 64 / lanes;
        blocks += a.long_blocks + (a.row_end - a.row_long + per - 1) / per;
    }
    if (blocks == 0) return true;
    const dim3 grid((unsigned)blocks, (unsigned)((k + 4 * lanes - 1) / (4 * lanes)));
    // (one call of the runtime, not one for the launch's shape and one for its status beside it: their time is a part of these products')
    void* args[] = {&a};
    return hipLaunchKernel(aligned ? kernel_lanes<false>(lanes, mode) : kernel_lanes<true>(lanes, mode), grid, dim3(256), args, 0, (hipStream_t)stream) == hipSuccess;
}

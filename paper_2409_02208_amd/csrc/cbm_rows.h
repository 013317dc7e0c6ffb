// How the gather kernels hold and move rows, and what they do to a finished one (gfx950 device code).
#pragma once

#include <hip/hip_runtime.h>

#include "cbm_internal.h"

namespace {

// Four columns of a row: what one lane holds.
struct alignas(16) Vec4 {
    float v[4];
};
typedef float float4a __attribute__((ext_vector_type(4)));

// Which four columns a lane holds, and how it moves them.
// RAGGED = false: k is a multiple of 4 and every row starts on a 16-byte boundary; lane l of a group holds the
// consecutive columns 4l .. 4l+3 of the group's column chunk: one aligned 128-bit access.
// RAGGED = true: any k, leading dimension and base address; lane l holds columns l, l + LANES, l + 2 LANES,
// l + 3 LANES of the chunk, so every access is a 32-bit one that the group's lanes make to consecutive words.
template <bool RAGGED, int LANES>
__device__ __forceinline__ Vec4 ld_row(const float* row, int c0, int k) {
    Vec4 r;
    if (!RAGGED) {
        const float4a t = *reinterpret_cast<const float4a*>(row + c0);
#pragma unroll
        for (int c = 0; c < 4; ++c) r.v[c] = t[c];
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) r.v[c] = c0 + c * LANES < k ? row[c0 + c * LANES] : 0.0f;
    }
    return r;
}
// Streaming store: rows of Y and partial sums are written once and not re-read by the same launch, so
// they should not displace the gathered rows of X from L2.
template <bool RAGGED, int LANES>
__device__ __forceinline__ void st_row(float* row, int c0, int k, const Vec4& x) {
    if (!RAGGED) {
        float4a t;
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = x.v[c];
        __builtin_nontemporal_store(t, reinterpret_cast<float4a*>(row + c0));
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c0 + c * LANES < k) __builtin_nontemporal_store(x.v[c], row + c0 + c * LANES);
    }
}
// first column of lane `sl` in column chunk `chunk` (a chunk = 4 LANES columns either way)
template <bool RAGGED, int LANES>
__device__ __forceinline__ int first_column(int chunk, int sl) {
    return RAGGED ? chunk * 4 * LANES + sl : (chunk * LANES + sl) * 4;
}

// MODE 0: Y = M X (M = the compressed matrix).
// MODE 1: Y = D^-1/2 M D^-1/2 X with M = A v I (the normalised adjacency).  MODE 2: MODE 1 then max(., 0).
// MODE 3: Y = D^-1 M X (mean over each row's entries: the GraphSAGE mean aggregator).
// MODE 4: Y = M X + s X (s = 1 + eps: the GIN aggregator).
// Column weights multiply gathered rows, row weights the stored row; the self term of MODE 4 is the
// row's own X row, fetched by its marker entry like any gathered row.
// A row that ANOTHER work item is compressed against (INTERNAL) is written as the bare running sum,
// because that work item continues from it (the row scale belongs to the update step, Section 2.2);
// cbm_finish_kernel applies the row weight / self term to those rows once every round is done.
template <int MODE>
struct Mode {
    static constexpr bool wcol = MODE == 1 || MODE == 2;
    static constexpr bool wrow = MODE == 1 || MODE == 2 || MODE == 3;
    static constexpr bool relu = MODE == 2;
    static constexpr bool self = MODE == 4;
    static constexpr bool weights = wcol || wrow;
};

// out = finish(acc): acc (+ self_w * own X row) (* row weight) (then ReLU)
template <bool RAGGED, int LANES, int MODE>
__device__ __forceinline__ void store_row(float* row, int c0, int k, Vec4 acc, bool finish, float w, const Vec4& own,
                                          float self_w) {
    if (finish) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (Mode<MODE>::self) acc.v[c] = fmaf(self_w, own.v[c], acc.v[c]);
            if (Mode<MODE>::wrow) acc.v[c] *= w;
            if (Mode<MODE>::relu) acc.v[c] = fmaxf(acc.v[c], 0.0f);
        }
    }
    st_row<RAGGED, LANES>(row, c0, k, acc);
}

// Some launches map workgroups to work items per XCD: workgroup b runs on XCD b mod 8 and takes its items from that XCD's block of the
// task list.
struct CbmSegMap {
    int64_t begin[CBM_XCD];
    int64_t count[CBM_XCD];
    int use;
};

}  // namespace

// Dense fp32 matmul C = A.B for few columns on the bf16 matrix cores, B held in registers: a panel of up to 64 of them, or up to four such panels side by
// side (grid dimension y).
//
// Operands are split into three bf16 parts as in cbm_gemm_split.hip, which says why that is as good as fp32, and multiplied in eight products instead of six where this
// kernel takes over from the fp32 ones: there a row of a single term is rounded once, and ml and lm are up to another rounding of a term.  (ll is 2^-34 of it.)  Where
// the kernels of six products would run otherwise (cbm_split_form) it makes six: 19717 x 500 . 500 x 64 15.5 -> 14.4, 20000 x 500 . 500 x 112 25 -> 23.
// Also different is who holds what: B is small, so each wave keeps the parts of its piece of B -- all columns, 32 STEPS of its rows -- in registers, split once,
// and streams 16 rows of A at a time past them (all columns: of the panel): no LDS, no barrier and no second look at B in the loop.  Where K is deeper than a wave can hold,
// SLICES waves, a workgroup, share K and add their sums through LDS, one barrier for 16 rows.  Rows of A go straight from memory into operand
// layout (lane l: row l % 16, eight k from 8 (l / 16) on); a step's registers are free when it is split, and the next rows are asked for there and then.
// Asking two tiles of rows ahead gains nothing, nor does adding up a tile's shares beside the next one's products.
//
// What bounds it: reading A and writing C (us, the kernels that ran before -> here; what a large copy's 4.66 TB/s would take): 132534 x 100 . 100 x 47
// 26.7 -> 22.1 (16.7), 132534 x 256 . 256 x 64 48 -> 38 (36), 132534 x 32 . 32 x 32 12.8 -> 8.4, 300000 x 16 . 16 x 16 13.0 -> 9.5 (8.2), 60000 x 500 . 500 x 64
// 43 -> 36 (29), 100000 x 301 . 301 x 40 51 -> 35 (29).  Few rows: a wave's piece of B and one or two tiles of rows, one after the other: 19717 x 500 . 500 x 64
// 21.4 -> 14.4 (9.6; 1,233 tiles are 4.8 for each compute unit), . 500 x 7 13.6 -> 8.6, 3000 x 512 . 512 x 64 9.9 -> 6.5; a call costs 5 us of host time beside it.
// Error against 64 bits in the 2-norm, Gaussian values: K = 100 1.8e-7 (fp32 kernels) -> 0.6e-7, 256 2.9e-7 -> 0.5e-7, 500 4.0e-7 -> 0.5e-7 (through parts
// without B held 0.76e-7).  One term a row 2.53e-8, at most 1.002 times 2^-24 of it (six products: 2.60e-8 and 1.6 to 1.7 times; fp32 2.53e-8 and once).  What the two
// products cost (us): 132534 x 100 . 100 x 47 20.0 -> 20.9, 132534 x 256 . 256 x 64 36 -> 39, 60000 x 500 . 500 x 64 31 -> 36, 132534 x 32 . 32 x 32 no time.  Values that are not finite (finite ones, one infinity in B, NaN all
// over A): 132534 x 100 . 100 x 47 22, 36, 62, 132534 x 256 . 256 x 64 42, 80, 167, 20000 x 500 . 500 x 64 16, 27, 52, 50000 x 300 . 300 x 33 21, 40, 71 (where each wave
// that added shares up went over all of K alone, between two barriers: 20000 x 500 . 500 x 64 110, 158, 50000 x 300 . 300 x 33 107, 216, 132534 x 256 . 256 x 64 207, 336).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "cbm_gemm_rules.h"
#include "cbm_internal.h"
#include "cbm_split.h"

namespace {

// Operands are split at 2^24 times their size and sums come back by 2^-48: nothing small is lost (cbm_gemm_split.hip).
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;
constexpr int PA[8] = {2, 1, 2, 0, 1, 1, 0, 0}, PB[8] = {1, 2, 0, 2, 1, 0, 1, 0};  // small ones first, that of the large parts last

struct Parts {
    bf16x8 p[3];  // h, m, l
};
__device__ __forceinline__ Parts split8(const float (&x)[8], uint32_t minus_low) {
    uintx4 q[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t h, m, l;
        split_pair_nearest(x[2 * i] * kUp, x[2 * i + 1] * kUp, minus_low, h, m, l);
        q[0][i] = h;
        q[1][i] = m;
        q[2][i] = l;
    }
    Parts r;
#pragma unroll
    for (int i = 0; i < 3; ++i) r.p[i] = __builtin_bit_cast(bf16x8, q[i]);
    return r;
}

struct Shape {
    int64_t M;
    int N, K;
    const float* A;
    int64_t lda;
    const float* B;
    int64_t ldb;
    float* C;
    int64_t ldc;
    bool six;  // products of parts instead of eight: where the kernels of cbm_gemm_split.hip would run otherwise (two tiles of columns: from 128 k on)
};

constexpr int held_waves(int slices) { return slices == 1 ? 4 : slices; }
// VEC: K is a multiple of 4 and rows of A start on 16-byte boundaries.  PRODUCTS of parts: eight, or without ml and lm six.
template <int NT, int STEPS, int SLICES, bool VEC, int PRODUCTS>
__global__ __launch_bounds__(64 * held_waves(SLICES), 2) void cbm_gemm_held_kernel(const Shape all) {
    Shape s = all;  // this panel's
    s.B += blockIdx.y * (16 * NT);
    s.C += blockIdx.y * (16 * NT);
    s.N = min(s.N - (int)blockIdx.y * (16 * NT), 16 * NT);
    constexpr int WAVES = held_waves(SLICES);
    constexpr int GROUPS = WAVES / SLICES;  // rows of 16 that a workgroup works on at a time
    static_assert(GROUPS == 1 || SLICES == 1, "waves that share K are a whole workgroup");
    __shared__ float red[SLICES > 1 ? 2 : 1][SLICES > 1 ? SLICES : 1][SLICES > 1 ? 8 * NT : 1][64];
    __shared__ uint32_t doubt[2][SLICES];  // by wave that added them up: the tiles of columns that hold a sum that is not finite
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, l16 = lane & 15;
    const int slice = SLICES > 1 ? wave : 0;
    const int k0 = slice * 32 * STEPS + 8 * (lane >> 4);  // this lane's k: 8 from here on, 32 further for each step
    uint32_t minus_low = 0xbf80u;
    asm("" : "+s"(minus_low));

    const int64_t tiles = (s.M + 15) / 16, stride = (int64_t)gridDim.x * GROUPS;
    int64_t tile = (int64_t)blockIdx.x * GROUPS + (SLICES > 1 ? 0 : wave);
    if (tile >= tiles) return;  // (waves that share K leave together)
    float x[STEPS][8];
    const int whole = (s.K - slice * 32 * STEPS) / 32;  // steps that lie inside K
    // loads stay inside A: what they bring from beyond K is cut, from beyond M never stored
    auto row_of = [&](int64_t t) { return s.A + min(16 * t + l16, s.M - 1) * s.lda; };
    // whether rows of 16 can be read whole steps at a time: what a step reads beyond K is then of the next rows, and all of it inside A
    auto inside = [&](int64_t t) { return VEC || (16 * t + 15) * s.lda + (slice + 1) * 32 * STEPS <= (s.M - 1) * s.lda + s.K; };
    auto load_a = [&](float (&r)[8], const float* row, int step, bool whole_steps) {
        int k = k0 + 32 * step;
        if (whole_steps) {
            floatx4 lo, hi;
            if constexpr (VEC) {
                if constexpr (NT * STEPS == 12 || (NT == 1 && STEPS == 3)) asm("" : "+v"(k));  // (its places are not worth registers of their own outside the loop where there are none to spare)
                lo = *reinterpret_cast<const floatx4*>(row + min(k, s.K - 4));
                hi = *reinterpret_cast<const floatx4*>(row + min(k + 4, s.K - 4));
            } else {
                __builtin_memcpy(&lo, row + k, sizeof(lo));
                __builtin_memcpy(&hi, row + k + 4, sizeof(hi));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                r[j] = lo[j];
                r[4 + j] = hi[j];
            }
        } else {
            asm("" : "+v"(k));  // (nor are its eight)
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = row[min(k + j, s.K - 1)];
        }
    };
    {
        const float* row = row_of(tile);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) load_a(x[i], row, i, inside(tile));
    }
    Parts b[STEPS][NT];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        float y[NT][8];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float* col = s.B + min(16 * t + l16, s.N - 1);
#pragma unroll
            for (int j = 0; j < 8; ++j) y[t][j] = col[(int64_t)min(k0 + 32 * i + j, s.K - 1) * s.ldb];
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int j = 0; j < 8; ++j) y[t][j] = k0 + 32 * i + j < s.K ? y[t][j] : 0.0f;
            b[i][t] = split8(y[t], minus_low);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // register v of lane l of a tile of 16 x 16: row 4 (l / 16) + v, column l % 16
    auto put = [&](int64_t row, int t, float sum) {
        const int c = 16 * t + l16;
        if (c < s.N && row < s.M) s.C[row * s.ldc + c] = sum;
    };
    // Rows 16 at .. + 15, columns 16 t .. + 15 on the fp32 matrix cores, over this wave's k: a sum of infinite, NaN or very large values, which the parts
    // do not give.  (A tile at a time, by a loop: its registers come beside all that the wave holds.)
    auto plain = [&](int64_t at, int t) {
        const float* row = row_of(at);
        const bool whole_steps = inside(at);
        const float* col = s.B + min(16 * t + l16, s.N - 1);
        floatx4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int i = 0; i < STEPS; ++i) {
            float a[8], y[8];
            load_a(a, row, i, whole_steps);
            int k = k0 + 32 * i;
            asm("" : "+v"(k));
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = col[(int64_t)min(k + j, s.K - 1) * s.ldb];
#pragma unroll
            for (int j = 0; j < 8; ++j)  // (beyond K both are zero: what stands there may be infinite)
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(k + j < s.K ? a[j] : 0.0f, k + j < s.K ? y[j] : 0.0f, sum, 0, 0, 0);
        }
        return sum;
    };
    // The waves' shares of the 16 rows, a register at a time: the large sums in 64 bits, where their sum loses nothing (in 32 bits K = 320 7.1e-8
    // instead of 5.5e-8) and does not overflow, with the small ones added at the end.
    constexpr int PER = (4 * NT + SLICES - 1) / SLICES;  // registers of a wave, one after the other
    auto add_up = [&](int buf) {
        uint32_t again = 0;
        float sum[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = PER * SLICES > 4 * NT ? min(slice * PER + i, 4 * NT - 1) : slice * PER + i;
            float few = red[buf][0][at][lane];
            double most = (double)red[buf][0][4 * NT + at][lane];
#pragma unroll
            for (int w = 1; w < SLICES; ++w) {
                few += red[buf][w][at][lane];
                most += (double)red[buf][w][4 * NT + at][lane];
            }
            sum[i] = (float)((most + (double)few) * (double)kDown);
            again |= (__ballot(!(fabsf(sum[i]) < INFINITY)) != 0 ? 1u : 0u) << (at / 4);
        }
        doubt[buf][slice] = again;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = slice * PER + i;
            if (PER * SLICES == 4 * NT || at < 4 * NT) put(16 * tile + 4 * (lane >> 4) + at % 4, at / 4, sum[i]);
        }
    };
    // Tiles of rows 16 at .. + 15 that add_up was not sure of, stored once more by the lanes that stored them: all waves come here after the barrier that
    // follows it, and share K as before.
    auto settle = [&](int buf, int64_t at, uint32_t unsure) {
        uint32_t again = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) again |= (__ballot(unsure >> t & 1u) != 0 ? 1u : 0u) << t;
        for (uint32_t left = again; left; left &= left - 1) {
            const int t = __builtin_ctz(left);
            const floatx4 sum = plain(at, t);
#pragma unroll
            for (int v = 0; v < 4; ++v) red[buf][slice][4 * t + v][lane] = sum[v];
        }
        __syncthreads();
        for (uint32_t left = again; left; left &= left - 1) {
            const int t = __builtin_ctz(left);
            for (int v = 0; v < 4; ++v) {
                if ((4 * t + v) / PER != slice) continue;
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < SLICES; ++w) sum += (double)red[buf][w][4 * t + v][lane];
                put(16 * at + 4 * (lane >> 4) + v, t, (float)sum);
            }
        }
        __syncthreads();  // (the next tile's shares go where these were)
    };
    for (int buf = 0;; buf ^= 1) {
        const int64_t then = min(tile + stride, tiles - 1);
        const float* next = row_of(then);
        const bool whole_steps = inside(then);
        floatx4 acc[NT], small[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = small[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            if (i >= whole) {
                int k = k0 + 32 * i;
                asm("" : "+v"(k));  // (nor are their conditions)
#pragma unroll
                for (int j = 0; j < 8; ++j) x[i][j] = k + j < s.K ? x[i][j] : 0.0f;
            }
            const Parts a = split8(x[i], minus_low);
            load_a(x[i], next, i, whole_steps);
#pragma unroll
            for (int q = 8 - PRODUCTS; q < 8; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    floatx4& sum = q < 7 ? small[t] : acc[t];
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[PA[q]], b[i][t].p[PB[q]], sum, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (SLICES == 1) {
            uint32_t again = 0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[t][v] = (acc[t][v] + small[t][v]) * kDown;
                bool bad = false;
#pragma unroll
                for (int v = 0; v < 4; ++v) bad = bad || !(fabsf(acc[t][v]) < INFINITY);
                again |= (__ballot(bad) != 0 ? 1u : 0u) << t;
#pragma unroll
                for (int v = 0; v < 4; ++v) put(16 * tile + 4 * (lane >> 4) + v, t, acc[t][v]);
            }
            for (; again; again &= again - 1) {  // (what was stored is stored once more: stores that may not be would have the next rows waited for with them)
                const int t = __builtin_ctz(again);
                const floatx4 sum = plain(tile, t);
#pragma unroll
                for (int v = 0; v < 4; ++v) put(16 * tile + 4 * (lane >> 4) + v, t, sum[v]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    red[buf][slice][4 * t + v][lane] = small[t][v];
                    red[buf][slice][4 * NT + 4 * t + v][lane] = acc[t][v];
                }
            __syncthreads();  // (the other buffer is free again when all have come here)
            const uint32_t unsure = doubt[buf ^ 1][lane % SLICES];
            add_up(buf);
            if (tile >= stride && __ballot(unsure != 0)) settle(buf ^ 1, tile - stride, unsure);
        }
        tile += stride;
        if (tile < tiles) continue;
        if constexpr (SLICES > 1) {
            __syncthreads();
            const uint32_t unsure = doubt[buf][lane % SLICES];
            if (__ballot(unsure != 0)) settle(buf, tile - stride, unsure);
        }
        return;
    }
}

// Workgroups: two waves a SIMD (eight sharing K: always), four where their registers leave room (300000 x 32 . 32 x 32 15.2 -> 13.8 us).
constexpr int held_grid(int nt, int steps, int slices) { return (steps * (12 * nt + 8) + 8 * nt + 60 <= 128 && slices != 8 ? 4096 : 2048) / held_waves(slices); }

template <int NT, int STEPS, int SLICES>
void launch(const Shape& s, hipStream_t stream) {
    constexpr int WAVES = held_waves(SLICES), GROUPS = WAVES / SLICES;
    const int64_t wanted = ((s.M + 15) / 16 + GROUPS - 1) / GROUPS;
    const int panels = (s.N + 16 * NT - 1) / (16 * NT);
    const dim3 grid((unsigned)cbm_panel_blocks(wanted, panels, held_grid(NT, STEPS, SLICES)), (unsigned)panels);
    const bool vec = s.K % 4 == 0 && s.lda % 4 == 0 && ((uintptr_t)s.A & 15) == 0;
    if constexpr (NT > 2 || STEPS * SLICES >= 4)
        if (s.six) {
            if (vec) hipLaunchKernelGGL((cbm_gemm_held_kernel<NT, STEPS, SLICES, true, 6>), grid, dim3(64 * WAVES), 0, stream, s);
            else hipLaunchKernelGGL((cbm_gemm_held_kernel<NT, STEPS, SLICES, false, 6>), grid, dim3(64 * WAVES), 0, stream, s);
            return;
        }
    if (vec) hipLaunchKernelGGL((cbm_gemm_held_kernel<NT, STEPS, SLICES, true, 8>), grid, dim3(64 * WAVES), 0, stream, s);
    else hipLaunchKernelGGL((cbm_gemm_held_kernel<NT, STEPS, SLICES, false, 8>), grid, dim3(64 * WAVES), 0, stream, s);
}

template <int NT, int SLICES>
bool launch_slices(const Shape& s, int steps, hipStream_t stream) {
    switch (steps) {
        case 1: launch<NT, 1, SLICES>(s, stream); return true;
        case 2: launch<NT, 2, SLICES>(s, stream); return true;
        case 3: launch<NT, 3, SLICES>(s, stream); return true;
        case 4:
            if constexpr (cbm_held_most_steps(NT) == 4) {
                launch<NT, 4, SLICES>(s, stream);
                return true;
            }
            return false;
        default: return false;
    }
}
template <int NT>
bool launch_nt(const Shape& s, const CbmHeldPlan& p, hipStream_t stream) {
    switch (p.slices) {
        case 1: return launch_slices<NT, 1>(s, p.each, stream);
        case 2: return launch_slices<NT, 2>(s, p.each, stream);
        case 4: return launch_slices<NT, 4>(s, p.each, stream);
        case 8: return launch_slices<NT, 8>(s, p.each, stream);
        default: return false;
    }
}

}  // namespace

cbm_status cbm_launch_gemm_held(int64_t M, int32_t N, int32_t K, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                int64_t ldc, void* stream, bool* taken) {
    *taken = false;
    // (for tests, which run several in one process: 5 = whatever K, with eight products, 0 to 4 = never, as another kernel is asked for)
    const char* e = std::getenv("CBM_GEMM_SPLIT");
    const bool asked = e && e[0] >= '0' && e[0] <= '5' && !e[1];
    if (asked ? e[0] != '5' || N > 256 : !cbm_held_takes(M, N, K, K % 4 == 0 && lda % 4 == 0 && ((uintptr_t)A & 15) == 0)) return CBM_OK;
    const Shape s{M, N, K, A, lda, B, ldb, C, ldc, !asked && cbm_split_form(M, N, K) != 0};
    const CbmHeldPlan p = cbm_held_plan(M, N, K);
    switch (p.tiles) {
        case 1: *taken = launch_nt<1>(s, p, (hipStream_t)stream); break;
        case 2: *taken = launch_nt<2>(s, p, (hipStream_t)stream); break;
        case 3: *taken = launch_nt<3>(s, p, (hipStream_t)stream); break;
        default: *taken = launch_nt<4>(s, p, (hipStream_t)stream); break;
    }
    if (!*taken) return CBM_OK;
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        cbm_set_error_detail("held matmul launch", hipGetErrorString(err));
        return CBM_ERR_HIP;
    }
    return CBM_OK;
}

// Dense fp32 matmul C = A.B on the bf16 matrix cores: both operands split into three bf16 parts that add up to the fp32 value
// exactly (8 + 8 + 8 significant bits, every part rounded to the nearest: x = h + m + l), six products of parts (hh, hm, mh, mm, hl,
// lh), 32-bit sums.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "cbm_gemm_rules.h"
#include "cbm_internal.h"
#include "cbm_split.h"

// The bf16 matrix cores are 16 times as fast as the fp32 ones, the six products leave 2.7.  Left out are ml, lm and ll: at most
// 2^-24 of a term (|m| <= 2^-8, |l| <= 2^-17 of the value), of either sign.  (By truncation m and l are twice and four times as large
// and have the value's sign: up to 7.8 * 2^-24 of a term, all on one side.)  The five small products have sums of their own: added
// to the large ones at every step, each of them would round a sum of full size.
// Error against 64 bits, fp32 kernels of cbm_gemm.hip -> these (2-norm, Gaussian values): K = 500 4.0e-7 -> 0.77e-7 up to 64 columns and
// 1.3e-7 beyond; ten non-zeros a row 5.9e-8 -> 3.0e-8, four 4.0e-8 -> 2.7e-8, one 2.5e-8 -> 2.6e-8 (at most 1.0 -> 1.7 times 2^-24).

namespace {

// Eight fp32 values (consecutive k of one row of A, or of one column of B) as three operands.
struct Parts {
    bf16x8 p[3];  // h, m, l
};
__device__ __forceinline__ Parts split8(const float (&x)[8], uint32_t minus_low) {
    uintx4 q[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t h, m, l;
        split_pair_nearest(x[2 * i], x[2 * i + 1], minus_low, h, m, l);
        q[0][i] = h;
        q[1][i] = m;
        q[2][i] = l;
    }
    Parts r;
#pragma unroll
    for (int i = 0; i < 3; ++i) r.p[i] = __builtin_bit_cast(bf16x8, q[i]);
    return r;
}

// the six products, the one of the large parts last; neighbouring instructions write different tiles
constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};

// FIRST: the first of b's N tiles
template <int FIRST, int N, int NT>
__device__ __forceinline__ void multiply(floatx16 (&acc)[NT], floatx16 (&small)[NT], const Parts& a, const Parts (&b)[N]) {
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int t = 0; t < N; ++t) {
            floatx16& sum = i < 5 ? small[FIRST + t] : acc[FIRST + t];
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[PA[i]], b[t].p[PB[i]], sum, 0, 0, 0);
        }
}

// Eight consecutive k of row `row` of A from k0 on, zero beyond K (addresses held inside the matrix).
template <bool VEC>
__device__ __forceinline__ void load_a(float (&x)[8], const float* __restrict__ row, int k0, int K) {
    if (VEC) {  // K and the row's address are multiples of 4
        const floatx4 lo = *reinterpret_cast<const floatx4*>(row + min(k0, K - 4)), hi = *reinterpret_cast<const floatx4*>(row + min(k0 + 4, K - 4));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = lo[j];
            x[4 + j] = hi[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = row[min(k0 + j, K - 1)];
    }
}
// No bf16 value has bits below 2^-133, and the matrix cores take what is below 2^-126 for zero: operands are split at 2^24 times
// their size, where the smallest fp32 value is 2^-125, and sums come back by 2^-48 (what is below 2^-126 then is below 2^-174 of
// the result).  Values and sums that are not finite, or are not any more at that size (from 2^104 and 2^80), give sums that are not
// finite: those are computed again on the fp32 matrix cores.  (Cheaper than to look for small values: with the largest operand kept
// beside the sums and small sums computed again, zeros could not be told from sums that had vanished, and 132534 x 256 . 256 x 256 took
// 138 us against 128.)
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;

__device__ __forceinline__ void cut_a(float (&x)[8], int k0, int K) {
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = k0 + j < K ? x[j] * kUp : 0.0f;
}
__device__ __forceinline__ bool doubtful(float v) { return !(fabsf(v) < INFINITY); }
// Rows row0 .. + 31, columns col0 .. + 31 of C on the fp32 matrix cores, for sums that the parts do not give.  Lane l has row, or
// column, l % 32 and four k from 4 (l / 32) on of every eight.  (132534 x 256 . 256 x 256, 131 us with finite values: one infinity in B
// 187 us, NaN all over A 444; 4,900 and 8,000 with a chain of multiply-adds per element.)
template <bool VEC>
__device__ __forceinline__ void plain_tile(int64_t M, int N, int K, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                        int64_t ldc, int64_t row0, int col0) {
    const int lane = threadIdx.x & 63, half = lane >> 5, c = col0 + (lane & 31);
    const float* a = A + min(row0 + (lane & 31), M - 1) * lda;
    const float* b = B + min(c, N - 1);
    floatx16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.0f;
    for (int k = 0; k < K; k += 8) {
        const int k0 = k + 4 * half;
        float x[4], y[4];
        if constexpr (VEC) {
            const floatx4 q = *reinterpret_cast<const floatx4*>(a + min(k0, K - 4));
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = q[j];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = a[min(k0 + j, K - 1)];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = b[(int64_t)min(k0 + j, K - 1) * ldb];
#pragma unroll
        for (int j = 0; j < 4; ++j)  // (beyond K both are zero: what stands there may be infinite)
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(k0 + j < K ? x[j] : 0.0f, k0 + j < K ? y[j] : 0.0f, s, 0, 0, 0);
    }
    if (c >= N) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int64_t r = row0 + 8 * (v / 4) + 4 * half + v % 4;
        if (r < M) C[r * ldc + c] = s[v];
    }
}

// Narrow C (up to 64 columns), for products that are short and deep: a workgroup has 32 rows of C, its four waves take the
// steps of 16 k in turn and add their sums through LDS.  Both operands come straight from memory in operand layout (lane l:
// row, or column, l % 32 and eight k from 8 (l / 32) on): B is small and stays in L2.  Loads run one step ahead (with parts by
// truncation, 19717 x 500 . 500 x 64: one step 24.9 us, three 27.8, the loads made past the end cost more than the wait; waves with all of
// K each 30).
constexpr int KS = 4, PF = 2;

template <int NT, bool VEC>
__global__ __launch_bounds__(256, 3) void cbm_gemm_narrow_kernel(int64_t M, int N, int K, const float* __restrict__ A, int64_t lda,
                                                                 const float* __restrict__ B, int64_t ldb, float* __restrict__ C, int64_t ldc) {
    __shared__ float red[KS - 1][NT * 16][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int64_t row0 = (int64_t)blockIdx.x * 32;
    const float* arow = A + min(row0 + l32, M - 1) * lda;
    const float* bcol[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bcol[t] = B + min(32 * t + l32, N - 1);
    floatx16 acc[NT], small[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = small[t][v] = 0.0f;
    uint32_t minus_low = 0xbf80u;
    asm("" : "+s"(minus_low));

    const int steps = (K + 15) / 16, first = wave;
    struct Step {
        float a[8], b[NT][8];
    };
    auto load = [&](Step& s, int i) {
        const int k0 = 16 * i + 8 * half;
        load_a<VEC>(s.a, arow, k0, K);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t at = (int64_t)min(k0 + j, K - 1) * ldb;
#pragma unroll
            for (int t = 0; t < NT; ++t) s.b[t][j] = bcol[t][at];
        }
    };
    auto use = [&](Step& s, int i) {
        cut_a(s.a, 16 * i + 8 * half, K);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) s.b[t][j] *= kUp;
        const Parts a = split8(s.a, minus_low);
        Parts b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = split8(s.b[t], minus_low);
        multiply<0>(acc, small, a, b);
    };
    if (first < steps) {  // (loads are always made, with the step held to this wave's last)
        const int last = first + (steps - 1 - first) / KS * KS;
        Step s[PF];
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            load(s[p], min(first + p * KS, last));
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int i = first; i <= last; i += PF * KS) {
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                if (i + p * KS <= last) use(s[p], i + p * KS);
                load(s[p], min(i + (p + PF) * KS, last));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the waves' shares, the small sums first and apart: the large ones then lose no bit to them before the last addition
    auto gather = [&](floatx16 (&x)[NT]) {
        if (wave > 0) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) red[wave - 1][16 * t + v][lane] = x[t][v];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int w = 0; w < KS - 1; ++w) x[t][v] += red[w][16 * t + v][lane];
    };
    gather(small);
    __syncthreads();
    gather(acc);
    if (wave > 0) return;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = (acc[t][v] + small[t][v]) * kDown;
    uint32_t again = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        bool bad = false;
#pragma unroll
        for (int v = 0; v < 16; ++v) bad = bad || doubtful(acc[t][v]);
        if (__ballot(bad)) {
            again |= 1u << t;
            continue;
        }
        const int c = 32 * t + l32;
        if (c < N)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t r = row0 + 8 * (v / 4) + 4 * half + v % 4;
                if (r < M) C[r * ldc + c] = acc[t][v];
            }
    }
    for (; again; again &= again - 1) plain_tile<VEC>(M, N, K, A, lda, B, ldb, C, ldc, row0, 32 * __builtin_ctz(again));
}

// Wider C: a workgroup of four waves has 128 rows by 32 NT columns.  B goes through LDS in chunks of 32 k, split as it is
// stored (two buffers, one barrier a chunk); A comes straight from memory.
constexpr int CK = 32;  // k per chunk

template <int NT, bool VEC>
__global__ __launch_bounds__(256, NT > 2 ? 2 : 3) void cbm_gemm_wide_kernel(int64_t M, int N, int K, const float* __restrict__ A,
                                                                            int64_t lda, const float* __restrict__ B, int64_t ldb,
                                                                            float* __restrict__ C, int64_t ldc) {
    constexpr int BN = 32 * NT;
    constexpr int PER = (CK / 8) * BN / 256;  // columns of eight k that a thread stages per chunk
    static_assert((CK / 8) * BN % 256 == 0, "every thread stages the same number");
    __shared__ uintx4 stage[2][3][CK / 8][BN];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int64_t row0 = (int64_t)blockIdx.x * 128 + 32 * wave;
    const int col0 = blockIdx.y * BN;
    const float* arow = A + min(row0 + l32, M - 1) * lda;
    floatx16 acc[NT], small[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = small[t][v] = 0.0f;
    uint32_t minus_low = 0xbf80u;
    asm("" : "+s"(minus_low));

    auto load_b = [&](float (&x)[PER][8], int chunk) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = threadIdx.x + 256 * i, k0 = chunk * CK + at / BN * 8;
            const float* col = B + min(col0 + at % BN, N - 1);
#pragma unroll
            for (int j = 0; j < 8; ++j) x[i][j] = col[(int64_t)min(k0 + j, K - 1) * ldb];
        }
    };
    auto store_b = [&](const float (&x)[PER][8], int buf) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = threadIdx.x + 256 * i;
            float up[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) up[j] = x[i][j] * kUp;
            const Parts p = split8(up, minus_low);
#pragma unroll
            for (int q = 0; q < 3; ++q) stage[buf][q][at / BN][at % BN] = __builtin_bit_cast(uintx4, p.p[q]);
        }
    };
    const int chunks = (K + CK - 1) / CK;
    float xb[PER][8], xa[2][8], na[2][8];
    load_b(xb, 0);
#pragma unroll
    for (int s = 0; s < 2; ++s) load_a<VEC>(xa[s], arow, 16 * s + 8 * half, K);
    store_b(xb, 0);
    __syncthreads();
    for (int c = 0; c < chunks; ++c) {
        const int next = min(c + 1, chunks - 1);
        load_b(xb, next);
#pragma unroll
        for (int s = 0; s < 2; ++s) load_a<VEC>(na[s], arow, next * CK + 16 * s + 8 * half, K);
        __builtin_amdgcn_sched_barrier(0);
        // units of work: a step of 16 k, two tiles of B; the next unit's parts of B are read while one is multiplied
        Parts b[2][2], a;
        auto read_b = [&](int u) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    b[u & 1][t].p[q] = __builtin_bit_cast(bf16x8, stage[c & 1][q][2 * (u / (NT / 2)) + half][32 * (u % (NT / 2) * 2 + t) + l32]);
        };
        auto unit = [&](auto u) {
            constexpr int s = u / (NT / 2), first = u % (NT / 2) * 2;
            if (first == 0) {
                cut_a(xa[s], c * CK + 16 * s + 8 * half, K);
                a = split8(xa[s], minus_low);
            }
            if (u + 1 < NT) read_b(u + 1);
            multiply<first>(acc, small, a, b[u & 1]);
            __builtin_amdgcn_sched_barrier(0);  // (one unit's parts at a time: more would not fit the registers)
        };
        read_b(0);
        unit(std::integral_constant<int, 0>{});
        unit(std::integral_constant<int, 1>{});
        if constexpr (NT > 2) {
            unit(std::integral_constant<int, 2>{});
            unit(std::integral_constant<int, 3>{});
        }
        store_b(xb, (c + 1) & 1);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) xa[s][j] = na[s][j];
    }
    if (row0 >= M) return;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = (acc[t][v] + small[t][v]) * kDown;
    uint32_t again = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        bool bad = false;
#pragma unroll
        for (int v = 0; v < 16; ++v) bad = bad || doubtful(acc[t][v]);
        if (__ballot(bad)) {
            again |= 1u << t;
            continue;
        }
        const int cc = col0 + 32 * t + l32;
        if (cc < N)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t r = row0 + 8 * (v / 4) + 4 * half + v % 4;
                if (r < M) C[r * ldc + cc] = acc[t][v];
            }
    }
    for (; again; again &= again - 1) plain_tile<VEC>(M, N, K, A, lda, B, ldb, C, ldc, row0, col0 + 32 * __builtin_ctz(again));
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
    hipStream_t stream;
};

template <int NT, bool VEC>
void narrow(const Shape& s) {
    hipLaunchKernelGGL((cbm_gemm_narrow_kernel<NT, VEC>), dim3((unsigned)((s.M + 31) / 32)), dim3(256), 0, s.stream, s.M, s.N, s.K, s.A, s.lda, s.B, s.ldb, s.C, s.ldc);
}
template <int NT, bool VEC>
void wide(const Shape& s) {
    const dim3 grid((unsigned)((s.M + 127) / 128), (unsigned)((s.N + 32 * NT - 1) / (32 * NT)));
    hipLaunchKernelGGL((cbm_gemm_wide_kernel<NT, VEC>), grid, dim3(256), 0, s.stream, s.M, s.N, s.K, s.A, s.lda, s.B, s.ldb, s.C, s.ldc);
}
template <bool VEC>
void pick(const Shape& s, int form) {
    switch (form) {
        case 1: return narrow<1, VEC>(s);
        case 2: return narrow<2, VEC>(s);
        case 3: return wide<2, VEC>(s);
        default: return wide<4, VEC>(s);
    }
}

}  // namespace

cbm_status cbm_launch_gemm_split(int64_t M, int32_t N, int32_t K, const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                 int64_t ldc, void* stream, bool* taken) {
    int form = cbm_split_form(M, N, K);
    // (for tests, which run several in one process: 0 = never, 1 to 4 = that kernel; anything else is not listened to)
    if (const char* e = std::getenv("CBM_GEMM_SPLIT"); e && e[0] >= '0' && e[0] <= '4' && !e[1]) form = e[0] - '0';
    if (form == 1 && N > 32) form = 2;
    if (form == 2 && N > 64) form = 3;
    *taken = form != 0;
    if (!form) return CBM_OK;
    const Shape s{M, N, K, A, lda, B, ldb, C, ldc, (hipStream_t)stream};
    const bool vec = K % 4 == 0 && lda % 4 == 0 && ((uintptr_t)A & 15) == 0;
    vec ? pick<true>(s, form) : pick<false>(s, form);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        cbm_set_error_detail("split matmul launch", hipGetErrorString(e));
        return CBM_ERR_HIP;
    }
    return CBM_OK;
}

// Row blocks: products of matrices whose neighbouring rows share most of their columns, on the matrix cores (gfx950, wave64).
//
// The paths of cbm_kernels.hip gather a row of X per delta.  Where 128 alike rows together need few distinct columns, one walk
// over those columns serves all of them: every column's row of X is read once per block and added to the sums of the rows that
// hold it -- a product of a 0/1 matrix (the block's bits) and the gathered rows of X, which is matrix-core work
// (protein recipe: 17.8 columns a row against 77 deltas of the tree and 322 entries; no rounds, no dependent launches).
// X stays 32-bit: a value is split into three bf16 values that add up to it exactly, a bit is exactly 1 in bf16, so the products
// are exact and the sums are 32-bit ones, of the whole row instead of along a path (protein: error against 64 bits 1.2e-7
// in the 2-norm, the paths' 3.7e-7).
//
// One workgroup of four waves has a block and a slab of 32 columns of X (slabs are the slow grid dimension: while one is
// walked, an XCD's share of X is its rows times 128 bytes).  The waves take the block's groups of 64 columns in turn, all of its
// four tiles of 32 rows each, and add their sums through LDS at the end.  A lane loads one column of eight rows of X (one
// 32-bit load a row: two rows of 128 bytes an instruction, 5.7 cycles; 128-bit loads take 16 and bring a lane four columns of
// one row, which is not what a matrix-core operand is) and splits them in registers: they are the B operand of
// v_mfma_f32_32x32x16_bf16 as they stand.  The A operand is a byte of bits through a table in LDS.  Tiles that hold none of a
// step's 16 columns are left out; which ones do comes with the columns (flag_active_tiles).
//
// What bounds it (protein recipe, k = 256; before: 0.79 ms on the paths, now 0.32): matrix cores 36 % and vector ALU 53 % of the
// cycles at a clock that the two bring down to 1.9 GHz; rows of X from L1 instead of L2 change 5 %, no weights or table 3 %.
// A step's instructions add up, whichever unit they go to: with two waves a SIMD instead of three 325 us instead of 290, with twice as many matrix
// instructions 371, with a third of them and no split 211, with rows from L1 260.  So what helps is fewer of them -- row offsets multiplied out once a
// column and tiles known to be empty without looking at their bits 292 -> 284 us (40,000 nodes, k = 32 13.0 -> 12.2, k = 47 18.4 -> 17.7) -- and not another
// arrangement: rows by 128-bit loads turned in LDS 339, the next step's split between the products of this one 318, a table read for active tiles
// only 295, workgroups that walk one block after another 434.
// Measured on the way: 64 columns a slab with scalar loads of the column numbers 0.52 ms (two waves per SIMD, waits for
// scalar loads), blocks of 64 rows 0.46 ms, all tiles without a test 0.51 ms, rows not sorted into tiles 0.41 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "cbm_internal.h"
#include "cbm_split.h"

namespace {

constexpr int WAVES = 4;  // waves per workgroup: they share a block's groups of columns
constexpr int T = CBM_BLOCK_TILES;
static_assert(T == WAVES, "wave s finishes tile s");
constexpr float kUp = CBM_BLOCK_UP, kDown = 1.0f / CBM_BLOCK_UP;

struct BlockMap {
    int64_t begin[CBM_XCD];
    int64_t count[CBM_XCD];
};

template <int MODE, bool BIG>
__global__ __launch_bounds__(64 * WAVES, BIG ? 2 : 3) void cbm_block_kernel(const CbmBlock* __restrict__ blocks, const BlockMap map,
                                                                  const uint32_t* __restrict__ rows,
                                                                  const uint32_t* __restrict__ cols,
                                                                  const float* __restrict__ wcols,
                                                                  const uintx4* __restrict__ masks,
                                                                  const float* __restrict__ X, int64_t ldxb, float* __restrict__ Y,
                                                                  int64_t ldy, const float* __restrict__ rw, float self_w, int k) {
    constexpr bool WCOL = MODE == 1 || MODE == 2 || MODE == 5, WROW = MODE >= 1 && MODE <= 3, RELU = MODE == 2, SELF = MODE == 4;
    __shared__ uintx4 lut[256];
    __shared__ uintx4 ids[WAVES][2][16];
    __shared__ floatx4 wts[WAVES][2][16];
    __shared__ float red[2][WAVES - 1][16][64];
    __shared__ uintx4 tile_rows[WAVES][8];
    __shared__ floatx4 tile_rw[WAVES][8];

    const int xcd = blockIdx.x % CBM_XCD;
    const int64_t nth = blockIdx.x / CBM_XCD;
    if (nth >= map.count[xcd]) return;
    const CbmBlock blk = blocks[map.begin[xcd] + nth];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5;
    {
        const uint32_t b = threadIdx.x;
        uintx4 e;
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ((b >> (2 * i)) & 1u) * 0x3f80u + ((b >> (2 * i + 1)) & 1u) * 0x3f800000u;
        lut[b] = e;
    }
    __syncthreads();
    // The rows of the tile that this wave will store and their weights, one load after the other, are asked for here and kept for the end
    // (k = 256 292 -> 286 us, communities of 1,024 nodes 9.8 -> 9.1).  Rows alone are asked for when the walk is over, beside the reduction: here
    // they cost what they would save (40,000 nodes, k = 32, no weights 13.9 -> 14.6).
    const uint32_t my_row = WROW ? rows[(size_t)blk.row0 + 32 * wave + (lane & 31)] : 0u;
    float my_rw = 0.0f;
    auto ask_weight = [&] {
        if (WROW && my_row != CBM_BLOCK_NO_ROW) my_rw = rw[my_row];
    };
    auto keep_rows = [&] {  // (both halves of the wave write the same)
        if (!WROW) return;
        reinterpret_cast<uint32_t*>(tile_rows[wave])[lane & 31] = my_row;
        reinterpret_cast<float*>(tile_rw[wave])[lane & 31] = my_rw;
    };

    const int lcol = blockIdx.y * 32 + (lane & 31);
    const int ccol = min(lcol, k - 1);  // loads stay inside the row; what they bring is never stored
    auto x_at = [&](uint32_t row) -> float {
        const char* base = reinterpret_cast<const char*>(X);
        if (BIG) return *reinterpret_cast<const float*>(base + (int64_t)row * ldxb + (int64_t)ccol * 4);
        return *reinterpret_cast<const float*>(base + (uint32_t)(__umul24(row, (uint32_t)ldxb) + (uint32_t)ccol * 4u));
    };

    // the same of a row by what stands in LDS for it: where it begins (one multiplication a column there instead of one a load here), or, BIG, its number
    auto x_from = [&](uint32_t at) -> float {
        if (BIG) return x_at(at);
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(X) + (at + (uint32_t)ccol * 4u));
    };

    floatx16 acc[T];
#pragma unroll
    for (int s = 0; s < T; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0.0f;
    uint32_t minus_low = 0xbf80u;
    asm("" : "+s"(minus_low));

    struct Ids {
        uintx4 v[2];
    };
    struct Weights {
        floatx4 v[2];
    };
    // step `st` of the group in buffer `buf`: the eight columns of this half-wave, their weights, their rows of X
    auto read_ids = [&](Ids& i, int buf, int st) {
        i.v[0] = ids[wave][buf][4 * st + 2 * half];
        i.v[1] = ids[wave][buf][4 * st + 2 * half + 1];
    };
    auto read_weights = [&](Weights& w, int buf, int st) {
        if (!WCOL) return;
        w.v[0] = wts[wave][buf][4 * st + 2 * half];
        w.v[1] = wts[wave][buf][4 * st + 2 * half + 1];
    };
    auto load_x = [&](float (&x)[8], const Ids& i) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = x_from(i.v[j / 4][j % 4]);
    };
    auto consume = [&](float (&x)[8], const Weights& w, uint32_t mask, uint32_t active) {
        uintx4 a[T];
#pragma unroll
        for (int s = 0; s < T; ++s) a[s] = lut[(mask >> (8 * s)) & 255u];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] *= WCOL ? w.v[j / 4][j % 4] : kUp;  // (the weights come times kUp)
        uintx4 P[3];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            uint32_t h, m, l;
            split_pair(x[2 * p], x[2 * p + 1], minus_low, h, m, l);
            P[0][p] = h;
            P[1][p] = m;
            P[2][p] = l;
        }
#pragma unroll
        for (int s = 0; s < T; ++s)
            // (a scalar: six vector instructions a step that looked at the bits are gone; nearly all tiles of hub blocks are active, and with weights, MODE 5, they
            // would lose 1 % by it: those without are MODE 0, as row blocks, and lose half of that, R-MAT scale 20, k = 64 104.9 -> 105.2 us)
            if (MODE == 5 ? __ballot(((mask >> (8 * s)) & 255u) != 0) != 0 : (active >> s & 1u) != 0) {
#pragma unroll
                for (int q = 2; q >= 0; --q)
                    acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[s]), __builtin_bit_cast(bf16x8, P[q]), acc[s], 0, 0, 0);
            }
    };
    if ((uint32_t)wave < blk.ngroups) {
        // every load is made, with the group held to this wave's last: a load that may not happen would turn the wait for an
        // older one into a wait for all of them
        const uint32_t last = blk.ngroups - 1 - (blk.ngroups - 1 - wave) % WAVES;
        const uint32_t* gc = cols + (size_t)blk.group0 * 64 + lane;
        const float* gw = wcols + (size_t)blk.group0 * 64 + lane;
        const uintx4* gm = masks + (size_t)blk.group0 * 64 + lane;
        auto put = [&](int buf, uint32_t id, float w) {
            reinterpret_cast<uint32_t*>(ids[wave][buf])[lane] = BIG ? id & ~CBM_BLOCK_ACTIVE : __umul24(id, (uint32_t)ldxb);
            if (WCOL) reinterpret_cast<float*>(wts[wave][buf])[lane] = w;
        };
        // (three buffers of rows in flight besides the one in use would cost a wave per SIMD; four names, three alive)
        float x[4][8];
        Ids i;
        Weights w0, w1;
        uint32_t g = wave;
        size_t at = (size_t)g * 64, next = (size_t)min(g + WAVES, last) * 64;
        uintx4 mask = gm[at];
        uint32_t nid = gc[at];
        uint32_t active = (uint32_t)__ballot(nid & CBM_BLOCK_ACTIVE), nactive = active;
        put(0, nid, WCOL ? gw[at] : 0.0f);
        nid = gc[next];
        float nw = WCOL ? gw[next] : 0.0f;
        uintx4 nmask = gm[next];
        ask_weight();
        read_ids(i, 0, 0);
        load_x(x[0], i);
        read_ids(i, 0, 1);
        load_x(x[1], i);
        keep_rows();
        read_ids(i, 0, 2);
        read_weights(w0, 0, 0);
        int buf = 0;
        for (;;) {
            // a step: rows of X two steps ahead, columns three, weights one
            load_x(x[2], i);
            read_ids(i, buf, 3);
            read_weights(w1, buf, 1);
            __builtin_amdgcn_sched_barrier(0);
            consume(x[0], w0, mask[0], active);

            load_x(x[3], i);
            put(buf ^ 1, nid, nw);
            nactive = (uint32_t)__ballot(nid & CBM_BLOCK_ACTIVE);
            next = (size_t)min(g + 2 * WAVES, last) * 64;
            nid = gc[next];
            if (WCOL) nw = gw[next];
            read_ids(i, buf ^ 1, 0);
            read_weights(w0, buf, 2);
            __builtin_amdgcn_sched_barrier(0);
            consume(x[1], w1, mask[1], active >> 4);

            load_x(x[0], i);
            read_ids(i, buf ^ 1, 1);
            read_weights(w1, buf, 3);
            __builtin_amdgcn_sched_barrier(0);
            consume(x[2], w0, mask[2], active >> 8);

            load_x(x[1], i);
            read_ids(i, buf ^ 1, 2);
            read_weights(w0, buf ^ 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            consume(x[3], w1, mask[3], active >> 12);

            if (g == last) break;
            g += WAVES;
            buf ^= 1;
            mask = nmask;
            active = nactive;
            nmask = gm[next];
        }
    } else {
        ask_weight();
        keep_rows();
    }

    // The waves' shares of a tile, added by the wave that will store it (wave s has tile s), two tiles at a time.
    uintx4 row4[4];  // rows 8 q + 4 half .. + 3 of the wave's tile
    if (!WROW) {
#pragma unroll
        for (int q = 0; q < 4; ++q) row4[q] = reinterpret_cast<const uintx4*>(rows + (size_t)blk.row0 + 32 * wave)[2 * q + half];
    }
    floatx16 fin;
#pragma unroll
    for (int pair = 0; pair < 2; ++pair) {
        if (pair) __syncthreads();
#pragma unroll
        for (int s = 2 * pair; s < 2 * pair + 2; ++s)
            if (wave != s) {
#pragma unroll
                for (int v = 0; v < 16; ++v) red[s & 1][wave < s ? wave : wave - 1][v][lane] = acc[s][v];
            }
        __syncthreads();
#pragma unroll
        for (int s = 2 * pair; s < 2 * pair + 2; ++s)
            if (wave == s) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    fin[v] = (acc[s][v] + red[s & 1][0][v][lane] + red[s & 1][1][v][lane] + red[s & 1][2][v][lane]) * kDown;
            }
    }
    auto store = [&](uint32_t row, float w, float v) {
        if (SELF) v = fmaf(self_w, x_at(row), v);
        if (WROW) v *= w;
        if (RELU) v = fmaxf(v, 0.0f);
        __builtin_nontemporal_store(v, Y + (int64_t)row * ldy + lcol);
    };
    // No bf16 value has bits below 2^-133, and the matrix cores take what is below 2^-126 for zero: x (times its weight) is split at
    // 2^24 times its size, where the smallest 32-bit value is 2^-125, so nothing is lost and a sum of zero is zero.
    // What does not come out that way is 0 x infinity: a value that is not finite (or not any more at that size: from 2^104)
    // anywhere among the block's rows of X turns every sum of its column in this tile into NaN.  A tile with a sum that is not
    // finite is summed again by its wave, with large values at another size in sums of their own and infinities and NaN counted (protein
    // recipe, k = 256: 0.33 ms; with one infinity in X 0.34, every 20th row the type's lowest value 2.1, all of X NaN 1.9; a walk that
    // selects entry by entry took 0.51, 5.1 and 5.2).
    bool plain = true;
#pragma unroll
    for (int v = 0; v < 16; ++v) plain = plain && fabsf(fin[v]) < INFINITY;
    if (__ballot(!plain)) {
        constexpr float kLarge = 0x1p88f;  // below it 4,096 values (a block's most) add up to less than 2^100
        floatx16 sum, large, up, down;     // up: infinities and NaN, down: minus infinities and NaN
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v] = large[v] = up[v] = down[v] = 0.0f;
        auto add = [&](floatx16& to, const float (&x)[8], const uintx4& bits) {
            uintx4 P[3];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t h, m, l;
                split_pair(x[2 * p], x[2 * p + 1], minus_low, h, m, l);
                P[0][p] = h;
                P[1][p] = m;
                P[2][p] = l;
            }
#pragma unroll
            for (int q = 2; q >= 0; --q)
                to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bits), __builtin_bit_cast(bf16x8, P[q]), to, 0, 0, 0);
        };
        auto count = [&](floatx16& to, const float (&x)[8], float which, const uintx4& bits) {
            uintx4 ones;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const bool lo = x[2 * p] == which || x[2 * p] != x[2 * p], hi = x[2 * p + 1] == which || x[2 * p + 1] != x[2 * p + 1];
                ones[p] = (lo ? 0x3f80u : 0u) | (hi ? 0x3f800000u : 0u);
            }
            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bits), __builtin_bit_cast(bf16x8, ones), to, 0, 0, 0);
        };
        // 16 columns a step, eight for each half of the wave; rows of X one step ahead, columns, bits and weights two
        const int last = 4 * (int)blk.ngroups - 1;
        const uintx4* gc = reinterpret_cast<const uintx4*>(cols + (size_t)blk.group0 * 64 + 8 * half);
        const floatx4* gw = reinterpret_cast<const floatx4*>(wcols + (size_t)blk.group0 * 64 + 8 * half);
        const uint32_t* gm = reinterpret_cast<const uint32_t*>(masks + (size_t)blk.group0 * 64 + lane);
        Ids ci;
        Weights w, nw;
        uint32_t held, nheld;
        float nx[8];
        auto fetch = [&](int i) {
            ci.v[0] = gc[4 * i];
            ci.v[1] = gc[4 * i + 1];
            if (WCOL) {
                nw.v[0] = gw[4 * i];
                nw.v[1] = gw[4 * i + 1];
            }
            nheld = gm[(size_t)(i / 4) * 256 + i % 4] >> (8 * wave) & 255u;
        };
        auto load_next = [&] {
#pragma unroll
            for (int j = 0; j < 8; ++j) nx[j] = x_at(ci.v[j / 4][j % 4] & ~CBM_BLOCK_ACTIVE);
        };
        fetch(0);
        load_next();
        w = nw;
        held = nheld;
        fetch(min(1, last));
        for (int i = 0; i <= last; ++i) {
            float x[8], y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = WCOL ? nx[j] * (w.v[j / 4][j % 4] * kDown) : nx[j];
            const uintx4 bits = lut[held];
            load_next();
            w = nw;
            held = nheld;
            fetch(min(i + 2, last));
            bool any_small = false, any_large = false, any_other = false;  // (one kind at a time is the rule: leave out the rest)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                any_small = any_small || fabsf(x[j]) < kLarge;
                any_large = any_large || (fabsf(x[j]) >= kLarge && fabsf(x[j]) < INFINITY);
                any_other = any_other || !(fabsf(x[j]) < INFINITY);
            }
            if (__ballot(any_small)) {
#pragma unroll
                for (int j = 0; j < 8; ++j) y[j] = fabsf(x[j]) < kLarge ? x[j] * kUp : 0.0f;
                add(sum, y, bits);
            }
            if (__ballot(any_large)) {
#pragma unroll
                for (int j = 0; j < 8; ++j) y[j] = fabsf(x[j]) >= kLarge && fabsf(x[j]) < INFINITY ? x[j] * kDown : 0.0f;
                add(large, y, bits);
            }
            if (__ballot(any_other)) {
                count(up, x, INFINITY, bits);
                count(down, x, -INFINITY, bits);
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            fin[v] = fmaf(large[v], kUp, sum[v] * kDown);
            if (up[v] > 0.0f) fin[v] = INFINITY;
            if (down[v] > 0.0f) fin[v] = up[v] > 0.0f ? NAN : -INFINITY;
        }
    }
    // register v of lane l of a 32 x 32 tile: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
    if (lcol < k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uintx4 row = row4[q];
            floatx4 w;
            if (WROW) {
                row = tile_rows[wave][2 * q + half];
                w = tile_rw[wave][2 * q + half];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (row[v] != CBM_BLOCK_NO_ROW) store(row[v], WROW ? w[v] : 1.0f, fin[4 * q + v]);
        }
    }
}

constexpr int kMostSlabs = 65535;  // a grid's second dimension: wider X (from 2,097,120 columns) takes several launches

struct Args {
    const cbm_handle* h;
    const float* X;
    int64_t ldx;
    int k;
    float* Y;
    int64_t ldy;
    const float* rw;
    float self_w;
    hipStream_t stream;
};

template <int MODE, bool BIG>
void launch(const Args& a) {
    BlockMap map;
    int64_t most = 0;
    for (int j = 0; j < CBM_XCD; ++j) {
        map.begin[j] = a.h->blk_begin[j];
        map.count[j] = a.h->blk_count[j];
        most = std::max(most, map.count[j]);
    }
    for (int c = 0; c < a.k; c += kMostSlabs * 32) {
        const int k = std::min(a.k - c, kMostSlabs * 32);
        hipLaunchKernelGGL((cbm_block_kernel<MODE, BIG>), dim3((unsigned)(CBM_XCD * most), (unsigned)((k + 31) / 32)), dim3(64 * WAVES), 0, a.stream,
                           a.h->d_blocks, map, a.h->d_block_rows, a.h->d_block_cols, a.h->d_block_w,
                           reinterpret_cast<const uintx4*>(a.h->d_block_masks), a.X + c, a.ldx * 4, a.Y + c, a.ldy, a.rw, a.self_w, k);
        if (a.k - c <= kMostSlabs * 32) break;  // (the next c may not be an int)
    }
}
template <bool BIG>
void launch_mode(const Args& a, int mode) {
    switch (mode) {
        case 0: return launch<0, BIG>(a);
        case 1: return launch<1, BIG>(a);
        case 2: return launch<2, BIG>(a);
        case 3: return launch<3, BIG>(a);
        case 4: return launch<4, BIG>(a);
        default: return launch<5, BIG>(a);
    }
}

void launch_size(const Args& a, int mode) {
    // 24-bit indices and 32-bit offsets where they reach: one instruction per address
    const int64_t n = std::max(a.h->n, a.h->m);
    const bool big = n >= (1 << 24) || a.ldx >= (1 << 22) || n * a.ldx * 4 >= (int64_t)UINT32_MAX;
    big ? launch_mode<true>(a, mode) : launch_mode<false>(a, mode);
}

}  // namespace

void cbm_launch_blocks(const cbm_handle* h, const float* X, int64_t ldx, int32_t k, float* Y, int64_t ldy, int mode, const float* rw,
                       float self_w, void* stream) {
    launch_size({h, X, ldx, k, Y, ldy, rw, self_w, (hipStream_t)stream}, mode);
}

void cbm_launch_hub_blocks(const cbm_handle* h, const float* X, int64_t ldx, int32_t k, float* scratch, int64_t ld_scratch, bool weighted,
                           void* stream) {
    launch_size({h, X, ldx, k, scratch, ld_scratch, nullptr, 0.0f, (hipStream_t)stream}, weighted ? 5 : 0);
}

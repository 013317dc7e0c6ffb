// Which dense products hold B in registers (cbm_gemm_held.hip) and how their waves share K; which of the others go through bf16 parts (cbm_gemm_split.hip).
#pragma once

#include <algorithm>
#include <cstdint>

// Panels of up to 64 columns, tiles of 16 columns in each, steps of 32 that K has, waves that share K (0: K is deeper than they can hold), steps of each.
struct CbmHeldPlan {
    int panels, tiles, steps, slices, each;
};
// Steps of 32 k that a wave can hold beside so many tiles of 16 columns: 12 registers each.
constexpr int cbm_held_most_steps(int tiles) { return tiles == 4 ? 3 : 4; }

// How many waves share K: those that pad it least and, of these, as few as there are (132534 x 100 . 100 x 47, 4 steps: one wave 20, four 23; 20000 x 256 .
// 256 x 47, 8 steps: four 8.1, eight 8.6) with no more than two steps each (x 16 one wave 13.7, four 11.4; 20000 x 500 . 500 x 47, 16 steps: four 13.9, eight
// 12.1), three tiles of columns up to 50,000 rows only (50000 x 128 . 128 x 47 one wave 13.4, four 12.6; 80000 rows 15.7, 16.4).  Two waves are for 5 or 6
// steps (250000 x 150 . 150 x 24 four 61, two 41).  Where there are not rows enough for all waves, as many as K takes: 8192 x 128 . 128 x 47 one wave 7.1, four
// 5.4, 5000 x 320 . 320 x 32 four 6.7, eight 6.1 (12,000 rows: 7.2, 7.8).  (Measured with six products of parts instead of eight.)
inline CbmHeldPlan cbm_held_plan(int64_t M, int32_t N, int32_t K) {
    CbmHeldPlan p{};
    p.panels = (N + 63) / 64;
    p.tiles = ((N + 15) / 16 + p.panels - 1) / p.panels;
    p.steps = (int)(((int64_t)K + 31) / 32);
    const int most = cbm_held_most_steps(p.tiles), enough = M <= 8192 ? 1 : p.tiles <= 2 || M <= 50000 ? 2 : most;
    for (int n : {1, 2, 4, 8}) {
        const int e = (p.steps + n - 1) / n;
        if (e > most || (p.slices && (p.each <= enough || (M > 8192 && n * e > p.slices * p.each)))) continue;
        p.slices = n;
        p.each = e;
    }
    return p;
}

// Where the lines lie, from 16,500 products of both (M from 500 to 300,000, K from 8 to 1,000, N from 2 to 256; us, the other kernels / these, in one
// process and in turn; where these are taken they are ahead by a third on average, and 0.6 % of the products inside the lines are slower by 5 % or more).
// `vec`: K is a multiple of 4 and rows of A start on 16-byte boundaries, which these kernels need more than the others.  What costs them is padding, of K to whole
// steps for each wave (33 to 64, 160 to 192), and panels, each of which splits A again; 32,768 and 65,536 rows suit the others best, whose waves then are all alike.
//
// Up to 64 columns:
//  K <= 32 and 33 to 48 columns: the staged kernel has tiles of that width (4096 x 32 . 32 x 48 3.2 / 3.7; from 8,192 rows on the panel kernel takes an aligned B,
//    6.2 / 3.8);  rows off 16-byte boundaries: 55803 x 15 . 15 x 24 5.3 / 6.8, 45071 x 13 . 13 x 40 5.8 / 6.4, 37443 x 23 . 23 x 64 ahead by 1.18;
//  K <= 96 off 16-byte boundaries: 28000 x 33 . 33 x 32 5.5 / 6.6, 50000 rows and 16 columns 6.9 / 8.6, 40000 x 61 ahead by 1.1, few rows or many by more;
//  5 steps padded to 6: 32768 x 160 . 160 x 8 7.0 / 8.5;  two tiles, and two steps too many: 65536 x 400 . 400 x 32 22 / 26.
// Two panels, up to 65,536 rows: the others are workgroups of 128 rows and 64 columns that split both operands (cbm_gemm_split.hip), in rounds of one for each
// compute unit; the two estimates below are least-squares fits (2,400 products, 5 and 6 % off), 5 % apart to be taken.  32768 x 160 . 160 x 128 15.1 / 19.0, 36000
// rows, K = 192 and 112 columns 22.6 / 19.6, 20000 x 500 . 500 x 112 34 / 23.  More rows: 128 columns leave the others nothing to pad (100000 x 256 . 256 x 128 59 / 50, 300000 rows
// 158 / 166, K = 400 232 / 277); 65 to 80 and 97 to 112 columns lose where K is deep and padded (200000 x 400 . 400 x 80 131 / 148), 81 to 96 gain (229 / 148).
// Three and four panels: K <= 32, where C is most of the traffic (300000 x 32 . 32 x 128 67 / 36, x 256 141 / 115, 20000 x 8 . 8 x 192 15 / 8), and few rows (2000 x 500 .
// 500 x 256 22 / 8.7).
// Below K = 8 a product is a few roundings, which the fp32 kernels make no fewer of than needed: theirs.
inline bool cbm_held_takes(int64_t M, int32_t N, int32_t K, bool vec) {
    if (K < 8 || N > 256) return false;
    const CbmHeldPlan p = cbm_held_plan(M, N, K);
    if (!p.slices) return false;
    const int padded = p.slices * p.each;  // steps
    if (N <= 64) {
        const bool between = M > 32768 && M <= 65536, full = between && M > 61440;
        if (K <= 32) {
            if (p.tiles == 3 && M < (N % 4 == 0 ? 8192 : 16385)) return false;
            return vec || !between || p.tiles == 4 || (p.tiles == 1 && !full);
        }
        if (K <= 96) return vec || M <= (p.tiles == 1 ? 16384 : 8192) || M > 65536 || ((M <= 16384 || (between && !full)) && 2 * 32 * padded <= 3 * K);
        if (p.tiles == 1 && p.steps == 5 && vec && N % 4 == 0) return M <= 24576 || M > 32768;
        return !(p.tiles == 2 && p.steps > 8 && padded > p.steps + 1 && vec && M > 50000 && M <= 65536);
    }
    if (K <= 32) return vec || (N > 80 && (N <= 192 || M <= 200000));  // (170000 x 30 . 30 x 66 20 / 24, 250000 x 30 . 30 x 250 85 / 93)
    if (N > 128) return M <= 2048;
    if (M <= 8192) return true;
    if (M <= 65536) {
        const double rows = 1e-3 * (double)M, rounds = (double)(((M + 127) / 128 * 2 + 255) / 256);
        double here = 6.2 + rows * (p.tiles == 4 ? 0.057 + 0.048 * padded : 0.012 + 0.0418 * padded), there = std::max(3.4 + 1.13 * p.steps, 5.6);
        there += (rounds - 1) * 0.7 * p.steps + 0.09 * rows;
        if (p.slices == 8) here += 0.4;
        if (p.slices == 1 && padded == 3) here += 0.09 * rows;
        if (!vec) {
            here += 0.007 * padded * rows;
            there += (0.85 * p.steps - 0.15) * rounds;
        }
        return here <= 0.95 * there;
    }
    if (K < 96 || !vec || (N > 80 && N <= 96)) return true;
    if (N > 116) return M <= (padded == p.steps ? 250000 : 110000) && padded < p.steps + 3;
    return K < 260 || padded == p.steps || (N > 80 && N % 4 != 0) || (K <= 512 && M <= 110000);
}

// Where the lines lie (microseconds, fp32 kernels of cbm_gemm.hip -> those of cbm_gemm_split.hip; M x K . K x N), for products that do not hold B in registers.  Measured at M from 1,000 to 132,534, K from
// 32 to 1,000 and 20 widths: nowhere inside the lines are they slower by more than the launch's own noise; some outside would be faster.
//  up to 64 columns (what is left: K beyond 768 or 1,024, and a few products that it would pad most): short and deep products, which leave the chip idle there -- 19717 x 500 . 500 x 64 26.1 -> 21.0, . 500 x 7
//    25.2 -> 13.4, 24000 x 128 . 128 x 64 13.0 -> 10.3, 3000 x 512 . 512 x 64 24 -> 10.  The line in M: at 28,000 rows the two are level
//    (200 x 64: 17.2, 16.6; 500 x 64: 27.0, 27.4), at 60,000 the fp32 kernels stream A at the rate of memory (200 x 64: 25.7, 28.6; 500 x 64:
//    42, 48; 500 x 32: 25.7, 31.1), and what lies between depends on N (40000 x 500 . 500 x 7: 40, 22).  The line in K: at 100 24,576 rows
//    gain (12.2, 10.4), at 64 they lose (9.0, 9.9);
//  more columns, few workgroups (tiles of 64 columns): 19717 x 256 . 256 x 256 42 -> 28, 6000 x 300 . 300 x 96 28 -> 15, 4000 x 96 . 96 x 96
//    11 -> 8 (K = 32: level);
//  more columns, many: 132534 x 256 . 256 x 256 156 -> 130, 132534 x 96 . 96 x 256 89 -> 66, 132534 x 250 . 250 x 250 234 -> 182,
//    if the last tile of 128 columns is not mostly padding (256 x 160: 105, 134) and K is not so short that the
//    products are bound by memory (132534 x 64 . 64 x 128: 32, 33).
// (0: the fp32 kernels; 1 to 4: one of the kernels there.)
inline int cbm_split_form(int64_t M, int32_t N, int32_t K) {
    if (N <= 64) return M <= 24576 && K >= 128 ? (N <= 32 ? 1 : 2) : 0;
    if ((M + 127) / 128 * ((N + 63) / 64) <= 1024) return K >= 32 ? 3 : 0;
    return K >= 96 && (N + 127) / 128 * 128 * 10 <= (int64_t)N * 11 ? 4 : 0;
}

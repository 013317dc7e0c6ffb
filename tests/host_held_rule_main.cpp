// Which dense products hold B in registers, and how waves share K there: against products that were measured with these kernels and with the others.
// Run by test_held_rule_host.py.
#include <cstdio>

#include "cbm_gemm_rules.h"

struct Measured {
    int64_t m;
    int k, n, vec;
    double others, held;  // us
};
// at least 8 % apart, on both sides of the lines
constexpr Measured kMeasured[] = {
    {4096, 32, 48, 1, 3.24, 3.68},    {8192, 32, 48, 1, 6.15, 3.79},    {4096, 32, 64, 1, 4.60, 4.13},     {55803, 15, 24, 0, 5.26, 6.78},   {37443, 23, 64, 0, 7.80, 6.59},
    {50000, 33, 16, 0, 6.85, 8.59},   {28000, 33, 32, 0, 5.49, 6.55},   {12000, 33, 8, 0, 5.02, 3.79},     {300000, 33, 16, 0, 23.05, 16.62},  {65536, 95, 14, 0, 10.99, 12.76},
    {32768, 160, 8, 1, 6.99, 8.46},   {36000, 160, 16, 1, 10.97, 9.12}, {65536, 400, 32, 1, 21.96, 25.99}, {36000, 400, 32, 1, 20.22, 16.57}, {132534, 100, 47, 1, 26.3, 20.9},
    {32768, 160, 128, 1, 15.09, 18.95}, {32768, 80, 128, 1, 11.51, 13.00}, {20000, 80, 96, 1, 9.67, 10.46}, {36000, 192, 112, 1, 22.55, 19.58}, {20000, 500, 112, 1, 33.58, 22.87},
    {50000, 100, 80, 1, 21.82, 16.02}, {8192, 256, 128, 1, 13.18, 8.57}, {300000, 400, 128, 1, 232.1, 277.3}, {100000, 256, 128, 1, 59.35, 49.61}, {300000, 640, 128, 1, 348.5, 380.9},
    {200000, 400, 80, 1, 131.1, 148.2}, {200000, 400, 96, 1, 229.2, 148.5}, {132534, 64, 128, 1, 31.88, 26.17},  {300000, 32, 128, 1, 67.7, 37.3}, {300000, 32, 256, 1, 139.4, 115.9},
    {2000, 500, 256, 1, 21.75, 8.90},  {20000, 400, 160, 1, 28.84, 32.49},
};

int main() {
    for (const Measured& x : kMeasured)
        if (cbm_held_takes(x.m, x.n, x.k, x.vec) != (x.held < x.others))
            return std::printf("%lld x %d . %d x %d: others %.2f us, B in registers %.2f\n", (long long)x.m, x.k, x.k, x.n, x.others, x.held), 1;
    for (int64_t m : {1, 8192, 8193, 50000, 50001, 300000})
        for (int n = 1; n <= 256; ++n)
            for (int k = 1; k <= 1100; ++k) {
                const CbmHeldPlan p = cbm_held_plan(m, n, k);
                const bool whole = p.panels * p.tiles * 16 >= n && p.tiles <= 4 && (p.panels - 1) * p.tiles * 16 < n;
                const bool deep = (k + 31) / 32 > 8 * cbm_held_most_steps(p.tiles);
                const bool fits = p.slices * p.each * 32 >= k && p.each >= 1 && p.each <= cbm_held_most_steps(p.tiles) && !(p.slices & (p.slices - 1)) && p.slices <= 8;
                if (!whole || p.steps != (k + 31) / 32 || (p.slices == 0) != deep || (p.slices && !fits))
                    return std::printf("plan of %lld x %d . %d x %d\n", (long long)m, k, k, n), 1;
                if (cbm_held_takes(m, n, k, k % 4 == 0) && (deep || k < 8)) return std::puts("takes what it cannot hold"), 1;
            }
    if (cbm_held_takes(1000, 257, 64, true)) return std::puts("more than four panels"), 1;
    std::puts("held rule ok");
    return 0;
}

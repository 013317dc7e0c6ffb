// Which tiles of a step hold any of its columns, as the device gets it in bit 31 of the columns: against the bits themselves.
#include <cstdio>
#include <random>

#include "cbm_block_plan.h"

int main() {
    std::mt19937 rng(7);
    for (size_t groups : {0, 1, 2, 37})
        for (int density : {0, 1, 40, 1000}) {  // of 1000 bits
            std::vector<uint32_t> cols(groups * 64), masks(groups * 256, 0);
            for (uint32_t& c : cols) c = rng() & 0x1fffffffu;
            for (uint32_t& w : masks)
                for (int b = 0; b < 32; ++b) w |= (uint32_t)((int)(rng() % 1000) < density) << b;
            const std::vector<uint32_t> got = flag_active_tiles(cols, masks);
            if (got.size() != cols.size()) return std::puts("size"), 1;
            for (size_t at = 0; at < got.size(); ++at) {
                bool active = false;
                if (at % 64 < 16)
                    for (int l = 0; l < 64; ++l) active = active || (masks[at / 64 * 256 + 4 * l + at % 64 / 4] >> (8 * (at % 4)) & 255u);
                if (got[at] != (cols[at] | (active ? CBM_BLOCK_ACTIVE : 0u))) return std::puts("flag"), 1;
            }
        }
    std::puts("active tiles ok");
}

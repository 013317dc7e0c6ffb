// The grid of dense products in panels of columns side by side: never more workgroups than run at once, each panel's on the XCDs of the others'.
// Run by test_panel_blocks_host.py.
#include <cstdio>

#include "cbm_internal.h"

int main() {
    for (int64_t resident : {256, 512, 1024, 2048})
        for (int panels = 1; panels <= 4; ++panels)
            for (int64_t wanted : {1, 7, 8, 9, 63, 85, 88, 125, 340, 341, 344, 1000, 5000, 100000}) {
                const int64_t each = cbm_panel_blocks(wanted, panels, resident);
                const bool enough = each >= 1 && (each >= wanted || (each + 8) * panels > resident);
                if (!enough || each * panels > resident || (panels > 1 && each % CBM_XCD) || each > wanted + 7)
                    return std::printf("%lld of %lld wanted, %d panels: %lld each\n", (long long)resident, (long long)wanted, panels, (long long)each), 1;
            }
    std::puts("panel blocks ok");
    return 0;
}

// The row blocks of small square matrices, decoded again: every entry of the matrix once, every row in one place, every
// index in range, every XCD's run of blocks disjoint.  Built with ASan/UBSan by test_row_blocks_host.py.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>
#include "cbm_internal.h"
void cbm_set_error_detail(const char*, const char*) {}
cbm_status cbm_device_candidates(int, int64_t, int64_t, const int64_t*, const int32_t*, const int64_t*, const int32_t*, int64_t,
                                 int64_t, int32_t, std::vector<int32_t>*, std::vector<int32_t>*, std::vector<int32_t>*) {
    return CBM_ERR_STATE;
}
cbm_status cbm_device_deltas(int, int64_t, const int64_t*, const int32_t*, const int32_t*, std::vector<int32_t>*, std::vector<int32_t>*,
                             std::vector<int64_t>*, std::vector<uint32_t>*) {
    return CBM_ERR_STATE;
}
const char* cbm_get_error_detail() { return ""; }

static int fail(const char* what, int trial) {
    std::printf("trial %d: %s\n", trial, what);
    return 1;
}

int main() {
    setenv("CBM_ROW_BLOCKS", "1", 1);
    std::mt19937 rng(7);
    const int sizes[] = {1, 2, 31, 32, 33, 127, 128, 129, 255, 257, 700, 1500};
    int trial = 0;
    for (int m : sizes)
        for (int form = 0; form < 4; ++form, ++trial) {
            std::vector<int64_t> rp(m + 1, 0);
            std::vector<int32_t> ci;
            for (int i = 0; i < m; ++i) {  // form 0: near the diagonal; 1: anywhere, with empty rows; 2: one full row; 3: directed chain
                std::set<int> s;
                if (form == 0)
                    for (int c = std::max(0, i - 9); c < std::min(m, i + 10); ++c) s.insert(c);
                if (form == 1 && i % 3)
                    for (int c = 0; c < 6; ++c) s.insert(rng() % m);
                if (form == 2 && (i == m / 2 || i % 5 == 0))
                    for (int c = 0; c < (i == m / 2 ? m : 1); ++c) s.insert(i == m / 2 ? c : (int)(rng() % m));
                if (form == 3 && i + 1 < m) s.insert(i + 1);
                ci.insert(ci.end(), s.begin(), s.end());
                rp[i + 1] = (int64_t)ci.size();
            }
            cbm_handle h;
            h.opts = cbm_build_opts{};
            h.opts.add_self_loops = trial % 2;
            h.opts.num_threads = 1 + trial % 3;
            h.opts.flags = CBM_FLAG_HOST_ONLY | (trial % 5 == 4 ? CBM_FLAG_TRANSPOSE : 0u);
            if (cbm_build_host(m, m, rp.data(), ci.data(), &h) != CBM_OK) return fail("build failed", trial);
            std::vector<int64_t> orp(m + 1);
            std::vector<int32_t> oci(h.stats.nnz + 1);
            if (cbm_decompress_host(&h, orp.data(), oci.data()) != CBM_OK) return fail("decompress failed", trial);
            if (h.row_blocks.size() != (size_t)(m + CBM_BLOCK_ROWS - 1) / CBM_BLOCK_ROWS) return fail("number of blocks", trial);
            if (h.block_rows.size() != h.row_blocks.size() * CBM_BLOCK_ROWS) return fail("places for rows", trial);
            std::vector<std::set<int>> got(m);
            std::vector<int> placed(m, 0), in_share(h.row_blocks.size(), 0);
            for (int j = 0; j < CBM_XCD; ++j)
                for (int64_t b = h.blk_begin[j]; b < h.blk_begin[j] + h.blk_count[j]; ++b) {
                    if (b < 0 || b >= (int64_t)h.row_blocks.size()) return fail("share out of range", trial);
                    ++in_share[b];
                }
            for (int c : in_share)
                if (c != 1) return fail("a block in no share, or in two", trial);
            for (const CbmBlock& b : h.row_blocks) {
                if (b.row0 + CBM_BLOCK_ROWS > h.block_rows.size() || (size_t)(b.group0 + b.ngroups) * 64 > h.block_cols.size() ||
                    (size_t)(b.group0 + b.ngroups) * 256 > h.block_masks.size())
                    return fail("block out of range", trial);
                for (int i = 0; i < CBM_BLOCK_ROWS; ++i) {
                    const uint32_t row = h.block_rows[b.row0 + i];
                    if (row != CBM_BLOCK_NO_ROW && (row >= (uint32_t)m || placed[row]++)) return fail("row placed twice or out of range", trial);
                }
                for (uint32_t g = b.group0; g < b.group0 + b.ngroups; ++g)
                    for (int p = 0; p < 64; ++p) {
                        const uint32_t col = h.block_cols[(size_t)g * 64 + p];
                        if (col >= (uint32_t)m) return fail("column out of range", trial);
                        for (int i = 0; i < CBM_BLOCK_ROWS; ++i) {
                            const uint32_t word = h.block_masks[(size_t)g * 256 + 4 * (i % 32 + 32 * (p % 16 / 8)) + p / 16];
                            if (!(word >> (8 * (i / 32) + p % 8) & 1u)) continue;
                            const uint32_t row = h.block_rows[b.row0 + i];
                            if (row == CBM_BLOCK_NO_ROW || !got[row].insert((int)col).second) return fail("entry twice or in no row", trial);
                        }
                    }
            }
            for (int i = 0; i < m; ++i)
                if (placed[i] != 1 || !std::equal(got[i].begin(), got[i].end(), oci.begin() + orp[i], oci.begin() + orp[i + 1]))
                    return fail("a row differs", trial);
        }
    std::puts("blocks ok");
    return 0;
}

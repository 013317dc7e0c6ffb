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

// Hub blocks: what the blocks hold of the split rows and what is left of them add up to the matrix, every scratch row is written
// once, and the combine list finds a row's parts side by side.
static int hubs() {
    setenv("CBM_ROW_BLOCKS", "0", 1);
    setenv("CBM_HUB_BLOCKS", "2", 1);
    setenv("CBM_SPLIT_MIN", "128", 1);
    std::mt19937 rng(11);
    int trial = 0, with = 0;
    for (int m : {40, 300, 1500})
        for (int n : {m, 900, 2500})
            for (int form = 0; form < 4; ++form, ++trial) {
                setenv("CBM_HUB_LEAST", form % 2 ? "2" : "4", 1);
                setenv("CBM_HUB_PIECE", form == 3 ? "1" : "3", 1);
                setenv("CBM_REST_WHOLE", form == 2 ? "0" : "96", 1);
                std::vector<int64_t> rp(m + 1, 0);
                std::vector<int32_t> ci;
                for (int i = 0; i < m; ++i) {
                    std::set<int> s;
                    const int len = i % 3 == 0 ? 150 + (int)(rng() % 500) : (int)(rng() % 20);
                    for (int c = 0; c < len; ++c) {
                        const double u = (rng() % 10000) / 10000.0;
                        s.insert((int)((n - 1) * u * u * u));  // popular columns first
                    }
                    ci.insert(ci.end(), s.begin(), s.end());
                    rp[i + 1] = (int64_t)ci.size();
                }
                cbm_handle h;
                h.opts = cbm_build_opts{};
                h.opts.add_self_loops = m == n && trial % 2;
                h.opts.num_threads = 1 + trial % 3;
                h.opts.flags = CBM_FLAG_HOST_ONLY;
                if (cbm_build_host(m, n, rp.data(), ci.data(), &h) != CBM_OK) return fail("hubs: build failed", trial);
                if (!h.hub_blocks) continue;  // a tree was found to pay
                ++with;
                std::vector<int64_t> orp(m + 1);
                std::vector<int32_t> oci(h.stats.nnz + 1);
                if (cbm_decompress_host(&h, orp.data(), oci.data()) != CBM_OK) return fail("decompress failed", trial);
                std::vector<int> written(h.num_slots, 0), row_of(h.num_slots, -1);
                for (const CbmTask& c : h.comb)
                    for (uint32_t s = 0; s < (c.len_flags & CBM_TASK_LEN_MASK); ++s) {
                        if ((int64_t)c.start + s >= h.num_slots || row_of[c.start + s] >= 0) return fail("hubs: combine list", trial);
                        row_of[c.start + s] = c.row;
                    }
                std::vector<std::set<int>> got(m);
                auto add = [&](int64_t slot, uint32_t col) { return col < (uint32_t)n && row_of[slot] >= 0 && got[row_of[slot]].insert((int)col).second; };
                int64_t in_share = 0;
                for (int j = 0; j < CBM_XCD; ++j) in_share += h.blk_count[j];
                if (in_share != (int64_t)h.row_blocks.size()) return fail("hubs: shares", trial);
                for (const CbmBlock& b : h.row_blocks) {
                    if (b.row0 + CBM_BLOCK_ROWS > h.block_rows.size() || (size_t)(b.group0 + b.ngroups) * 64 > h.block_cols.size())
                        return fail("hubs: block out of range", trial);
                    for (int i = 0; i < CBM_BLOCK_ROWS; ++i) {
                        const uint32_t slot = h.block_rows[b.row0 + i];
                        if (slot != CBM_BLOCK_NO_ROW && (slot >= (uint32_t)h.num_slots || written[slot]++)) return fail("hubs: slot", trial);
                        for (uint32_t g = b.group0; g < b.group0 + b.ngroups; ++g)
                            for (int p = 0; p < 64; ++p) {
                                const uint32_t word = h.block_masks[(size_t)g * 256 + 4 * (i % 32 + 32 * (p % 16 / 8)) + p / 16];
                                if (!(word >> (8 * (i / 32) + p % 8) & 1u)) continue;
                                if (slot == CBM_BLOCK_NO_ROW || !add(slot, h.block_cols[(size_t)g * 64 + p])) return fail("hubs: entry", trial);
                            }
                    }
                }
                int64_t walked = 0;
                for (const CbmTask& t : h.tasks) {
                    const uint32_t len = t.len_flags & CBM_TASK_LEN_MASK;
                    if ((size_t)t.start + len > h.stream.size()) return fail("hubs: work item out of range", trial);
                    if (t.len_flags & CBM_TASK_SEGMENT) {
                        if (t.row < 0 || t.row >= h.num_slots || written[t.row]++) return fail("hubs: segment's slot", trial);
                        for (uint32_t i = 0; i < len; ++i)
                            if (!add(t.row, h.stream[t.start + i])) return fail("hubs: segment's entry", trial);
                        walked += len;
                        continue;
                    }
                    for (uint32_t i = 0; i + 1 < len; ++i)
                        if (!got[t.row].insert((int)h.stream[t.start + i]).second) return fail("hubs: whole row", trial);
                }
                if (walked != h.seg_deltas) return fail("hubs: deltas of the segments", trial);
                for (int w : written)
                    if (w != 1) return fail("hubs: a slot never written", trial);
                for (int i = 0; i < m; ++i)
                    if (!std::equal(got[i].begin(), got[i].end(), oci.begin() + orp[i], oci.begin() + orp[i + 1])) return fail("hubs: a row differs", trial);
                // the scratch that cbm_spmm_noalloc goes by is that of the same handle without hub blocks
                setenv("CBM_HUB_BLOCKS", "0", 1);
                cbm_handle plain;
                plain.opts = h.opts;
                if (cbm_build_host(m, n, rp.data(), ci.data(), &plain) != CBM_OK || plain.num_slots != h.noalloc_slots)
                    return fail("hubs: scratch without them", trial);
                setenv("CBM_HUB_BLOCKS", "2", 1);
            }
    if (with < 18) return fail("hubs: too few", with);
    unsetenv("CBM_SPLIT_MIN");
    std::puts("hubs ok");
    return 0;
}

int main() {
    if (int rc = hubs()) return rc;
    setenv("CBM_HUB_BLOCKS", "0", 1);
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

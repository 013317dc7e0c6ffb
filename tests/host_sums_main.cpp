// The shared sums of small square matrices, put together again: every row's sets, single columns and own column add up to the row, every
// index is in range, every item is in one XCD's run, and the sets do not depend on the number of threads.  Built with ASan/UBSan by
// test_shared_sums_host.py.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
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
    setenv("CBM_ROW_BLOCKS", "0", 1);
    setenv("CBM_HUB_BLOCKS", "0", 1);
    setenv("CBM_SHARED_SUMS", "1", 1);
    std::mt19937 rng(5);
    int trial = 0, with = 0, without = 0;
    long saved = 0;
    for (int n : {1, 2, 5, 40, 300, 1500})
        for (int form = 0; form < 8; ++form, ++trial) {
            std::vector<std::set<int>> a(n);
            const int groups = n / 4 + 1;
            for (int g = 0; g < groups; ++g) {  // cliques; blocks of other rows than columns; all of them with holes
                std::set<int> rows, cols;
                const int size = 2 + (int)(rng() % (form == 7 ? 600 : 30));
                for (int i = 0; i < size; ++i) rows.insert((int)(rng() % n));
                if (form % 4 == 1) for (int i = 0; i < size; ++i) cols.insert((int)(rng() % n));
                else cols = rows;
                for (int r : rows)
                    for (int c : cols)
                        if (form % 4 != 2 || rng() % 20) a[r].insert(c);
                if (form == 7 && g > 4) break;
            }
            if (form == 3) for (int c = 0; c < n; ++c) a[n / 2].insert(c), a[c].insert(n / 2);  // a row of every column
            for (int i = 0; i < n; ++i)
                if (form < 4 || rng() % 2) a[i].erase(i);
            std::vector<int64_t> rp(n + 1, 0);
            std::vector<int32_t> ci;
            for (int i = 0; i < n; ++i) {
                ci.insert(ci.end(), a[i].begin(), a[i].end());
                rp[i + 1] = (int64_t)ci.size();
            }
            cbm_handle h[2];
            for (int t = 0; t < 2; ++t) {
                h[t].opts = cbm_build_opts{};
                h[t].opts.add_self_loops = trial % 2;
                h[t].opts.num_threads = t ? 3 : 1;
                h[t].opts.flags = CBM_FLAG_HOST_ONLY | (form == 5 ? CBM_FLAG_TRANSPOSE : 0u);
                if (cbm_build_host(n, n, rp.data(), ci.data(), &h[t]) != CBM_OK) return fail("build failed", trial);
            }
            if (h[0].num_sums != h[1].num_sums || h[0].sum_entries != h[1].sum_entries) return fail("depends on the number of threads", trial);
            if (h[0].num_sums == 0) continue;
            ++with;
            const cbm_handle& x = h[0];
            std::vector<int64_t> orp(n + 1);
            std::vector<int32_t> oci(x.stats.nnz + 1);
            if (cbm_decompress_host(&x, orp.data(), oci.data()) != CBM_OK) return fail("decompress failed", trial);
            if ((int64_t)x.sum_items.size() != x.num_sums + n) return fail("number of items", trial);
            std::vector<int> seen(n, 0);
            int64_t longest[2] = {0, 0}, entries = 0;
            for (size_t i = 0; i < x.sum_items.size(); ++i) {
                const CbmSumItem& it = x.sum_items[i];
                const bool row = (int64_t)i >= x.num_sums;
                const uint32_t len = it.len & ~CBM_SUM_OWN;
                if (it.start != (uint32_t)entries || (size_t)it.start + len > x.sum_entries.size()) return fail("entries out of range", trial);
                entries += len;
                longest[row] = std::max<int64_t>(longest[row], len);
                std::map<int, int> sum;
                for (uint32_t p = it.start; p < it.start + len; ++p) {
                    const uint32_t e = x.sum_entries[p];
                    if (!(e & CBM_SUM_BIT)) {
                        if (e >= (uint32_t)n) return fail("column out of range", trial);
                        ++sum[(int)e];
                        continue;
                    }
                    if (!row || (int64_t)(e & ~CBM_SUM_BIT) >= x.num_sums) return fail("set out of range", trial);
                    const CbmSumItem& s = x.sum_items[e & ~CBM_SUM_BIT];
                    for (uint32_t q = s.start; q < s.start + s.len; ++q) ++sum[(int)x.sum_entries[q]];
                }
                if (!row) continue;
                if (it.row < 0 || it.row >= n || seen[it.row]++) return fail("a row twice or none", trial);
                if (it.own) sum[it.row] += it.own;
                if (sum.count(it.row) && sum[it.row] == 0) sum.erase(it.row);
                std::map<int, int> want;
                bool holds = false;
                for (int64_t p = orp[it.row]; p < orp[it.row + 1]; ++p) want[oci[p]] = 1, holds = holds || oci[p] == it.row;
                if (sum != want) return fail("a row's parts do not add up to it", trial);
                if (holds != ((it.len & CBM_SUM_OWN) != 0)) return fail("own column", trial);
                if (!holds)  // sets that hold the row's column come first, -own of them
                    for (uint32_t p = it.start; p < it.start + len && (x.sum_entries[p] & CBM_SUM_BIT); ++p) {
                        const CbmSumItem& s = x.sum_items[x.sum_entries[p] & ~CBM_SUM_BIT];
                        const bool mine = std::count(x.sum_entries.begin() + s.start, x.sum_entries.begin() + s.start + s.len, (uint32_t)it.row) > 0;
                        if (mine != ((int)(p - it.start) < -it.own)) return fail("sets with the own column come first", trial);
                        without += !mine;
                    }
            }
            if (entries != (int64_t)x.sum_entries.size()) return fail("entries left over", trial);
            saved += x.stats.nnz - entries;
            for (int half = 0; half < 2; ++half) {
                if (longest[half] != x.sum_longest[half]) return fail("longest", trial);
                int64_t at = half ? x.num_sums : 0;
                for (int j = 0; j < CBM_XCD; ++j) {
                    if (x.sum_begin[half][j] != at || x.sum_count[half][j] < 0) return fail("runs", trial);
                    at += x.sum_count[half][j];
                }
                if (at != (half ? x.num_sums + n : x.num_sums)) return fail("runs do not cover the items", trial);
            }
        }
    if (with < 15 || saved <= 0 || without == 0) return fail("too few plans", with);
    std::printf("sums ok: %d plans, %ld entries saved\n", with, saved);
    return 0;
}

// The automatic choice of row and hub blocks, on host-only handles (which do without blocks by default): who takes them, who does not,
// and what is left of a plan that is given up.  Run by test_row_blocks_host.py.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <string>
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

struct Matrix {
    int m;
    std::vector<int64_t> rp{0};
    std::vector<int32_t> ci;
    void add(const std::set<int>& row) {
        ci.insert(ci.end(), row.begin(), row.end());
        rp.push_back((int64_t)ci.size());
    }
};
// rows that share most of their columns with their neighbours
static Matrix band(int m, int reach) {
    Matrix a{m};
    for (int i = 0; i < m; ++i) {
        std::set<int> s;
        for (int c = i - reach; c <= i + reach; ++c) s.insert((c + m) % m);
        a.add(s);
    }
    return a;
}
static Matrix scattered(int m, int degree) {
    Matrix a{m};
    std::mt19937 rng(5);
    for (int i = 0; i < m; ++i) {
        std::set<int> s;
        while ((int)s.size() < degree) s.insert((int)(rng() % m));
        a.add(s);
    }
    return a;
}
// alike rows wherever the estimate looks (32 evenly spread ones and their nearest), scattered ones between
static Matrix mixed(int m, int degree) {
    Matrix a{m};
    std::mt19937 rng(5);
    const int every = m / 32;
    for (int i = 0; i < m; ++i) {
        std::set<int> s;
        if (i % every < 128)
            for (int c = 0; c < 128; ++c) s.insert(i / every * every + c);
        while ((int)s.size() < degree) s.insert((int)(rng() % m));
        a.add(s);
    }
    return a;
}
// popular columns, rows of up to a few hundred entries
static Matrix popular(int m) {
    Matrix a{m};
    std::mt19937 rng(5);
    for (int i = 0; i < m; ++i) {
        std::set<int> s;
        const int len = i % 4 == 0 ? 300 + (int)(rng() % 900) : (int)(rng() % 20);
        for (int c = 0; c < len; ++c) {
            const double u = (rng() % 1000000) / 1000000.0;
            s.insert((int)((m - 1) * u * u * u));
        }
        a.add(s);
    }
    return a;
}

static bool build(const Matrix& a, cbm_handle* h, uint32_t flags = CBM_FLAG_HOST_ONLY, int max_depth = 0) {
    h->opts = cbm_build_opts{};
    h->opts.num_threads = 4;
    h->opts.flags = flags;
    h->opts.max_depth = max_depth;
    return cbm_build_host(a.m, a.m, a.rp.data(), a.ci.data(), h) == CBM_OK;
}
static bool none(const cbm_handle& h) {
    return h.row_blocks.empty() && h.block_rows.empty() && h.block_cols.empty() && h.block_masks.empty() && !h.hub_blocks && !h.in_row_blocks();
}
#define WANT(what) \
    if (!(what)) return std::printf("line %d: %s\n", __LINE__, #what), 1

int main() {
    {   // by default a host-only handle has neither
        cbm_handle h;
        WANT(build(band(6000, 40), &h) && none(h));
        cbm_handle p;
        WANT(build(popular(12000), &p) && none(p));
    }
    setenv("CBM_ROW_BLOCKS", "2", 1);
    setenv("CBM_HUB_BLOCKS", "3", 1);
    {
        const Matrix alike = band(6000, 40);
        cbm_handle h, fixed, exact;
        WANT(build(alike, &h) && h.in_row_blocks() && h.row_blocks.size() == 47);
        WANT(build(alike, &fixed, CBM_FLAG_HOST_ONLY, 16) && none(fixed));                         // a tree that was asked for
        WANT(build(alike, &exact, CBM_FLAG_HOST_ONLY | CBM_FLAG_EXACT_TREE) && none(exact));
        setenv("CBM_ROW_BLOCKS", "0", 1);
        cbm_handle off;
        WANT(build(alike, &off) && none(off) && off.parent == h.parent && off.stream == h.stream && off.num_slots == h.num_slots);
        setenv("CBM_ROW_BLOCKS", "2", 1);
    }
    {   // too small, too thin, one row too long, nothing in common
        cbm_handle small, thin, few, longest;
        WANT(build(band(500, 40), &small) && none(small));
        WANT(build(band(6000, 7), &thin) && none(thin));
        WANT(build(scattered(6000, 40), &few) && none(few));
        Matrix hub = band(6000, 40);
        std::vector<int32_t> all(6000);
        for (int c = 0; c < 6000; ++c) all[c] = c;
        hub.ci.erase(hub.ci.begin() + hub.rp[7], hub.ci.begin() + hub.rp[8]);
        hub.ci.insert(hub.ci.begin() + hub.rp[7], all.begin(), all.end());
        for (int i = 8; i <= 6000; ++i) hub.rp[i] += 6000 - 81;
        WANT(build(hub, &longest) && none(longest));
    }
    {   // estimated to pay, built, found not to, and given up
        const Matrix a = mixed(32 * 512, 60);
        cbm_handle h, off;
        WANT(build(a, &h) && none(h));
        setenv("CBM_ROW_BLOCKS", "0", 1);
        WANT(build(a, &off) && off.stream == h.stream && off.tasks.size() == h.tasks.size());
        setenv("CBM_ROW_BLOCKS", "2", 1);
    }
    {
        const Matrix a = popular(12000);
        cbm_handle h, again, off, other;
        WANT(build(a, &h) && h.hub_blocks && !h.in_row_blocks() && h.num_slots > 0);
        WANT(build(scattered(6000, 300), &other) && none(other));  // long rows, but no popular columns
        setenv("CBM_MOST_SLOTS", std::to_string(h.num_slots - 1).c_str(), 1);
        WANT(h.noalloc_slots < h.num_slots);                       // (else the limit refuses the handle either way)
        WANT(build(a, &again) && none(again));                     // more scratch than there is: built again without
        unsetenv("CBM_MOST_SLOTS");
        setenv("CBM_HUB_BLOCKS", "0", 1);
        WANT(build(a, &off) && off.stream == again.stream && off.num_slots == again.num_slots && again.noalloc_slots == off.num_slots &&
             off.seg_deltas == again.seg_deltas && off.stats.num_tasks == again.stats.num_tasks);
    }
    std::puts("policy ok");
    return 0;
}

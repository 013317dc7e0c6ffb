// Builds that run out of memory in one of the builder's own threads: the exception reaches the caller (cbm_build turns it into a
// status) instead of ending the process.  And what the threads hold together stays bounded, however many there are.  Run by
// test_row_blocks_host.py.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <malloc.h>
#include <new>
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

static thread_local bool caller = false;
static std::atomic<long> until{-1};  // allocations of other threads until one fails; negative: none will

static std::atomic<long> now{0}, most{0};  // bytes

void* operator new(size_t bytes) {
    if (!caller && until.load() >= 0 && until.fetch_sub(1) == 0) throw std::bad_alloc();
    void* p = std::malloc(bytes ? bytes : 1);
    if (!p) throw std::bad_alloc();
    const long at = now += (long)malloc_usable_size(p);
    for (long m = most; m < at && !most.compare_exchange_weak(m, at);) {
    }
    return p;
}
void operator delete(void* p) noexcept {
    now -= (long)malloc_usable_size(p);
    std::free(p);
}
void operator delete(void* p, size_t) noexcept { operator delete(p); }

static std::vector<int64_t> rp;
static std::vector<int32_t> ci;
static void matrix(int m, int n) {  // long rows with popular columns among short ones
    std::mt19937 rng(11);
    rp.assign(m + 1, 0);
    ci.clear();
    for (int i = 0; i < m; ++i) {
        std::set<int> s;
        const int len = i % 3 == 0 ? 150 + (int)(rng() % 500) : (int)(rng() % 20);
        for (int c = 0; c < len; ++c) {
            const double u = (rng() % 10000) / 10000.0;
            s.insert((int)((n - 1) * u * u * u));
        }
        ci.insert(ci.end(), s.begin(), s.end());
        rp[i + 1] = (int64_t)ci.size();
    }
}

// 8,192 rows and 32 M columns, 64 threads: 1.35 GB with tables per thread of at most 1 GiB together, 3.6 with one for every thread
static int bounded() {
    const int m = 8192, n = 32 << 20;
    setenv("CBM_ROW_BLOCKS", "0", 1);
    setenv("CBM_HUB_BLOCKS", "2", 1);
    matrix(m, n);
    cbm_handle h;
    h.opts = cbm_build_opts{};
    h.opts.num_threads = 64;
    h.opts.flags = CBM_FLAG_HOST_ONLY;
    most = now.load();
    const long before = now;
    if (cbm_build_host(m, n, rp.data(), ci.data(), &h) != CBM_OK) return std::puts("build failed"), 1;
    std::printf("hub blocks %d, %.2f GB at most\n", (int)h.hub_blocks, (most - before) / 1e9);
    return !h.hub_blocks || most - before > 2200000000L;
}

int main() {
    caller = true;
    setenv("CBM_SPLIT_MIN", "128", 1);
    if (bounded()) return 1;
    const int m = 1500;
    matrix(m, m);
    for (int hubs = 0; hubs < 2; ++hubs) {
        setenv("CBM_ROW_BLOCKS", hubs ? "0" : "1", 1);
        setenv("CBM_HUB_BLOCKS", hubs ? "2" : "0", 1);
        int failed = 0;
        for (long at = 0;; at += 1 + at / 16) {
            cbm_handle h;
            h.opts = cbm_build_opts{};
            h.opts.num_threads = 3;
            h.opts.flags = CBM_FLAG_HOST_ONLY;
            until = at;
            bool thrown = false;
            try {
                if (cbm_build_host(m, m, rp.data(), ci.data(), &h) != CBM_OK) return std::puts("build failed"), 1;
            } catch (const std::bad_alloc&) {
                thrown = true;
            }
            const bool reached = until.exchange(-1) < 0;
            if (thrown != reached) return std::puts("a failed allocation was swallowed, or none failed"), 1;
            if (!thrown) {
                if (h.row_blocks.empty()) return std::puts("no blocks"), 1;
                break;
            }
            ++failed;
        }
        if (failed < 10) return std::puts("too few"), 1;
    }
    std::puts("allocations ok");
    return 0;
}

// Shared sums of a square matrix: column sets that many rows hold in full, each summed once (host side, once per handle).
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "cbm_internal.h"

// The rows of A v I are written as disjoint unions of shared sets and single columns (the diagonal aside: a row may be in several
// sets that hold its own column, and adds it as often as it has to be there in the end, a whole number that may be negative).
// A clique of s nodes is one set with s rows: 2 s gathered rows instead of s (s - 1).
struct SharedSums {
    std::vector<int64_t> set_ptr{0};     // columns of each set, ascending
    std::vector<int32_t> set_cols;
    std::vector<int64_t> row_ptr;        // sets of each row (m + 1)
    std::vector<int32_t> row_sets;
    std::vector<int32_t> own;            // how often a row adds its own column beyond its sets: 1 or 0 if it holds it, minus its sets that do
    std::vector<uint8_t> covered;        // entries that a set of their row brings
    int64_t num_sets() const { return (int64_t)set_ptr.size() - 1; }
};

class SharedSumFinder {
public:
    // `holds_own_`: which rows hold their own column
    SharedSumFinder(int64_t m_, const int64_t* rowptr_, const int32_t* colidx_, const uint8_t* holds_own_)
        : m(m_), rowptr(rowptr_), colidx(colidx_), holds_own(holds_own_) {}

    // Gathered rows of X or of a set's sum per entry of the matrix, from `count` evenly spread rows: what whole neighbourhoods
    // would give, before sets of different rows get in each other's way.  A few million steps of looking at entries have to do: where
    // neighbourhoods are so large that they are spent early, the rows looked at by then speak for the rest.  Rows are looked at side by side, as
    // many at a time as the steps of those before suggest: the answer does not depend on the number of threads.
    template <class Parallel>
    double sample(int64_t count, Parallel&& parallel) {
        start();
        double gathers = 0, entries = 0;
        int64_t steps = 0;
        const int64_t step = std::max<int64_t>(1, m / count), rows = (m + step - 1) / step;
        for (int64_t b = 0, n; b < rows && steps <= kSampleSteps; b += n) {
            n = std::min(rows - b, b == 0 ? 8 : std::max<int64_t>(8, (kSampleSteps - steps) / (steps / b + 1)));
            std::vector<Left> left((size_t)n);
            parallel(n, [&](int64_t i0, int64_t i1) {
                Work w;
                for (int64_t i = i0; i < i1; ++i) left[i] = left_of((b + i) * step, w);
            });
            for (int64_t i = 0; i < n && steps <= kSampleSteps; ++i) {
                entries += (double)(rowptr[(b + i) * step + 1] - rowptr[(b + i) * step]);
                gathers += left[i].entries + left[i].sets;
                steps += left[i].steps;
            }
        }
        return entries > 0 ? gathers / entries : 1.0;
    }
    // What sets would leave of the longest of these rows: rows of the plan are not split, and a product waits for the longest.
    template <class Parallel>
    int64_t longest_left(const std::vector<int32_t>& rows, Parallel&& parallel) {
        start();
        std::vector<double> left(rows.size(), 0.0);
        parallel((int64_t)rows.size(), [&](int64_t i0, int64_t i1) {
            Work w;
            for (int64_t i = i0; i < i1; ++i) {
                const Left l = left_of(rows[i], w);
                left[i] = l.entries - (double)l.missed;
            }
        });
        return rows.empty() ? 0 : (int64_t)*std::max_element(left.begin(), left.end());
    }

    // Sets are proposed for many rows at a time from what is covered so far, side by side, and taken one after the other in row
    // order: the result does not depend on the number of threads.  `parallel(total, fn)` runs fn(begin, end) over [0, total).
    template <class Parallel>
    SharedSums find(Parallel&& parallel) {
        constexpr int64_t kBatches = 64, kPasses = 4;
        start();
        std::vector<std::vector<int32_t>> rows_of;  // rows of each set taken
        SharedSums out;
        std::vector<int32_t> seeds((size_t)m), again;
        for (int64_t i = 0; i < m; ++i) seeds[i] = (int32_t)i;
        int64_t steps = 0;
        const int64_t budget = 64 * rowptr[m] + (1 << 24);
        for (int pass = 0; pass < kPasses && !seeds.empty() && steps < budget; ++pass) {
            again.clear();
            const int64_t total = (int64_t)seeds.size();
            for (int64_t b = 0; b < kBatches && steps < budget; ++b) {  // every 64th row: neighbours rarely meet in a batch
                const int64_t count = (total - b + kBatches - 1) / kBatches;
                if (count <= 0) break;
                std::vector<std::vector<Found>> found((size_t)count);
                std::vector<int64_t> took((size_t)count, 0);
                parallel(count, [&](int64_t i0, int64_t i1) {
                    Work w;
                    for (int64_t i = i0; i < i1; ++i) {
                        w.steps = 0;
                        propose(seeds[i * kBatches + b], false, w, found[i]);
                        took[i] = w.steps;
                    }
                });
                for (int64_t i = 0; i < count; ++i) {
                    steps += took[i];
                    if (i + 1 < count)
                        for (const Found& f : found[i + 1])
                            for (size_t r = 0; r < f.rows.size(); ++r) {
                                __builtin_prefetch(&covered[f.places[f.at[r]]], 1);
                                __builtin_prefetch(&covered[f.places[f.at[r + 1] - 1]], 1);
                                __builtin_prefetch(&sets_of[f.rows[r]], 1);
                            }
                    bool lost = false;
                    for (Found& f : found[i]) lost = !take(f, out, rows_of) || lost;
                    if (lost) again.push_back(seeds[i * kBatches + b]);
                }
            }
            std::sort(again.begin(), again.end());
            seeds.swap(again);
        }
        out.row_ptr.assign((size_t)m + 1, 0);
        for (const auto& rows : rows_of)
            for (int32_t r : rows) ++out.row_ptr[r + 1];
        for (int64_t i = 0; i < m; ++i) out.row_ptr[i + 1] += out.row_ptr[i];
        out.row_sets.resize((size_t)out.row_ptr[m]);
        std::vector<int64_t> at(out.row_ptr.begin(), out.row_ptr.end() - 1);
        for (size_t g = 0; g < rows_of.size(); ++g)
            for (int32_t r : rows_of[g]) out.row_sets[at[r]++] = (int32_t)g;
        out.own.resize((size_t)m);
        for (int64_t i = 0; i < m; ++i) out.own[i] = holds_own[i] - sets_of[i];
        out.covered.swap(covered);
        return out;
    }

private:
    static constexpr int64_t kLongestRow = 2048;  // entries of a row that takes part
    static constexpr size_t kLeastSet = 4, kMostSet = 512;
    static constexpr int64_t kSampleSteps = 1 << 22;
    static constexpr int64_t kLeastGain = 2;      // gathered rows that a set has to save
    struct Found {
        std::vector<int32_t> cols, rows;
        std::vector<uint32_t> places;  // the entries that the set brings, row after row
        std::vector<uint32_t> at;      // rows.size() + 1 offsets into places
    };
    struct Work {
        std::vector<int32_t> set;
        std::vector<uint64_t> bits, keep;
        std::vector<uint8_t> row_in, col_in, mine;
        std::vector<int32_t> support;
        struct Hit {
            uint32_t member, place;
        };
        std::vector<Hit> hits;         // for each member's row in turn, the members it can still be given and where
        std::vector<uint32_t> hits_at;
        int64_t steps = 0;
    };
    int64_t m;
    const int64_t* rowptr;
    const int32_t* colidx;
    const uint8_t* holds_own;
    std::vector<uint8_t> covered;
    std::vector<int32_t> sets_of;  // sets of a row that hold its own column

    void start() {  // nothing is covered
        covered.assign((size_t)rowptr[m], 0);
        sets_of.assign((size_t)m, 0);
    }
    // Row u while nothing is covered: its entries that no set brings (`missed` of them were not looked at, for want of steps), its sets with its
    // share of making them, and what looking took.
    struct Left {
        double entries = 0, sets = 0;
        int64_t missed = 0, steps = 0;
    };
    Left left_of(int64_t u, Work& w) {
        std::vector<Found> found;
        w.steps = 0;
        Left r;
        r.entries = (double)(rowptr[u + 1] - rowptr[u]);
        r.missed = propose(u, true, w, found);
        for (const Found& f : found) {
            const int64_t mine = std::lower_bound(f.rows.begin(), f.rows.end(), (int32_t)u) - f.rows.begin();
            if (mine == (int64_t)f.rows.size() || f.rows[mine] != u) continue;
            r.entries -= (double)(f.at[mine + 1] - f.at[mine]);
            r.sets += 1.0 + (double)(f.cols.size() + 1) / (double)f.rows.size();
        }
        r.steps = w.steps;
        return r;
    }
    int64_t find_entry(int64_t i, int32_t j) const {
        const int32_t *b = colidx + rowptr[i], *e = colidx + rowptr[i + 1];
        const int32_t* at = std::lower_bound(b, e, j);
        return at != e && *at == j ? at - colidx : -1;
    }
    // gathered rows that a set saves row r: its entries for one sum, and its own column where that starts or ceases to be added
    int64_t saved(int32_t r, bool own, int64_t entries) const {
        if (!own) return entries - 1;
        const int32_t before = holds_own[r] - sets_of[r];
        return entries - 1 - (before - 1 != 0) + (before != 0);
    }

    // For every entry (u, v), v > u, that no set brings yet and whose mirror image none brings: what is common to the rows u and v
    // is the first guess at a set.  Rows and columns that most of the others do not share are dropped, and rows that do not hold all
    // of what is left.
    // `all`: the row is only looked at, and from v < u too; returns how many of its entries were left out when that had taken its steps.
    int64_t propose(int64_t u, bool all, Work& w, std::vector<Found>& found) {
        const int64_t ub = rowptr[u], ue = rowptr[u + 1];
        if (ue - ub > kLongestRow || ue - ub + 1 < (int64_t)kLeastSet) return 0;
        w.mine.assign(covered.begin() + ub, covered.begin() + ue);
        for (int64_t p = ub; p < ue; ++p) {
            const int32_t v = colidx[p];
            if (w.mine[p - ub] || v == u || (!all && v < u)) continue;
            if (all && w.steps > kSampleSteps) return std::count(w.mine.begin() + (p - ub), w.mine.end(), 0);
            const int64_t vb = rowptr[v], ve = rowptr[v + 1];
            if (ve - vb > kLongestRow) continue;
            const int64_t back = find_entry(v, (int32_t)u);
            if (back < 0 || covered[back]) continue;
            w.set.clear();
            w.steps += ue - ub + ve - vb;
            bool u_in = false, v_in = false;  // (both are members: a row's own column is always its to give)
            const int32_t lo = std::min<int32_t>((int32_t)u, v), hi = std::max<int32_t>((int32_t)u, v);
            auto add = [&](int32_t x) {
                if (!u_in && x > lo) w.set.push_back(lo), u_in = true;
                if (!v_in && x > hi) w.set.push_back(hi), v_in = true;
                w.set.push_back(x);
            };
            for (int64_t a = ub, b = vb; a < ue && b < ve;) {
                const int32_t x = colidx[a], y = colidx[b];
                if (x == y && x != u && x != v && !w.mine[a - ub] && !covered[b] && w.set.size() < kMostSet) add(x);
                a += x <= y;
                b += y <= x;
            }
            if (!u_in) w.set.push_back(lo);
            if (!v_in) w.set.push_back(hi);
            const size_t s = w.set.size(), words = (s + 63) / 64;
            if (s < kLeastSet) continue;
            w.bits.assign(s * words, 0);
            w.hits.clear();
            w.hits_at.assign(1, 0u);
            for (size_t i = 0; i < std::min<size_t>(s, 8); ++i) __builtin_prefetch(&rowptr[w.set[i]]);
            for (size_t i = 0; i < s; ++i) {  // which members each member's row can still be given
                if (i + 8 < s) __builtin_prefetch(&rowptr[w.set[i + 8]]);
                if (i + 4 < s) {  // (rows are a few cache lines, seldom near each other)
                    const int64_t next = rowptr[w.set[i + 4]], len = std::min<int64_t>(rowptr[w.set[i + 4] + 1] - next, 256);
                    for (int64_t l = 0; l < len; l += 16) __builtin_prefetch(&colidx[next + l]);
                    for (int64_t l = 0; l < len; l += 64) __builtin_prefetch(&covered[next + l]);
                }
                const int32_t r = w.set[i];
                const int64_t rb = rowptr[r], re = rowptr[r + 1];
                if (re - rb <= kLongestRow) {
                    w.bits[i * words + i / 64] |= 1ull << (i % 64);
                    w.steps += re - rb;
                    for (int64_t q = rb, j = 0; q < re && j < (int64_t)s;) {
                        const int32_t x = colidx[q], y = w.set[j];
                        if (x == y && x != r && !covered[q]) {
                            w.bits[i * words + j / 64] |= 1ull << (j % 64);
                            w.hits.push_back({(uint32_t)j, (uint32_t)q});
                        }
                        q += x <= y;
                        j += y <= x;
                    }
                }
                w.hits_at.push_back((uint32_t)w.hits.size());
            }
            w.row_in.assign(s, 1);
            w.col_in.assign(s, 1);
            int64_t nr = (int64_t)s, nc = (int64_t)s;
            auto held = [&](size_t i) {
                int64_t h = 0;
                for (size_t k = 0; k < words; ++k) h += __builtin_popcountll(w.bits[i * words + k] & w.keep[k]);
                return h;
            };
            auto columns_kept = [&] {
                w.keep.assign(words, 0);
                for (size_t j = 0; j < s; ++j)
                    if (w.col_in[j]) w.keep[j / 64] |= 1ull << (j % 64);
            };
            for (int it = 0; it < 3; ++it) {
                const int64_t per = it == 1 ? 8 : 1;  // entries held for each one missing: first the majority, then nearly all, then all
                columns_kept();
                nr = 0;
                for (size_t i = 0; i < s; ++i) {
                    const int64_t h = held(i), missing = nc - h, hits = h - w.col_in[i];
                    w.row_in[i] = it < 2 ? hits > per * missing + 1 : missing == 0 && hits > 1;
                    nr += w.row_in[i];
                }
                w.support.assign(s, 0);
                for (size_t i = 0; i < s; ++i)
                    if (w.row_in[i])
                        for (size_t k = 0; k < words; ++k)
                            for (uint64_t x = w.bits[i * words + k]; x; x &= x - 1) ++w.support[k * 64 + __builtin_ctzll(x)];
                nc = 0;
                for (size_t j = 0; j < s; ++j) {
                    const int64_t missing = nr - w.support[j], hits = w.support[j] - w.row_in[j];
                    w.col_in[j] = hits > (it == 1 ? 8 : 1) * missing + 1;
                    nc += w.col_in[j];
                }
            }
            columns_kept();
            Found f;
            for (size_t j = 0; j < s; ++j)
                if (w.col_in[j]) f.cols.push_back(w.set[j]);
            f.at.push_back(0);
            int64_t gain = -nc - 1;
            for (size_t i = 0; i < s; ++i) {
                if (held(i) != nc) continue;
                const int64_t g = saved(w.set[i], w.col_in[i], nc - w.col_in[i]);
                if (g <= 0) continue;
                gain += g;
                f.rows.push_back(w.set[i]);
                for (uint32_t k = w.hits_at[i]; k < w.hits_at[i + 1]; ++k)
                    if (w.col_in[w.hits[k].member]) f.places.push_back(w.hits[k].place);
                f.at.push_back((uint32_t)f.places.size());
            }
            if (gain < kLeastGain) continue;
            const auto me = std::lower_bound(f.rows.begin(), f.rows.end(), (int32_t)u);
            if (me != f.rows.end() && *me == u)
                for (uint32_t i = f.at[me - f.rows.begin()]; i < f.at[me - f.rows.begin() + 1]; ++i) w.mine[f.places[i] - ub] = 1;
            found.push_back(std::move(f));
        }
        return 0;
    }
    // Take a set for those of its rows whose entries are all still free, if it still pays; false if rows were lost.
    bool take(Found& f, SharedSums& out, std::vector<std::vector<int32_t>>& rows_of) {
        std::vector<int32_t> rows;
        std::vector<size_t> which;
        int64_t gain = -(int64_t)f.cols.size() - 1;
        for (size_t i = 0; i < f.rows.size(); ++i) {
            bool free = true;
            for (uint32_t k = f.at[i]; k < f.at[i + 1] && free; ++k) free = !covered[f.places[k]];
            if (!free) continue;
            const int64_t n = (int64_t)(f.at[i + 1] - f.at[i]);
            const int64_t g = saved(f.rows[i], n < (int64_t)f.cols.size(), n);
            if (g <= 0) continue;
            gain += g;
            rows.push_back(f.rows[i]);
            which.push_back(i);
        }
        const bool whole = rows.size() == f.rows.size();
        if (gain < kLeastGain) return whole;
        for (size_t w : which) {
            for (uint32_t k = f.at[w]; k < f.at[w + 1]; ++k) covered[f.places[k]] = 1;
            sets_of[f.rows[w]] += f.at[w + 1] - f.at[w] < f.cols.size();  // (one column is not among its entries: its own)
        }
        out.set_cols.insert(out.set_cols.end(), f.cols.begin(), f.cols.end());
        out.set_ptr.push_back((int64_t)out.set_cols.size());
        rows_of.push_back(std::move(rows));
        return whole;
    }
};

// Row blocks of a matrix: which rows, which columns, which bits (host side, once per handle).
#pragma once

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <vector>

#include "cbm_internal.h"

// The rows among row s's columns that share most columns with it (counted on about 64 evenly spread ones of theirs), in
// descending order: `wanted(y)` says which rows count, `take(y)` gets them.  `mark` holds no s.
template <class Wanted, class Take>
inline void nearest_rows(int32_t s, const int64_t* rowptr, const int32_t* colidx, Wanted&& wanted, std::vector<int32_t>& mark, Take&& take) {
    std::vector<std::pair<int32_t, int32_t>> near;
    for (int64_t p = rowptr[s]; p < rowptr[s + 1]; ++p) mark[colidx[p]] = s;
    for (int64_t p = rowptr[s]; p < rowptr[s + 1]; ++p) {
        const int32_t y = colidx[p];
        if (y == s || !wanted(y)) continue;
        const int64_t stride = std::max<int64_t>(1, (rowptr[y + 1] - rowptr[y]) / 64);
        int32_t shared = 0;
        for (int64_t q = rowptr[y]; q < rowptr[y + 1]; q += stride) shared += mark[colidx[q]] == s;
        near.push_back({-shared, y});
    }
    std::sort(near.begin(), near.end());
    for (const auto& c : near) take(c.second);
}

// Rows in an order that puts rows with much the same columns next to each other, for a square matrix whose columns are
// nodes like its rows: a row is followed by those of its unplaced neighbours that share most columns with it, `group` rows
// in all; the next row comes from the breadth-first frontier.
inline std::vector<int32_t> block_order(int64_t m, const int64_t* rowptr, const int32_t* colidx, int64_t group) {
    std::vector<int32_t> order, queue, mark((size_t)m, -1);
    std::vector<uint8_t> placed((size_t)m, 0), queued((size_t)m, 0);
    order.reserve((size_t)m);
    auto enqueue = [&](int32_t y) {
        if (placed[y] || queued[y]) return;
        queued[y] = 1;
        queue.push_back(y);
    };
    size_t head = 0;
    int64_t fresh = 0;
    while ((int64_t)order.size() < m) {
        while (head < queue.size() && placed[queue[head]]) ++head;
        while (head == queue.size() && placed[fresh]) ++fresh;
        const int32_t s = head < queue.size() ? queue[head++] : (int32_t)fresh;
        const size_t first = order.size();
        placed[s] = 1;
        order.push_back(s);
        nearest_rows(s, rowptr, colidx, [&](int32_t y) { return !placed[y]; }, mark, [&](int32_t y) {
            if ((int64_t)(order.size() - first) < group) {
                placed[y] = 1;
                order.push_back(y);
            } else {
                enqueue(y);
            }
        });
        for (size_t i = first + 1; i < order.size(); i += 8)
            for (int64_t q = rowptr[order[i]]; q < rowptr[order[i] + 1]; ++q) enqueue(colidx[q]);
    }
    return order;
}

// Order the `count` rows of a block so that runs of `tile` rows are alike: a run is the row with the fewest columns in
// common with the first row placed (or, for the first run, with the block's first row) and the rows that share most with it.
// `place` is all -1 on entry and on return.
inline void tiles_of_alike_rows(uint32_t* rows, int count, int tile, const int64_t* rowptr, const int32_t* colidx,
                                std::vector<int32_t>& place, std::vector<uint64_t>& bits) {
    int32_t ncols = 0;
    for (int i = 0; i < count; ++i)
        for (int64_t p = rowptr[rows[i]]; p < rowptr[rows[i] + 1]; ++p)
            if (place[colidx[p]] < 0) place[colidx[p]] = ncols++;
    const size_t words = ((size_t)ncols + 63) / 64;
    bits.assign(words * (size_t)count, 0);
    for (int i = 0; i < count; ++i)
        for (int64_t p = rowptr[rows[i]]; p < rowptr[rows[i] + 1]; ++p) {
            const int32_t c = place[colidx[p]];
            bits[words * (size_t)i + (size_t)c / 64] |= 1ull << (c % 64);
        }
    for (int i = 0; i < count; ++i)
        for (int64_t p = rowptr[rows[i]]; p < rowptr[rows[i] + 1]; ++p) place[colidx[p]] = -1;
    auto common = [&](int a, int b) {
        const uint64_t *x = bits.data() + words * (size_t)a, *y = bits.data() + words * (size_t)b;
        int s = 0;
        for (size_t w = 0; w < words; ++w) s += __builtin_popcountll(x[w] & y[w]);
        return s;
    };
    std::vector<int> with(count), left(count), order;
    std::vector<std::pair<int, int>> near;
    for (int i = 0; i < count; ++i) left[i] = i;
    int first = 0;
    while (!left.empty()) {
        int seed = left[0];
        for (int i : left) with[i] = common(first, i);
        for (int i : left)
            if (with[i] < with[seed]) seed = i;
        if (order.empty()) first = seed;
        near.clear();
        for (int i : left)
            if (i != seed) near.push_back({-common(seed, i), i});
        const size_t take = std::min<size_t>((size_t)tile - 1, near.size());
        std::partial_sort(near.begin(), near.begin() + take, near.end());
        order.push_back(seed);
        for (size_t i = 0; i < take; ++i) order.push_back(near[i].second);
        left.clear();
        for (size_t i = take; i < near.size(); ++i) left.push_back(near[i].second);
        std::sort(left.begin(), left.end());
    }
    std::vector<uint32_t> out((size_t)count);
    for (int i = 0; i < count; ++i) out[i] = rows[order[i]];
    std::copy(out.begin(), out.end(), rows);
}

// The blocks' columns as the device has them: bit 31 of a group's column 4 i + s says whether tile s holds any of the columns of step i (its bytes in
// `masks`: word i of each of the group's 64 lanes), so that the kernel knows it for a whole group by one comparison of what it loads anyway.
inline std::vector<uint32_t> flag_active_tiles(const std::vector<uint32_t>& cols, const std::vector<uint32_t>& masks) {
    std::vector<uint32_t> flagged(cols);
    for (size_t g = 0; g < cols.size() / 64; ++g)
        for (int i = 0; i < 4; ++i) {
            uint32_t any = 0;
            for (int l = 0; l < 64; ++l) any |= masks[g * 256 + 4 * (size_t)l + i];
            for (int s = 0; s < 4; ++s)
                if (any >> (8 * s) & 255u) flagged[g * 64 + 4 * i + s] |= CBM_BLOCK_ACTIVE;
        }
    return flagged;
}

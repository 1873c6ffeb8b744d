// Batches over short keys: which way a pass goes, its groups of rows and the
// workspace behind it: host arithmetic, no device code.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace sense {

// A pass (up to 64 queries) scores every row and takes the top k of the scores,
// or goes by groups of rows.
// Groups read and select a sixteenth of the scores, and cost two launches and
// the rescore of k groups: they pay where a pass's score matrix (ng queries by n
// rows) is large and k is not.  Measured over 64-dim bf16 rows, fp32 queries, us
// a search of one pass, every score / groups:
//   k = 64      2 queries   16       33          64
//     33000     26 / 29     29 / 32  31 / 34     38 / 35
//     50000     21 / 31     29 / 31  33 / 34     39 / 35
//     65536     21 / 31     24 / 31  29 / 34     36 / 36
//     90000     24 / 31     28 / 32  36 / 35     44 / 37
//     131072    24 / 32     30 / 32  40 / 35     50 / 39
//   k = 4       64 queries: 33000 35 / 34, 50000 30 / 35, 65536 32 / 35, 90000
//               41 / 36; 33 queries: 90000 33 / 35, 131072 37 / 36
//   k = 256     64 queries: 65536 44 / 65, 131072 61 / 70
// Up to kShortDirectMax rows every score always (32768 x 64 queries, k = 64: 29
// and 35 us); beyond kShortGroupsMin rows groups always.
constexpr int64_t kShortDirectMax = 32768, kShortGroupsMin = 131072;
constexpr bool short_by_groups(int64_t n, int ng, int k) {
    if (n <= kShortDirectMax) return false;
    if (n > kShortGroupsMin) return true;
    const int64_t scores = (int64_t)ng * n, unit = (int64_t)1 << 20;
    return k <= 128 && scores > (k < 32 ? 4 * unit : (n < 65536 ? 2 : 3) * unit);
}

// Rows per group: at most 16384 groups (one block's selection) up to a million
// rows; groups of 64 beyond (one wave's rescore).
constexpr int kMaxGroupRows = 64;
constexpr int64_t kSelectGroups = 16384;
constexpr int short_group_rows(int64_t n) {
    const int64_t g = 16 * ((n + 16 * kSelectGroups - 1) / (16 * kSelectGroups));
    return (int)(g < kMaxGroupRows ? g : kMaxGroupRows);
}
constexpr int64_t short_groups(int64_t n) {
    return (n + short_group_rows(n) - 1) / short_group_rows(n);
}
// The most groups that any row count up to `rows` has (more rows may have fewer,
// longer ones).
constexpr int64_t short_groups_most(int64_t rows) {
    const int64_t by16 = (rows + 15) / 16, by64 = (rows + 63) / 64;
    const int64_t most = by16 < kSelectGroups ? by16 : kSelectGroups;
    return most > by64 ? most : by64;
}

constexpr size_t short_round(size_t x) { return (x + 255) / 256 * 256; }

// Bytes of the scores of a pass over n rows of g queries, or of its group maxima
// followed (at short_keys_offset) by the keys of its k best groups' rows.
constexpr size_t short_keys_offset(int64_t groups, int g) {
    return short_round((size_t)g * (size_t)groups * 4);
}
constexpr size_t short_area_bytes(int64_t n, int g, int k) {
    const size_t scores = (size_t)g * (size_t)n * 4;
    const size_t keys = (size_t)g * (size_t)k * (size_t)short_group_rows(n) * 8;
    size_t most = 0;
    // The last pass of a batch has fewer queries and may go the other way.
    if (!short_by_groups(n, 1, k)) most = scores;
    if (short_by_groups(n, g, k)) {
        const size_t groups = short_keys_offset(short_groups(n), g) + keys;
        most = most > groups ? most : groups;
    }
    return most;
}
// The same for every row count up to a growing store's capacity.
constexpr size_t short_area_most(int64_t capacity, int g, int k) {
    const int64_t direct = capacity < kShortGroupsMin ? capacity : kShortGroupsMin;
    const size_t scores = (size_t)g * (size_t)direct * 4;
    if (capacity <= kShortDirectMax) return scores;
    const size_t groups = short_keys_offset(short_groups_most(capacity), g) +
                          (size_t)g * (size_t)k * (size_t)short_group_rows(capacity) * 8;
    return scores > groups ? scores : groups;
}

}  // namespace sense

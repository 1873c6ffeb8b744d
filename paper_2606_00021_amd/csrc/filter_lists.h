// Grid and candidate lists of a filtered batch pass over long keys: host
// arithmetic, no device code.
#pragma once

#include <stdint.h>

namespace sense {

constexpr int kFilterRows = 256;    // rows of one block of the pass
constexpr int kFilterSlots = 128;   // list entries set aside for one workgroup

// Workgroups of a pass over n_rows: one per compute unit at most, each with an
// equal run of whole blocks.  Not monotone: with 256 compute units 768 blocks
// take 256 workgroups (3 blocks each) and 769 take 193 (4 each).
constexpr int64_t filter_groups(int64_t n_rows, int64_t cus) {
    const int64_t blocks = (n_rows + kFilterRows - 1) / kFilterRows;
    const int64_t run = blocks <= cus ? 1 : (blocks + cus - 1) / cus;
    return (blocks + run - 1) / run;
}

// Slots of all workgroups of a pass over n_rows; the overflow list, of up to
// every row, follows them.
constexpr int64_t filter_slots(int64_t n_rows, int64_t cus) {
    return filter_groups(n_rows, cus) * kFilterSlots;
}

// Entries of one query's list that serve a store of n rows or, of a growing one
// (capacity > 0), every row count up to its capacity: a smaller count may take
// more workgroups than the capacity does, but never more than one per block of
// the capacity or one per compute unit.
constexpr int64_t filter_list_entries(int64_t n, int64_t capacity, int64_t cus) {
    if (capacity <= 0) return filter_slots(n, cus) + n;
    const int64_t blocks = (capacity + kFilterRows - 1) / kFilterRows;
    return (blocks < cus ? blocks : cus) * kFilterSlots + capacity;
}

}  // namespace sense

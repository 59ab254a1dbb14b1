// Which form of the batched M2L a build may take by the memory that it needs.  Plain
// arithmetic and control flow, used by the plan and, compiled for the host, by its tests.
#pragma once

#include <cstddef>
#include <cstdint>

namespace vfmm {

constexpr size_t MAX_TABLE_BYTES = size_t(8) << 30;   // operator table
constexpr size_t MAX_COLUMN_BYTES = size_t(8) << 30;  // columns of the groups by operator
// all buffers of the float64 form's batched translations, a ninth of the card (256^3
// particles at p = 10: about 13 GB); the translations one at a time need none of them
constexpr size_t MAX_F64_BYTES = size_t(32) << 30;

// Bytes that the float64 groups by block need at most: group table, groups with
// their slots, operators, multipoles by row, partial sums of the work items.  rows:
// (p + 1)^2, pad: rows padded to 16; per_item: groups of a work item.
inline size_t f64_block_bytes(int rows, int pad, int per_item, int64_t cells, int64_t blocks, int64_t keys,
                              int64_t groups) {
    const double table = 16.0 * blocks * keys, lists = (16.0 + 256.0) * groups;
    const double ops = 8.0 * pad * pad * keys, mult = 24.0 * pad * (cells + 1);
    const double items = (double)groups / per_item + blocks, part = 24.0 * rows * 64 * items;
    const double all = table + lists + ops + mult + part;
    return all < 1e18 ? (size_t)all : size_t(1e18);
}

// The first of the forms 0 .. n - 1 whose buffers could be allocated: plan(k) makes
// form k or throws; out_of_memory(e) tells failed allocations (after which drop()
// gives back what the form holds) from other errors, which pass through, as does
// the last form's failure if required.  n: none.
template <class Error, class Plan, class Drop, class OutOfMemory>
int first_form_that_fits(int n, bool required, Plan plan, Drop drop, OutOfMemory out_of_memory) {
    for (int k = 0; k < n; ++k) {
        try {
            plan(k);
            return k;
        } catch (const Error &e) {
            drop();
            if (!out_of_memory(e) || (required && k + 1 == n)) throw;
        }
    }
    return n;
}

}  // namespace vfmm

// Sample sort of (key, value) pairs (sort.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fks {

// The separators of a sorted or Eytzinger map.  Level l (1 = lowest) holds the keys at in-order
// positions 2^gran * 16^(l-1) * (j + 1) - 1 that part two groups of the level below (for the
// Eytzinger layout positions of the perfect tree of its depth; all of these nodes exist).  A group
// is a 128-byte line of sixteen entries; levels are filled up to whole lines with all-ones words.
constexpr uint32_t kSepLevels = 8;
struct SepIndex {
    uint32_t levels;                    // at least 1
    uint32_t gran;                      // log2 of the in-order keys per lowest separator
    uint64_t count[kSepLevels + 1];     // entries of level l
    uint64_t at[kSepLevels + 1];        // where level l starts in the index
    uint64_t total;                     // entries of all levels, filled up
    uint32_t depth;                     // Eytzinger: floor(log2 n)
    uint64_t first_node;                // Eytzinger: leftmost of the nodes below the separators
};

// Outcome words of a sort, cleared by it.
struct SortFlags {
    uint32_t dup;        // two keys are equal
    uint32_t overflow;   // a region was too small for its keys: the output is not complete
};

// Largest n that sample_sort takes, and the scratch it needs.
constexpr uint64_t kSampleSortMax = 256ull * 256 * 1344;
size_t sample_sort_scratch(uint64_t n);

// The pairs in ascending order of their keys, or (eytz) in the level order of the complete
// binary search tree, and the separators of that layout.  Stream-ordered; the keys are distinct
// unless flags->dup is set.
void sample_sort(const uint64_t* keys, const uint32_t* vals, uint64_t n, bool eytz, uint64_t* keys_out,
                 uint32_t* vals_out, const SepIndex& sep, uint64_t* index, SortFlags* flags, void* scratch,
                 hipStream_t st);

}  // namespace fks

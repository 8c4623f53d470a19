// Counts of pairs in two-level binning (pair_bins.hip): the bins that a run of
// entries touches and the coarse bins, packed as bins << 32 | coarse bins and added
// with saturation.
//
// A coarse bin is touched through at least one of its bins, so the coarse count
// is never above the bins': while the bins' count is below 2^32 no half carries,
// and from 2^32 on the sum has overflowed and stays at its greatest value, which
// no pair capacity reaches (MAX_PAIR_CAP).  So a sum that a capacity holds is exact
// in both halves, and the coarse pairs of the entries kept fit where their bins' do.
#pragma once

#include <stdint.h>

constexpr int64_t MAX_PAIR_CAP = 0xFFFFFFFEll;

__host__ __device__ __forceinline__ uint64_t sat_add(uint64_t a, uint64_t b) {
    const uint64_t s = a + b;
    return s < a ? ~0ull : s;
}

// An entry with counts c (its own, exact) after entries with counts `at` (their saturated sum),
// under a capacity of key_cap <= MAX_PAIR_CAP pairs: whether it is written, and whether it is
// the one that crosses the capacity (it and every later entry are dropped whole).
struct PairCut {
    bool kept, crosses;
};
__host__ __device__ __forceinline__ PairCut pair_cut(uint64_t at, uint64_t c, uint64_t key_cap) {
    const uint64_t off = at >> 32, nt = c >> 32;
    const bool fits = off + nt <= key_cap;
    return PairCut{nt != 0 && fits, nt != 0 && off <= key_cap && !fits};
}

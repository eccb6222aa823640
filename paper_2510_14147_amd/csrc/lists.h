// Sizes of the matrix filter's closed-form work lists.  Host arithmetic
// without any HIP type, so that the limits can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace fnn {

constexpr int GP = 64;  // rows per pack (max) on the MFMA path
constexpr int GW = 4;   // packs per group = waves per work-group

// Entries of the list of every pack pair over np packs: group g against
// every pack from its own first (GW g) on.
inline int64_t dense_entries(int64_t np)
{
    const int64_t ng = (np + GW - 1) / GW;
    return ng * np - GW * (ng * (ng - 1) / 2);
}

// The entries, and the units that they are cut into (fewer), are numbered in
// 32 bits, with room for a loop's last step past them.  8.39M rows in full
// packs.
constexpr int64_t LIST_MAX = INT32_MAX - 4096;
inline bool list_fits(int64_t entries) { return entries <= LIST_MAX; }
inline bool dense_fits(int64_t np) { return list_fits(dense_entries(np)); }

}  // namespace fnn

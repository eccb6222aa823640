// Sizes of the matrix filter's closed-form work lists, and the rule that takes
// them in place of a traversal's.  Host arithmetic without any HIP type, so
// that the limits can be checked without a GPU.
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

// What a traversal costs beside the filter, milliseconds: launches and host
// reads, per point (its levels' tests), and per pack pair it keeps
// (expansion, two radix sorts, unique groups).  Measured: 20K to 60K points
// in 20 clusters, 5 % kept, 0.4 to 0.7 ms; 200K points 1.3 to 2.1 ms; 988258
// codes, 76.7M pairs kept, 30 ms.
constexpr double TRAV_MS = 0.4, TRAV_POINT_MS = 4e-6, TRAV_PAIR_MS = 4.2e-7;

// The filter may take every pair of n points from the closed-form list
// instead of the traversal's (any pair set that contains the needed ones
// gives the exact graph): at once while the whole list costs no more than a
// traversal's launches and host reads, else where a sample of the tree's pack
// pairs under the traversal's own test (the share `gone` pruned) says that
// what it could prune is worth less than itself.  Never where the list's
// entries have no 32-bit numbers: then the traversal runs, whatever it keeps.
//
// That price holds for a filter that passes few pairs besides the edges.  One
// whose rounding margin is wide against eps^2 (`wide`) passes pairs that a
// traversal would have dropped, at 0.1 ns and 20 bytes each where a screened
// pair is 0.05 to 0.25 ps: there every pair is taken only where next to none
// could be pruned.
enum Dense { DENSE_NO, DENSE_YES, DENSE_SAMPLE };
inline Dense dense_rule(int64_t n, int64_t npacks, double pair_ms, bool wide)
{
    if (n < 1 || !dense_fits((n + GP - 1) / GP))
        return DENSE_NO;
    if (wide)
        return npacks >= 256 ? DENSE_SAMPLE : DENSE_NO;
    return 0.5 * n * n * pair_ms <= TRAV_MS + TRAV_POINT_MS * n ? DENSE_YES : DENSE_SAMPLE;
}
inline bool dense_sampled(int64_t n, int64_t npacks, double pair_ms, bool wide, double gone)
{
    if (wide)
        return gone <= 0.01;
    const double kept = 0.5 * (1.0 - gone) * npacks * (double)npacks;
    return gone * 0.5 * n * n * pair_ms <=
           TRAV_MS + TRAV_POINT_MS * n + TRAV_PAIR_MS * kept;
}

}  // namespace fnn

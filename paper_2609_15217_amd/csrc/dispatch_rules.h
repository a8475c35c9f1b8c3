/* Which kernel a uniform batch runs: the rules that refine the dispatch table
 * (measured with the factors written, textbook pivoting). Host code. */
#ifndef LUPP_DISPATCH_RULES_H
#define LUPP_DISPATCH_RULES_H

#include <cstdint>

#include "lupp.h"

namespace lupp {

struct Choice {
    int variant;  /* LUPP_VARIANT_THREAD / LUPP_VARIANT_LANES / kVariantNarrow */
    int lanes;
    int wpb;
};

/* The lanes solver with half the lanes (twice the rows per lane) of the
 * variants lupp_force_variant names: chosen by auto_choice only. */
constexpr int kVariantNarrow = 3;

/* The calls a table entry binds as it stands, without refinement: all of them
 * where the caller set it, those that were timed where it was autotuned. */
enum EntryBinds : uint8_t { kBindsFactors = 1, kBindsSolveOnly = 2, kBindsTiled = 4, kBindsAll = 7 };

/* Refinement of a built-in table entry by what the table does not hold: large
 * batches that only solve (LUPP_KEEP_A). The table is tuned with the factors
 * written, where stores of whole lines decide and more lanes per system win;
 * without them instructions decide, and fewer lanes with more rows each spend
 * fewer per system. Measured at 2^20 systems (n <= 16) and 2^18 (above), us,
 * solve-only, table entry -> this one:
 *   AoS  n = 3: 30.7 -> 24.4 (thread); n = 8: 156 -> 136, n = 5: 86.8 -> 64.2
 *        (4 lanes); n = 12: 392 -> 289 (4 lanes, 3 rows each); n = 16: 667 ->
 *        618 (8 lanes against 16); n = 24: 555 -> 435 (8 lanes, 3 rows each);
 *        n = 32 at 2^20: 3538 -> 3425 (2 waves per workgroup against 4)
 *   SoA  n = 12: 466 -> 335 (4 lanes against the thread kernel, which wins up
 *        to n = 10: 225 against 247); n = 24: 654 -> 529
 * The interleaved layout stores whole lines with any segment width, so 8 lanes
 * also win there with the factors (n = 24: 767 -> 711; n = 17: 421 -> 353). */
inline Choice auto_choice(int n, int layout, int bucket, bool factors, const Choice &c)
{
    if (bucket == 0) return c;
    const bool aos = layout == LUPP_AOS;
    if (n >= 17 && n <= 24 && (!aos || !factors)) return {kVariantNarrow, 8, 1};
    if (factors) return c;
    if (!aos) return (n == 11 || n == 12) ? Choice{kVariantNarrow, 4, 0} : c;
    if (n == 2 || n == 3) return {LUPP_VARIANT_THREAD, 1, 1};
    if (n >= 5 && n <= 8) return {LUPP_VARIANT_LANES, 4, 2};
    if (n >= 9 && n <= 12) return {kVariantNarrow, 4, 2};
    if (n >= 13 && n <= 16) return {LUPP_VARIANT_LANES, 8, 4};
    if (n >= 27) return {LUPP_VARIANT_LANES, 16, 2};
    return c;
}

/* Tile-local pivoting runs other kernels (kernels_lanes.h) than those the
 * table's entries were measured with. Packed batches of n = 9..16 are faster
 * with two rows per lane there (tile 4, 524288 systems, factors, us, table's
 * entry -> this: n = 9: 236 -> 212; n = 12: 371 -> 315; n = 16: 582 -> 487),
 * small interleaved ones from n = 22 on with 16 lanes (4096 systems: n = 28:
 * 40.5 -> 39.3; n = 32: 47.9 -> 47.0; n = 17 would lose, 22.9 -> 23.4). The
 * other entries measured within 3% of the best. */
inline Choice tiled_choice(int n, int layout, int bucket, const Choice &c)
{
    if (layout == LUPP_SOA)
        return bucket == 0 && n >= 22 ? Choice{LUPP_VARIANT_LANES, 16, 0} : c;
    return bucket == 1 && n >= 9 && n <= 16 ? Choice{LUPP_VARIANT_LANES, 8, 4} : c;
}

inline Choice refined_choice(int n, int layout, int bucket, bool factors, bool tiled, unsigned binds,
                             const Choice &c)
{
    if ((binds & (tiled ? kBindsTiled : factors ? kBindsFactors : kBindsSolveOnly)) != 0) return c;
    return tiled ? tiled_choice(n, layout, bucket, c) : auto_choice(n, layout, bucket, factors, c);
}

}  // namespace lupp

#endif

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
 * fewer per system. Measured on N(0, 1) systems at 2^20 systems (n <= 16) and
 * 2^18 (above), us, solve-only, table entry -> this one:
 *   AoS  n = 3: 30.7 -> 24.4 (thread); n = 8: 156 -> 136, n = 5: 86.8 -> 64.2
 *        (4 lanes); n = 12: 392 -> 289 (4 lanes, 3 rows each); n = 16: 667 ->
 *        618 (8 lanes against 16); n = 24: 555 -> 435 (8 lanes, 3 rows each)
 *   SoA  n = 12: 393 -> 337 (4 lanes against the thread kernel); n = 24:
 *        654 -> 529
 * The interleaved layout stores whole lines with any segment width, so 8 lanes
 * also win there with the factors (n = 24: 767 -> 711; n = 17: 421 -> 353).
 * The line at the large entries' 32768 systems: time of this choice over that
 * of the table's entry at 32768 / 50000 / 100000 / 200000 systems, over the
 * sizes of a row: AoS 2..3 0.97-0.99 / 0.97-0.98 / 0.98-1.00 / 0.82-1.01,
 * 5..8 0.99-1.03 / 0.96-1.00 / 0.91-0.98 / 0.89-0.94, 9..12 0.91-0.97 /
 * 0.91-0.94 / 0.83-0.86 / 0.74-0.76, 13..16 0.95-0.97 / 0.94-1.02 /
 * 0.92-0.98 / 0.87-0.92, 17..24 0.87-1.00 / 0.85-0.93 / 0.79-0.92 /
 * 0.75-0.89; SoA 12 0.83 / 0.96 / 0.77 / 0.69, 17..24 0.93-1.00 / 0.83-0.94 /
 * 0.79-0.92 / 0.75-0.90, with the factors 0.88-1.03 / 0.85-0.95 / 0.81-0.96 /
 * 0.80-0.96.
 * The thread kernel skips row interchanges that no lane of a wave asks for, so
 * systems that pivot on the diagonal are faster on it: interleaved n = 12,
 * diagonally dominant, 65536 / 200000 / 2^20 systems: 22.7 / 63.8 / 322 us
 * against 29.5 / 65.6 / 335 here (N(0, 1): 30.7 / 96.6 / 393 against 29.9 /
 * 66.1 / 337). At n = 11 that costs more (18.7 / 47.1 / 263 against 26.0 /
 * 58.2 / 288) than N(0, 1) systems gain (24.9 / 71.0 / 310 against 26.3 /
 * 58.6 / 287): it stays with the thread kernel. */
inline Choice auto_choice(int n, int layout, int bucket, bool factors, const Choice &c)
{
    if (bucket == 0) return c;
    const bool aos = layout == LUPP_AOS;
    if (n >= 17 && n <= 24 && (!aos || !factors)) return {kVariantNarrow, 8, 1};
    if (factors) return c;
    if (!aos) return n == 12 ? Choice{kVariantNarrow, 4, 0} : c;
    if (n == 2 || n == 3) return {LUPP_VARIANT_THREAD, 1, 1};
    if (n >= 5 && n <= 8) return {LUPP_VARIANT_LANES, 4, 2};
    if (n >= 9 && n <= 12) return {kVariantNarrow, 4, 2};
    if (n >= 13 && n <= 16) return {LUPP_VARIANT_LANES, 8, 4};
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

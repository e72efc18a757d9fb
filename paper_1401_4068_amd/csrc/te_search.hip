// te_search.hip -- which search kernel runs a launch over ordered chunks, and the kernels of
// single chunks at k = 4.

#include "te_search.h"

namespace te {

namespace {

// LDS bytes per workgroup (the rows are dynamic shared memory).
size_t lds_bytes(int d_y, int d_x, bool sets, int waves_per_wg)
{
    const int v = sets ? set_variants(d_y, d_x) : 1;
    const int nr = 1 + d_y + v * d_x + v;
    return (size_t)waves_per_wg * kWave * (size_t)((nr + 3) & ~3) * sizeof(float);
}

// The kernel of a launch; w waves to a block, 0: persistent waves, `slots` blocks of candidates
// counted together in pass 2.
search_fn pick(int d_y, int d_x, int k, int slots, bool sets, int w)
{
    if (k < 1 || k > kMaxK || (sets && k != 4))
        return nullptr;
    if (sets)
        return pick_search_sets(d_y, d_x, slots, w);
    if (k != 4)
        return k <= 8 ? pick_search_small_k(d_y, d_x, k, w) : pick_search_large_k(d_y, d_x, w);
    switch (w) {
    case 0: return slots == 1 ? pick_single<5, false, 1, 0>(d_y, d_x) : pick_single<5, false, 2, 0>(d_y, d_x);
    case 2: return pick_single<5, false, 1, 2>(d_y, d_x);
    case 4: return pick_single<5, false, 1, 4>(d_y, d_x);
    case 8: return pick_single<5, false, 1, 8>(d_y, d_x);
    default: return nullptr;
    }
}

}  // namespace

// The persistent search over ordered chunks, single or in sets (k = 4); no kernel where there is none.
// Blocks of candidates counted together in pass 2 at k = 4: the tuned slot count 4 -> 1, 8 or 16 -> 2.
ordered_search pick_ordered(int d_y, int d_x, int k, int slots, bool sets, int waves_per_wg)
{
    ordered_search s{nullptr, 0};
    if (slots != 4 && slots != 8 && slots != 16)
        return s;
    s.fn = pick(d_y, d_x, k, slots == 4 ? 1 : 2, sets, 0);
    s.lds = lds_bytes(d_y, d_x, sets, waves_per_wg);
    return s;
}

// Waves to a block for a launch of n_items blocks; 0: persistent waves, a block each.  With few
// blocks the chip has more SIMDs than items and a wave, alone on its SIMD, issues an instruction
// every 6 clocks: the time is one block's chain of instructions.  W waves to a block cut that chain
// by W, at the price of W walks over the boxes and of insertions for 64 / W references at a time.
// Measured, us per call of one launch (persistent / W = 2 / 4 / 8):
//   k = 4, 32 blocks (N = 2 000, D = 5)      174 /  - / 103 /  92
//   k = 4, 750 blocks (N = 48 000, D = 7)    1152 / 804 / 624 / 575
//   k = 4, 7 900 blocks (N = 5 000, D = 7)   1136 / 720 / 775 / 969
//   k = 4, 31 600 blocks                     2339 / 2334 / 2697 / 3630
//   k = 1, 940 / 3 760 / 24 400 blocks       224 / 159 / 134 / 140, 551 / 221 / 221 / 276, 1241 / 711 / 867 / 1201
//   k = 6, 940 / 8 200 / 24 400 blocks       282 / 214 / 174 / 185, 890 / 521 / 549 / 765, 1306 / 1216 / 1366 / 2047
//   k = 8, 940 / 8 200 / 24 400 blocks       299 / 234 / 188 / 189, 897 / 588 / 608 / 834, 1333 / 1392 / 1532 / 2254
//   k = 12, 940 / 8 200 / 24 400 blocks      332 /  - / 238 /  - , 855 /  - / 823 /  - , 1425 /  - / 2124 /  -
//   sets (3, 3), 224 / 1 088 / 2 688 / 8 704 blocks (N = 2 000)   442 / 311 / 212 / 169, 478 / 368 / 355 / 366,
//                                            615 / 619 / 588 / 688, 1243 / 1498 / 1581 / 1967
//   sets (2, 2), 224 / 1 088 / 2 688 / 8 704 / 17 408 blocks      287 / 235 / 167 / 136, 321 / 281 / 235 / 284,
//                                            468 / 426 / 400 / 514, 1033 / 921 / 1002 / 1395, 1397 / 1675 / 1869 / 2673
// A set's pairs of up to nine coordinates leave the persistent waves idle up to 9 000 blocks, wider ones do not.
int waves_to_a_block(int64_t n_items, int set_coords, int k)
{
    if (set_coords > 0)
        return n_items <= 512 ? 8 : (n_items <= 3072 ? 4 : (set_coords <= 9 && n_items <= 9216 ? 2 : 0));
    if (k > 8)
        return n_items <= 8192 ? 4 : 0;
    if (n_items <= 832)
        return 8;
    return n_items <= 4096 ? 4 : (n_items <= (k <= 6 ? 24576 : 16384) ? 2 : 0);
}

// The search with w waves to a block (w from waves_to_a_block, not 0): one workgroup of w waves per item.
ordered_search pick_shared(int d_y, int d_x, int k, bool sets, int w)
{
    return ordered_search{pick(d_y, d_x, k, 1, sets, w), lds_bytes(d_y, d_x, sets, w)};
}

}  // namespace te

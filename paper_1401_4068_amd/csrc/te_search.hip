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
// Longer lists cost it more: every wave fills its own, and merges them.  Persistent waves pay at the end
// of a launch, 0.2 to 0.55 ms if its items come in a queue per XCD (every wave tries them all), so the
// lines lie higher there.
// Measured: ratios of the searches' times, geometric means over six (d_y, d_x) from (1, 1) to (4, 4) and spaces of
// 620 to 16 000 points, at as many blocks.
//   8 waves against 4, 700 / 800 / 900 / 1 000: k = 1 0.995 / 1.034 / 1.100 / 1.116, k = 4 0.956 / 0.994 / 1.041 / 1.055,
//     k = 8 0.971 / 1.016 / 1.056 / 1.067 (large spaces gain longer: five of 10 240 points, (3, 3), 198 against 231 us)
//   2 waves against 4, 3 000 / 4 100 / 6 200: k = 1 0.955 / 0.931 / 0.886, k = 4 1.007 / 0.978 / 0.938, k = 6 1.023 /
//     0.989 / 0.947
//   2 waves against persistent ones and one queue, 8 200 / 12 500 / 16 400 / 25 000: k = 1 0.799 / 0.877 / 0.933 /
//     0.997, k = 3 0.875 / 0.944 / 0.997 / 1.060, k = 4 0.905 / 0.966 / 1.025 / 1.082, k = 6 1.026 / 1.076 / 1.131 / 1.202;
//     queues, 16 400 / 24 600 / 32 800 / 49 000: k = 1 0.50 / 0.70 / 0.75 / 0.85, k = 4 0.61 / 0.82 / 0.87 / 0.97,
//     k = 6 0.74 / 0.96 / 1.01 / 1.11, k = 8 0.82 / 1.05 / 1.10 / 1.21 (the line is where spaces of
//     15 500 points stop gaining: 0.90 / 0.98 / 1.13 at k = 4)
//   4 waves against persistent ones and one queue, 2 000 / 3 000 / 4 100 / 6 200: k = 8 0.820 / 0.940 / 0.997 / 1.101,
//     k = 9 0.884 / 0.994 / 1.050, k = 12 0.969 / 1.092 / 1.147, k = 15 1.045 / 1.206 / 1.259;
//     queues, 6 200 / 8 200 / 12 500 / 16 400: k = 9 0.77 / 0.95 / 1.00 / 1.10, k = 12 0.88 / 1.08 / 1.13 / 1.24,
//     k = 15 0.99 / 1.21 / 1.26 / 1.37
//   sets (queues), 8 / 4 / 2 waves against persistent ones:
//     (1, 1) 512 / 700 / 1 000 blocks 0.51 / 0.54 / 0.81, 0.56 / 0.55 / 0.78, 0.69 / 0.59 / 0.75; 3 000 / 9 200 / 12 500
//       1.09 / 0.83 / 0.86, 1.40 / 0.97 / 0.89, 1.62 / 1.11 / 0.99
//     (2, 2) 0.46 / 0.48 / 0.76, 0.51 / 0.50 / 0.74, 0.66 / 0.58 / 0.75; 1.24 / 0.93 / 0.98, 1.60 / 1.09 / 1.00,
//       1.74 / 1.16 / 1.04
//     (3, 3) 0.41 / 0.43 / 0.68, 0.45 / 0.44 / 0.67, 0.57 / 0.51 / 0.67; 1.13 / 0.96 / 1.01, 1.50 / 1.18 / 1.09
//     (4, 4) 0.39 / 0.43 / 0.66, 0.43 / 0.44 / 0.65, 0.57 / 0.50 / 0.68; 1.10 / 0.94 / 1.07, 1.39 / 1.10 / 1.20
// A set's pairs of up to nine coordinates leave the persistent waves idle up to 9 000 blocks, wider ones do not.
int waves_to_a_block(int64_t n_items, int set_coords, int k, bool queues)
{
    if (set_coords > 0)
        return n_items <= 704 ? 8 : (n_items <= 3072 ? 4 : (set_coords <= 9 && n_items <= 9216 ? 2 : 0));
    if (k > 8) {
        const int four = k <= 11 ? (queues ? 12288 : 3072) : (queues ? 6144 : 2048);
        return n_items <= four ? 4 : 0;
    }
    if (n_items <= 832)
        return 8;
    if (n_items <= 4096)
        return 4;
    const int two = queues ? (k <= 6 ? 24576 : 16384) : (k <= 3 ? 20480 : k == 4 ? 14336 : k <= 6 ? 8192 : 0);
    return n_items <= two ? 2 : 0;
}

// The search with w waves to a block (w from waves_to_a_block, not 0): one workgroup of w waves per item.
ordered_search pick_shared(int d_y, int d_x, int k, bool sets, int w)
{
    return ordered_search{pick(d_y, d_x, k, 1, sets, w), lds_bytes(d_y, d_x, sets, w)};
}

}  // namespace te

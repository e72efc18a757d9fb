// te_search_small_k.hip -- the search kernels over single chunks at k <= 8 (k = 4 has its own).

#include "te_search.h"

namespace te {

namespace {

template <int W>
search_fn pick_cap(int d_y, int d_x, int k)
{
    return k < 4 ? pick_single<5, true, 1, W>(d_y, d_x) : pick_single<9, true, 1, W>(d_y, d_x);
}

}  // namespace

search_fn pick_search_small_k(int d_y, int d_x, int k, int w)
{
    switch (w) {
    case 0: return pick_cap<0>(d_y, d_x, k);
    case 2: return pick_cap<2>(d_y, d_x, k);
    case 4: return pick_cap<4>(d_y, d_x, k);
    case 8: return pick_cap<8>(d_y, d_x, k);
    default: return nullptr;
    }
}

}  // namespace te

// te_search_sets.hip -- the search kernels over sets of a window's chunks (k = 4).

#include "te_search.h"

namespace te {

namespace {

template <int SLOTS, int W>
search_fn pick_sets(int d_y, int d_x)
{
#define TE_KERNEL(A, B) search_sets_kernel<A, B, set_variants(A, B), SLOTS, W>
    TE_SEARCH_KERNELS(TE_KERNEL);
#undef TE_KERNEL
}

}  // namespace

search_fn pick_search_sets(int d_y, int d_x, int slots, int w)
{
    switch (w) {
    case 0: return slots == 1 ? pick_sets<1, 0>(d_y, d_x) : pick_sets<2, 0>(d_y, d_x);
    case 2: return pick_sets<1, 2>(d_y, d_x);
    case 4: return pick_sets<1, 4>(d_y, d_x);
    case 8: return pick_sets<1, 8>(d_y, d_x);
    default: return nullptr;
    }
}

}  // namespace te

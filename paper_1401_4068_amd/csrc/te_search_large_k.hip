// te_search_large_k.hip -- the search kernels over single chunks at any k up to kMaxK.

#include "te_search.h"

namespace te {

search_fn pick_search_large_k(int d_y, int d_x, int w)
{
    switch (w) {
    case 0: return pick_single<kMaxK + 1, true, 1, 0>(d_y, d_x);
    case 4: return pick_single<kMaxK + 1, true, 1, 4>(d_y, d_x);
    default: return nullptr;
    }
}

}  // namespace te

// The merge kernel (merge.hpp) instantiated for coordinate lists.
#include "merge.hpp"

namespace nacho {

hipError_t merge_coo(int dtype, bool multiply, const MergeLaunch &a)
{
    return multiply ? launch_types<SPADD_COO, true>(dtype, a) : launch_types<SPADD_COO, false>(dtype, a);
}

}  // namespace nacho

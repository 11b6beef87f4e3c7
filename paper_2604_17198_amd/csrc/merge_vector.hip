// The merge kernel (merge.hpp) instantiated for sparse vectors.
#include "merge.hpp"

namespace nacho {

hipError_t merge_vector(int dtype, bool multiply, const MergeLaunch &a)
{
    return multiply ? launch_types<SPADD_VECTOR, true>(dtype, a) : launch_types<SPADD_VECTOR, false>(dtype, a);
}

hipError_t merge_vector_search(int dtype, const MergeLaunch &a)
{
    return launch_types<SPADD_VECTOR, false, false, true>(dtype, a);
}

}  // namespace nacho

// The merge kernel (merge.hpp) instantiated for DCSR sums.
#include "merge.hpp"

namespace nacho {

hipError_t merge_dcsr(int dtype, const MergeLaunch &a) { return launch_types<SPADD_DCSR, false>(dtype, a); }

}  // namespace nacho

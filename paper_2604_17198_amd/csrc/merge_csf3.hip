// The merge kernel (merge.hpp) instantiated for third-order tensors.
#include "merge.hpp"

namespace nacho {

hipError_t merge_csf3(int dtype, const MergeLaunch &a) { return launch_types<SPADD_CSF3, false>(dtype, a); }

}  // namespace nacho

// The merge kernel (merge.hpp) instantiated for CSR sums.
#include "merge.hpp"

namespace nacho {

hipError_t merge_csr(int dtype, const MergeLaunch &a) { return launch_types<SPADD_CSR, false>(dtype, a); }

}  // namespace nacho

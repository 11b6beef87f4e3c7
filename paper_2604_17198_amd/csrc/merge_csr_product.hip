// The merge kernel (merge.hpp) instantiated for CSR products.
#include "merge.hpp"

namespace nacho {

hipError_t merge_csr_product(int dtype, const MergeLaunch &a) { return launch_types<SPADD_CSR, true>(dtype, a); }

}  // namespace nacho

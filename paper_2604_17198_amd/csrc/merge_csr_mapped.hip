// The merge kernel (merge.hpp) instantiated for DCSR products (remapped CSR operands).
#include "merge.hpp"

namespace nacho {

hipError_t merge_csr_mapped(int dtype, const MergeLaunch &a) { return launch_types<SPADD_CSR, true, true>(dtype, a); }

}  // namespace nacho

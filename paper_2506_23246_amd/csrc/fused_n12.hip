// Instantiation of the fused kernel for 12 qubits.
#include "fused_kernel.hpp"

namespace qp {
hipError_t launch_fused_12(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st) {
  return launch_fused_n<12>(mode, a, grid, exs, dyn, st);
}
}  // namespace qp

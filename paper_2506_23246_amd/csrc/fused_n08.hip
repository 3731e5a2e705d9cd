// Instantiation of the fused kernel for 8 qubits.
#include "fused_kernel.hpp"

namespace qp {
hipError_t launch_fused_8(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st) {
  return launch_fused_n<8>(mode, a, grid, exs, dyn, st);
}
}  // namespace qp

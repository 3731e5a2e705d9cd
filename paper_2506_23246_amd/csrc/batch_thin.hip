// The uneven batch's class kernels for batches with thin circuits.
#include <hip/hip_runtime.h>

#include "batch_kernel.hpp"

namespace qp {

hipError_t launch_batch_thin(int seg, int grid, size_t dyn, hipStream_t s, const BatchCirc* circs, const BatchItem* items,
                             int nitems, int* counter, float* mpart, float* lpart) {
  return launch_batch_class<true>(seg, grid, dyn, s, circs, items, nitems, counter, mpart, lpart);
}

hipError_t prepare_batch_thin(int max_cols, int max_cols_big) { return prepare_batch_classes<true>(max_cols, max_cols_big); }

}  // namespace qp

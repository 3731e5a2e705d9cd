// Uniform, read-only kernel data (plan, tables) is read through the constant address space, so the
// compiler emits scalar loads (SGPRs) instead of per-lane vector loads that stall a wave.
#pragma once
#include <hip/hip_runtime.h>

namespace qp {

#define QP_CONST __attribute__((address_space(4)))
template <typename T> using CP = const QP_CONST T*;
template <typename T> __device__ __forceinline__ CP<T> to_const(const T* p) { return (CP<T>)(p); }

}  // namespace qp

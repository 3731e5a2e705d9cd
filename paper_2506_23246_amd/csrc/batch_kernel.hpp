// Persistent tile kernel of the uneven batch: one instantiation per qubit-count class.
#pragma once
#include <hip/hip_runtime.h>

#include "batch.hpp"
#include "fused_kernel.hpp"

namespace qp {

// Two exchange planes: the function holds every qubit count's tile code of its class under one
// 256-VGPR cap; with four planes the all-counts kernel spilled 292 bytes per lane, whose scratch
// (38 MB over 2048 waves) overflowed the L2 and nearly doubled the kernel's HBM traffic.
constexpr int kBEXS = 2;

// Dynamic LDS of a T-thread k_batch: per-wave gate statistics, phase moments, readout scratch.
inline size_t batch_dyn_lds_bytes(int T, int max_cols) {
  return (size_t)(T / 64) * max_cols * sizeof(float) + (size_t)(T / 64) * 40 * sizeof(float);
}

// The tiles of one work item.
template <int N, int NLO, int NHI, int T, bool THIN>
__device__ __forceinline__ void batch_case(const BatchCirc& C, const BatchItem& it, float2* buf, float* slots,
                                           float* mslots, float* red, float& lacc) {
  if constexpr (NLO <= N && N <= NHI) {
    for (int t = it.tile0; t < it.tile0 + it.ntile; ++t)
      fused_tile<N, T, kBEXS, kModeMaxwell, false, THIN && (N >= kThinQubits)>(C.a, t, buf, slots, mslots, red, lacc);
  }
}

// One kernel per class of qubit counts [NLO, NHI] on T-thread workgroups: each class's tile code
// gets its own register allocation, at the 256-VGPR cap all the same: 3..8, 9..11 and 12 qubits spill 201, 145
// and 83 VGPRs (396, 372 and 260 bytes a lane; 312 MB of HBM traffic a launch of the 32-circuit, 4..10-qubit batch
// for 38 MB of inputs and results), where a kernel of one count spills 2 to 4 up to 9 qubits: the tile bodies are
// inlined into one function.  12 qubits need 512 threads: a tile is one point on 512 threads.
template <int NLO, int NHI, int T, bool THIN>
__global__ __launch_bounds__(T, 2) void k_batch(const BatchCirc* __restrict__ circs, const BatchItem* __restrict__ items,
                                             int nitems, int* __restrict__ counter, float* __restrict__ mpart,
                                             float* __restrict__ lpart) {
  constexpr int WAVES = T / 64;
  constexpr int PLANE = T * 8;
  __shared__ float4 planes[kBEXS * PLANE / 2];   // exchange planes (see fused_tile)
  extern __shared__ float4 smem4[];
  float2* buf = reinterpret_cast<float2*>(planes);
  float* slots = reinterpret_cast<float*>(smem4);
  __shared__ int s_item;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (;;) {
    if (tid == 0) s_item = atomicAdd(counter, 1);
    __syncthreads();
    const int id = s_item;
    __syncthreads();
    if (id >= nitems) break;
    const BatchItem it = items[id];
    const BatchCirc& C = circs[it.circ];
    const int F = C.F, NM = C.a.n_mom;
    float* mslots = slots + WAVES * F * kGS;   // [WAVES][F][kGS] statistics, [WAVES][NM] moments
    float* red = mslots + WAVES * NM;
    for (int i = tid; i < WAVES * (F * kGS + NM); i += T) slots[i] = 0.f;
    __syncthreads();
    float lacc = 0.f;
    switch (C.n) {
      case 3: batch_case<3, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 4: batch_case<4, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 5: batch_case<5, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 6: batch_case<6, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 7: batch_case<7, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 8: batch_case<8, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 9: batch_case<9, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 10: batch_case<10, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 11: batch_case<11, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      case 12: batch_case<12, NLO, NHI, T, THIN>(C, it, buf, slots, mslots, red, lacc); break;
      default: break;
    }
    __syncthreads();
    const int ncol = F * kGS + NM;
    float* mp = mpart + C.mpart_off + (long long)it.slot * ncol;
    for (int i = tid; i < F * kGS; i += T) {
      float s = 0.f;
      for (int w = 0; w < WAVES; ++w) s += slots[w * F * kGS + i];
      mp[i] = s;
    }
    for (int i = tid; i < NM; i += T) {
      float s = 0.f;
      for (int w = 0; w < WAVES; ++w) s += mslots[w * NM + i];
      mp[F * kGS + i] = s;
    }
    for (int off = 32; off >= 1; off >>= 1) lacc += __shfl_xor(lacc, off);
    if (lane == 0) red[wave * 40] = lacc;
    __syncthreads();
    if (tid == 0) {
      float s = 0.f;
      for (int w = 0; w < WAVES; ++w) s += red[w * 40];
      lpart[C.item_lp0 + it.slot] = s;
    }
    __syncthreads();
  }
}

// Launches the class kernel of segment `seg` (see BatchSegment) on `grid` workgroups, and its dynamic LDS limit.
template <bool THIN>
hipError_t launch_batch_class(int seg, int grid, size_t dyn, hipStream_t s, const BatchCirc* circs, const BatchItem* items,
                              int nitems, int* counter, float* mpart, float* lpart) {
  switch (seg) {
    case kSegLo:
      hipLaunchKernelGGL((k_batch<3, kBatchSplit, 256, THIN>), dim3(grid), dim3(256), dyn, s, circs, items, nitems,
                         counter, mpart, lpart);
      break;
    case kSegHi:
      hipLaunchKernelGGL((k_batch<kBatchSplit + 1, 11, 256, THIN>), dim3(grid), dim3(256), dyn, s, circs, items,
                         nitems, counter, mpart, lpart);
      break;
    case kSegBig:
      hipLaunchKernelGGL((k_batch<kBatchBig, kBatchBig, 512, THIN>), dim3(grid), dim3(512), dyn, s, circs, items,
                         nitems, counter, mpart, lpart);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template <bool THIN>
hipError_t prepare_batch_classes(int max_cols, int max_cols_big) {
  const int lds = (int)batch_dyn_lds_bytes(256, max_cols), lds_big = (int)batch_dyn_lds_bytes(512, max_cols_big);
  hipError_t e = hipSuccess;
  if (max_cols > 0) {
    e = hipFuncSetAttribute((const void*)k_batch<3, kBatchSplit, 256, THIN>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)k_batch<kBatchSplit + 1, 11, 256, THIN>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  }
  if (e == hipSuccess && max_cols_big > 0)
    e = hipFuncSetAttribute((const void*)k_batch<kBatchBig, kBatchBig, 512, THIN>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds_big);
  return e;
}
// A batch with a thin circuit runs the kernels with thin layers (in a unit of their own, so that they compile
// in parallel): with its branches the 32-circuit, 4..10-qubit batch of full layers takes 16.3 ms, without 15.8.
hipError_t launch_batch_thin(int seg, int grid, size_t dyn, hipStream_t s, const BatchCirc* circs, const BatchItem* items,
                             int nitems, int* counter, float* mpart, float* lpart);
hipError_t prepare_batch_thin(int max_cols, int max_cols_big);
}  // namespace qp

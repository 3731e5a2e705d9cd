// Fused per-point circuit kernels for gfx950 (MI355X): helper kernels and dispatch.
// The fused kernel template itself is in fused_kernel.hpp (see the description below).
//
// One workgroup evaluates a tile of collocation points.  Every point's statevector psi and its
// three input tangents dpsi_t, dpsi_x, dpsi_y (and, in the adjoint, lambda and mu_t, mu_x, mu_y)
// live in registers: a thread owns 8 amplitudes of each statevector, addressed by three
// "register" index bits; the other n-3 index bits select the thread inside the point's thread
// group.  The circuit runs as sweep layers (QSweep): an exchange through LDS that applies the
// CNOT index map, one tabulated phase per amplitude, and one real rotation per qubit.
//
// Forward-mode tangents: a gate U acts on psi and on each dpsi_c identically because the
// variational gates do not depend on the input point; only the encoding does, and its derivative
// seeds dpsi at the start.  Readout: f_i = sum_j z_i(j)|psi_j|^2,
// g_ic = 2 sum_j z_i(j) Re(conj(psi_j) dpsi_c,j) (section "QPINN architecture": Pauli-Z per qubit).
//
// Adjoint with uncompute: with lambda = dL/dpsi*, mu_c = dL/d(dpsi_c)* at the circuit end, each layer
// (in reverse order) takes psi, dpsi_c, lambda, mu_c back through its inverse and adds per gate
//   S_k = Im <lambda|sigma_k|psi> + sum_c Im <mu_c|sigma_k|dpsi_c>, k = x, y, z;
// the parameter gradient is a fixed contraction of S (grads_dev.hpp), after the FP64 reduction.
//
// Arithmetic is complex64 with FP32 accumulation; per-workgroup partials are reduced across
// workgroups in a fixed order in FP64 (separate kernels), so results are deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "qp_internal.hpp"
#include "fused.hpp"
#include "grads_dev.hpp"
#include "rot_dev.hpp"
#include "sweep_tables_dev.hpp"

namespace qp {


hipError_t launch_fused_3(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_4(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_5(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_6(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_7(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_8(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_9(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_10(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_11(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
hipError_t launch_fused_12(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);

// Tables of the sweep layers (FP64, once per call; fp32: the gate matrices formed in FP32, kept for
// comparison, QP_FLAG_GATES_FP32).
__global__ __launch_bounds__(kTabThreads) void k_sweep_tables(SweepPlan plan, const float* __restrict__ params,
                                                              SweepTabs t, int fp32) {
  sweep_tables(plan, params, t, blockIdx.x, fp32);
}

// Random-Fourier-feature angles: phi = [cos(Bp); sin(Bp)], theta = W phi, J = W dphi/dp.
//
// A workgroup takes 32 points.  Chunk by chunk its threads form the features' sines (one per thread and
// step), then a thread per point and qubit adds the chunk up, feature by feature.  With a thread per
// point doing both, 65536 points were one wave per SIMD, waiting on its own chain (8 qubits, 64 features:
// 86 -> 20 us).
constexpr int kRffPoints = 32, kRffChunk = 32, kRffThreads = 256;
__global__ __launch_bounds__(kRffThreads) void k_rff_angles(const QPlanDev* __restrict__ plan,
                                                            const float* __restrict__ points, long long P,
                                                            float* __restrict__ angles, float* __restrict__ jac) {
  __shared__ float2 cs[kRffChunk][kRffPoints];
  __shared__ float sB[kRffChunk][3];
  const char* pb = reinterpret_cast<const char*>(plan);
  const float* B = reinterpret_cast<const float*>(pb + plan->off_rff_B);
  const float* W = reinterpret_cast<const float*>(pb + plan->off_rff_W);
  const int n = plan->n, F = plan->n_feat, tid = threadIdx.x;
  const int i = tid % kRffPoints, q0 = tid / kRffPoints;
  constexpr int kQ = kRffThreads / kRffPoints, kPer = (kMaxQubits + kQ - 1) / kQ;   // qubits q0, q0 + kQ, ..
  const long long p = (long long)blockIdx.x * kRffPoints + i;
  float t = 0.f, x = 0.f, y = 0.f;
  if (p < P) { t = points[p * 3]; x = points[p * 3 + 1]; y = points[p * 3 + 2]; }
  float th[kPer], j0[kPer], j1[kPer], j2[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) th[e] = j0[e] = j1[e] = j2[e] = 0.f;
  for (int f0 = 0; f0 < F; f0 += kRffChunk) {
    const int nf = F - f0 < kRffChunk ? F - f0 : kRffChunk;
    __syncthreads();   // the chunk before is read
    for (int k = tid; k < nf * 3; k += kRffThreads) sB[k / 3][k % 3] = B[f0 * 3 + k];
    for (int k = q0; k < nf; k += kQ) {
      const float b0 = B[(f0 + k) * 3], b1 = B[(f0 + k) * 3 + 1], b2 = B[(f0 + k) * 3 + 2];
      const float pr = b0 * t + b1 * x + b2 * y;
      float s, c;
      sincosf(pr, &s, &c);
      cs[k][i] = make_float2(c, s);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int q = q0 + e * kQ;
      if (q >= n) break;
      const float* w = W + (size_t)q * 2 * F + f0;
      for (int k = 0; k < nf; ++k) {
        const float wc = w[k], ws = w[F + k];
        const float c = cs[k][i].x, s = cs[k][i].y;
        th[e] += wc * c + ws * s;
        const float dd = ws * c - wc * s;   // d/dproj of (wc cos + ws sin)
        j0[e] += dd * sB[k][0]; j1[e] += dd * sB[k][1]; j2[e] += dd * sB[k][2];
      }
    }
  }
  if (p >= P) return;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int q = q0 + e * kQ;
    if (q >= n) break;
    angles[p * n + q] = th[e];
    jac[(p * n + q) * 3 + 0] = j0[e];
    jac[(p * n + q) * 3 + 1] = j1[e];
    jac[(p * n + q) * 3 + 2] = j2[e];
  }
}

// Number of points in the dielectric half (x >= x_if); one workgroup, deterministic.
__global__ void k_count_diel(const float* __restrict__ points, long long P, float x_if, int* __restrict__ counts) {
  __shared__ int sh[16];
  int c = 0;
  for (long long p = threadIdx.x; p < P; p += blockDim.x) c += points[p * 3 + 1] >= x_if ? 1 : 0;
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sh[w];
    counts[0] = (int)(P - s);
    counts[1] = s;
  }
}

// FP64 cross-workgroup reduction of the M partials (one wave per entry) and of the loss.
__global__ void k_reduce_m(const float* __restrict__ mpart, int nblk, int ncol,
                           const float* __restrict__ lpart, double* __restrict__ m64,
                           double* __restrict__ loss) {
  const int col = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (col > ncol) return;
  double s = 0.0;
  if (col < ncol) {
    for (int b = lane; b < nblk; b += 64) s += (double)mpart[(long long)b * ncol + col];
  } else if (lpart) {
    for (int b = lane; b < nblk; b += 64) s += (double)lpart[b];
  }
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) {
    if (col < ncol) m64[col] = s;
    else if (loss) *loss = s;
  }
}

// d L / d theta_k for every parameter (FP64; see grads_dev.hpp).
__global__ void k_param_grads(const QPlanDev* __restrict__ plan, const float* __restrict__ params,
                              const double* __restrict__ m64, SweepTabs t, float* __restrict__ grads) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= plan->n_params) return;
  grads[k] = (float)param_grad_one(plan, params, m64, t, k);
}

int fused_threads(int n) { return fused_wg_threads(n); }
int fused_max_wg_per_cu(int n) { return fused_threads(n) == 512 ? 1 : 4; }
int fused_points_per_tile(int n) { return fused_threads(n) / (1 << (n - 3)); }
size_t fused_lds_bytes(int n, int exs, int n_fused, int n_mom) {
  const int T = fused_threads(n);
  return (size_t)exs * T * 8 * sizeof(float2) + (size_t)(T / 64) * (n_fused * kGS + n_mom) * sizeof(float) +
         (size_t)(T / 64) * 40 * sizeof(float);
}

size_t fused_dyn_lds(int n, int n_fused, int n_mom) {
  return (size_t)(fused_threads(n) / 64) * (n_fused * kGS + n_mom + 40) * sizeof(float);
}

hipError_t launch_fused(int n, int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st) {
  switch (n) {
    case 3: return launch_fused_3(mode, a, grid, exs, dyn, st);
    case 4: return launch_fused_4(mode, a, grid, exs, dyn, st);
    case 5: return launch_fused_5(mode, a, grid, exs, dyn, st);
    case 6: return launch_fused_6(mode, a, grid, exs, dyn, st);
    case 7: return launch_fused_7(mode, a, grid, exs, dyn, st);
    case 8: return launch_fused_8(mode, a, grid, exs, dyn, st);
    case 9: return launch_fused_9(mode, a, grid, exs, dyn, st);
    case 10: return launch_fused_10(mode, a, grid, exs, dyn, st);
    case 11: return launch_fused_11(mode, a, grid, exs, dyn, st);
    case 12: return launch_fused_12(mode, a, grid, exs, dyn, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_sweep_tables(const SweepPlan& plan, bool phases, const float* params, const SweepTabs& t, int fp32,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_sweep_tables, dim3(sweep_table_blocks(plan.n, plan.n_sweeps - plan.sweep_first, phases)), dim3(kTabThreads), 0, st, plan, params, t, fp32);
  return hipGetLastError();
}

hipError_t launch_rff(const QPlanDev* plan, const float* points, long long P, float* angles, float* jac, hipStream_t st) {
  if (P == 0) return hipSuccess;
  hipLaunchKernelGGL(k_rff_angles, dim3((unsigned)((P + kRffPoints - 1) / kRffPoints)), dim3(kRffThreads), 0, st, plan, points, P, angles, jac);
  return hipGetLastError();
}

hipError_t launch_count(const float* points, long long P, float x_if, int* counts, hipStream_t st) {
  hipLaunchKernelGGL(k_count_diel, dim3(1), dim3(1024), 0, st, points, P, x_if, counts);
  return hipGetLastError();
}

hipError_t launch_reduce(const float* mpart, int nblk, int ncol, const float* lpart, double* m64, double* loss, hipStream_t st) {
  const int cols = ncol + 1;   // + loss
  const int waves_per_block = 4;
  hipLaunchKernelGGL(k_reduce_m, dim3((cols + waves_per_block - 1) / waves_per_block), dim3(64 * waves_per_block), 0, st,
                     mpart, nblk, ncol, lpart, m64, loss);
  return hipGetLastError();
}

hipError_t launch_param_grads(const QPlanDev* plan, int K, const float* params, const double* m64, const SweepTabs& t,
                              float* grads, hipStream_t st) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_param_grads, dim3((K + 127) / 128), dim3(128), 0, st, plan, params, m64, t, grads);
  return hipGetLastError();
}

}  // namespace qp

// Launch interface of the fused register/LDS kernels (fused.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../../include/qpinn.h"
#include "qp_internal.hpp"

namespace qp {

// Per-call tables of the sweep layers (sweep_tables_dev.hpp).
struct SweepTabs {
  float* gtab;       // [F + 1][kGT] gate matrices U (entry F: identity), then the coefficients of the
                     // rounds' phase stages (32-bit fractions of a turn)
  float* tcoef;      // [n_sweeps][kTC] tan(b/2) by position
  float2* ptab;      // [n_sweeps - sweep_first + 1][2^n] phase times cosines, [thread][register]; last: behind the last layer
  double* gpar;      // [F][kGP] how a gate's statistics are read
  double* lscale;    // [n_sweeps] scale of a layer's diagonal sums
  uint32_t* xmask;   // [n_sweeps + 1] X mask of each layer; last: of the product state
};

// What the table kernel needs of the plan's header, passed by value (one dependent load less).
struct SweepPlan {
  const QPlanDev* plan;
  int32_t n, n_params, n_fused, n_sweeps, sweep_first, off_fused, off_sweeps;
};

struct FusedArgs {
  const QPlanDev* plan;
  const float* gtab;      // SweepTabs
  const float* tcoef;
  const float2* ptab;
  const uint32_t* xmask;
  const float* points;    // [P][3]
  const float* angles;    // [P][n]   (angle-given or RFF encodings)
  const float* jac;       // [P][n][3]
  long long P;
  int ntiles;
  int n_gates;            // fused gates (n_fused: those with statistics, 0 in the forward modes)
  int n_fused;
  float* out;             // [P][m] or null
  float* tan;             // [P][m][3] or null
  const float* d_out;     // VJP seeds [P][m] or null
  const float* d_tan;     // VJP seeds [P][m][3] or null
  int loss_kind;
  int loss_sum;           // 1: plain sums (weights 1) instead of means
  float eps_r, x_if;
  const int* counts;      // [2]: points with x < x_if, points with x >= x_if
  float* mpart;           // [grid][F][kGS]
  float* lpart;           // [grid]
  float* d_angles;        // [P][n] dL/d angles (angle-given encoding) or null
  float* d_jac;           // [P][n][3] dL/d Jacobian or null
  int thin;               // the circuit's layers leave positions out
  int n_mom;              // phase-stage moments per workgroup partial (after the F * kGS statistics)
  const float* f_mir;     // kModeTotal: outputs of the mirror images [n_mir][P][m] (y-mirror first)
  int n_mir;              // kModeTotal: 1 (y-mirror) or 2 (and x-mirror)
  float w_sym, w_energy;  // kModeTotal: weights of the symmetry and energy terms
};

int fused_threads(int n);
// Largest persistent grid, in workgroups per CU, that a launch may ask for: one 512-thread
// workgroup (12 qubits) or four 256-thread ones.  About 256 VGPRs per lane keep two waves per
// SIMD resident, so a grid above two 256-thread workgroups per CU runs in generations.
int fused_max_wg_per_cu(int n);
int fused_points_per_tile(int n);
// LDS of a launch shape as the shape rules count it: exs planes, statistics, scratch.
size_t fused_lds_bytes(int n, int exs, int n_fused, int n_mom);
// Dynamic LDS of a launch (statistics and scratch; the planes are static).
size_t fused_dyn_lds(int n, int n_fused, int n_mom);
hipError_t launch_fused(int n, int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st);
// Blocks of one circuit's tables: the gate matrices, 256 entries each of the layers' phases (and of the
// one behind the last layer), and the rounds' phase stages if it has any.
QP_HD inline int sweep_table_blocks(int n, int layers, bool phases) {
  return 1 + (layers + 1) * ((1 << n) > 256 ? (1 << n) / 256 : 1) + (phases ? 1 : 0);
}
hipError_t launch_sweep_tables(const SweepPlan& plan, bool phases, const float* params, const SweepTabs& t, int fp32,
                               hipStream_t st);
hipError_t launch_rff(const QPlanDev* plan, const float* points, long long P, float* angles, float* jac, hipStream_t st);
hipError_t launch_count(const float* points, long long P, float x_if, int* counts, hipStream_t st);
hipError_t launch_reduce(const float* mpart, int nblk, int ncol, const float* lpart, double* m64, double* loss, hipStream_t st);
hipError_t launch_param_grads(const QPlanDev* plan, int K, const float* params, const double* m64, const SweepTabs& t,
                              float* grads, hipStream_t st);

}  // namespace qp

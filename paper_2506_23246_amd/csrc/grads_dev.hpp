// Parameter gradient from the reduced gate statistics (FP64, the final reduction stage).
// A fused gate is U = R_{c-1} ... R_0 with R = exp(-i theta P / 2), so dU/dtheta_c = U (-i/2) G_c
// with the rotated generator G_c = W^H P_c W, W = R_{c-1} ... R_0 (the components before c).
// With lambda and psi both taken before the gate,
//   d L / d theta_c = 2 Re <lambda_after| dU |psi> = Im <lambda|G_c|psi> = sum_k n_k S_k,
// where G_c = n_x X + n_y Y + n_z Z and S_k = Im <lambda|sigma_k|psi> is what the adjoint sweep
// accumulates per gate, there behind the RZ(c) of the gate's ZYZ split (QSweep), so G_c's axis is
// turned about z by c.  A gate of the opening layer has its statistic taken after the gate
// (lambda_after, psi_after = U psi); the same derivative is then Im <lambda_after|G'_c|psi_after>
// with G'_c = U G_c U^H = V P_c V^H, V = R_{n-1} ... R_{c+1} the components after c (R_c
// commutes with P_c).
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/qpinn.h"
#include "qp_internal.hpp"
#include "fused.hpp"
#include "rot_dev.hpp"

namespace qp {

// Axis (n_x, n_y, n_z) of V P V^H, V = [[a, -b*], [b, a*]] by its first column.
__device__ inline void pauli_axis(int kind, double2 a, double2 b, double* n) {
  const double2 ab = make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
  const double ap = a.x * a.x - a.y * a.y, aq = -2.0 * a.x * a.y;   // (a*)^2
  const double bp = b.x * b.x - b.y * b.y, bq = 2.0 * b.x * b.y;    // b^2
  const bool x = kind == QP_RX, y = kind == QP_RY;
  n[0] = x ? ap - bp : (y ? -(aq + bq) : 2.0 * (a.x * b.x + a.y * b.y));
  n[1] = x ? aq - bq : (y ? ap + bp : 2.0 * (a.x * b.y - a.y * b.x));
  n[2] = x ? -2.0 * ab.x : (y ? -2.0 * ab.y : a.x * a.x + a.y * a.y - b.x * b.x - b.y * b.y);
}

__device__ inline double param_grad_one(const QPlanDev* __restrict__ plan, const float* __restrict__ params,
                                        const double* __restrict__ s64, const SweepTabs& T, int k) {
  const char* pb = reinterpret_cast<const char*>(plan);
  const QFused* fused = reinterpret_cast<const QFused*>(pb + plan->off_fused);
  const int* ptr = reinterpret_cast<const int*>(pb + plan->off_csr_ptr);
  const int* idx = reinterpret_cast<const int*>(pb + plan->off_csr_idx);
  double gsum = 0.0;
  for (int e = ptr[k]; e < ptr[k + 1]; ++e) {
    // (one fetch of all that belongs to the gate, then one of its parameters: the kernel is a chain of fetches)
    const int fi = idx[e] >> 2, ci = idx[e] & 3;
    const QFused fu = fused[fi];
    const double* S = s64 + fi * kGS;
    const double* g = T.gpar + (long long)fi * kGP;
    const double Sx = S[0], Sy = S[1], Sz = S[2], gc = g[0], gs = g[1], gxy = g[2], gz = g[3];
    // the components after c (statistic behind the gate) or before it: V P V^H or W^H P W, W^H of first column
    // (a*, -b)
    const int c0 = fu.head ? ci + 1 : 0, c1 = fu.head ? fu.ncomp : ci;
    float th[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) th[c] = params[c < fu.ncomp ? fu.param[c] : fu.param[0]];
    double2 a = make_double2(1.0, 0.0), b = make_double2(0.0, 0.0);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int c = c0 + o;
      if (c >= c1) break;
      double sn, cs;
      sincos(0.5 * (double)(c == 0 ? th[0] : (c == 1 ? th[1] : th[2])), &sn, &cs);
      column_rot(c == 0 ? fu.kind[0] : (c == 1 ? fu.kind[1] : fu.kind[2]), cs, sn, a, b);
    }
    if (!fu.head) { a.y = -a.y; b.x = -b.x; b.y = -b.y; }
    double nv[3];
    pauli_axis(ci == 0 ? fu.kind[0] : (ci == 1 ? fu.kind[1] : fu.kind[2]), a, b, nv);
    // the cosines left out when the statistics were taken, and the sign of Y and Z behind an X mask
    const double nx = gc * nv[0] - gs * nv[1], ny = gs * nv[0] + gc * nv[1];
    gsum += nx * Sx * gxy + (gz < 0.0 ? -ny : ny) * Sy * gxy + nv[2] * Sz * gz;
  }
  // CRZ(c, t) occurrences: dL/dtheta = (W_t - W_ct) / 2 from the layer's parity sums, which follow the
  // fused-gate statistics (see QPhaseStage)
  if (plan->n_phase > 0) {
    const int* pptr = reinterpret_cast<const int*>(pb + plan->off_pcsr_ptr);
    const int* pidx = reinterpret_cast<const int*>(pb + plan->off_pcsr_idx);
    const QPhaseStage* stages = reinterpret_cast<const QPhaseStage*>(pb + plan->off_phase);
    const QPhaseGate* pg = reinterpret_cast<const QPhaseGate*>(pb + plan->off_phase_gates);
    const QSweep* sweeps = reinterpret_cast<const QSweep*>(pb + plan->off_sweeps);
    const int n = plan->n;
    for (int e = pptr[k]; e < pptr[k + 1]; ++e) {
      const QPhaseGate G = pg[pidx[e]];
      const double* W = s64 + plan->n_fused * kGS + stages[sweeps[G.layer].phase].mom_off;
      const uint32_t x = T.xmask[G.layer];
      const double zc = ((x >> (n - 1 - G.c)) & 1u) ? -1.0 : 1.0, zt = ((x >> (n - 1 - G.t)) & 1u) ? -1.0 : 1.0;
      const int a = G.c < G.t ? G.c : G.t, b = G.c < G.t ? G.t : G.c;
      gsum += 0.5 * T.lscale[G.layer] * zt * (W[G.t] - zc * W[n + phase_pair_index(n, a, b)]);
    }
  }
  return gsum;
}

}  // namespace qp

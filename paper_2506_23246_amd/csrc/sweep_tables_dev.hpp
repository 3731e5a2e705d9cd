// Per-call tables of the sweep layers, formed in FP64 from the parameters and rounded once
// (independent of the point count): the tangents of the layers' rotations, the
// phase (times the rotations' cosines) of every basis index in front of each layer, the X masks, and
// what the gradient kernel needs to read the statistics.  See QSweep.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <type_traits>

#include "const_dev.hpp"
#include "fused.hpp"
#include "qp_internal.hpp"
#include "rot_dev.hpp"

namespace qp {

// U of a fused gate from its parameters.
template <typename R>
__device__ inline void fused_product(const QFused& fu, const float* __restrict__ params, R* u) {
  set_identity(u);
#pragma unroll 1
  for (int c = 0; c < fu.ncomp; ++c) {
    R s, co;
    if constexpr (sizeof(R) == 4) sincosf(0.5f * params[fu.param[c]], &s, &co);
    else sincos(0.5 * (double)params[fu.param[c]], &s, &co);
    left_mul_rot<R>(fu.kind[c], co, s, u);
  }
}

// Half angles in FP64.  sincospi of theta / (2 pi) needs no long argument reduction, but the rounding of that
// product grows with theta: up to 2^20 it is below 2^-33 turns, 2^-9 of an FP32 rounding; beyond, sincos's
// exact reduction.  (The rounds' matrices come from sincos: adjoint and forward have to be of one circuit.)
constexpr int kTabThreads = 256;   // of a block of the table kernel
constexpr double kInv2Pi = 0.15915494309189533577;
__device__ __forceinline__ bool long_angle(float theta) { return !(fabsf(theta) <= 1048576.f); }
__device__ __forceinline__ void half_angle(float theta, double* s, double* c) {
  if (__builtin_expect(long_angle(theta), 0)) sincos(0.5 * (double)theta, s, c);
  else sincospi(kInv2Pi * (double)theta, s, c);
}
// theta / (2 pi), less a multiple of 2 (theta / 2 less whole turns) for a long angle.
__device__ __forceinline__ double turns_of(float theta) {
  if (__builtin_expect(long_angle(theta), 0)) {
    double s, c;
    sincos(0.5 * (double)theta, &s, &c);
    return 2.0 * kInv2Pi * atan2(s, c);
  }
  return kInv2Pi * (double)theta;
}

// The matrix of gate f for the rounds and the encoding, formed in FP64 and rounded once (fp32: in FP32,
// kept for comparison); f = n_fused: the identity (absent gates of a round).
__device__ inline void gate_entry(const QPlanDev* __restrict__ plan, const float* __restrict__ params, int f, int fp32,
                                  float* __restrict__ gtab) {
  float* o = gtab + (size_t)f * kGT;
  if (f == plan->n_fused) {
    float u[8];
    set_identity(u);
    store_gate_entry(o, u);
    return;
  }
  const QFused& fu = (reinterpret_cast<const QFused*>(reinterpret_cast<const char*>(plan) + plan->off_fused))[f];
  if (fp32) {
    float u[8];
    fused_product<float>(fu, params, u);
    store_gate_entry(o, u);
  } else {
    double u[8];
    fused_product<double>(fu, params, u);
    store_gate_entry(o, u);
  }
}

// U = e^{i g} RZ(a) RY(b) RZ(c): u00 = e^{-i(a+c)/2} cos(b/2), u10 = e^{i(a-c)/2} sin(b/2).  The phases of
// u00 and u10 give e^{ia} and e^{ic}; RZ(a) is diag(1, e^{ia}) up to a global phase, which no result
// depends on.  flip: RY(b) = RY(pi) RY(b - pi) where |tan(b/2)| > 1; t is the tangent that is left.
struct Zyz {
  double2 a, c;   // e^{ia}, e^{ic}
  double t, cosb;
  int flip;
};
__device__ inline double2 cmul(double2 x, double2 y) { return make_double2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x); }
__device__ inline int zyz_flip(double2 u0, double2 u1) { return u1.x * u1.x + u1.y * u1.y > u0.x * u0.x + u0.y * u0.y; }
__device__ inline Zyz zyz_split(double2 u0, double2 u1) {
  Zyz z;
  const double n0 = u0.x * u0.x + u0.y * u0.y, n1 = u1.x * u1.x + u1.y * u1.y;
  const double i0 = rsqrt(n0), i1 = rsqrt(n1), r0 = n0 > 0.0 ? n0 * i0 : 0.0, r1 = n1 > 0.0 ? n1 * i1 : 0.0;
  const double2 p0 = r0 > 0.0 ? make_double2(u0.x * i0, u0.y * i0) : make_double2(1.0, 0.0);
  const double2 p1 = r1 > 0.0 ? make_double2(u1.x * i1, u1.y * i1) : make_double2(1.0, 0.0);
  const double2 q = cmul(p0, p1);
  z.a = cmul(p1, make_double2(p0.x, -p0.y));
  z.c = make_double2(q.x, -q.y);
  z.flip = zyz_flip(u0, u1);
  z.t = z.flip ? -r0 * i1 : r1 * i0;
  z.cosb = z.flip ? r1 : r0;   // (U has unit determinant)
  return z;
}

constexpr int kFlipLayers = 1024;   // layers whose flips the table kernel holds at a time

// CRZ angles of up to kTabThreads gates at a time, formed once by a block's threads and read by all: a thread that
// formed them itself went through the stage's gates one fetch and one conversion after the other (4 layers of all pairs, 7
// qubits, 42 CRZ a layer: 15.8 -> 9.2 us; 11 qubits, 110 a layer: 38.2 -> 28.2).
struct PhaseChunk {
  double turns[kTabThreads];
  uint32_t ct[kTabThreads];   // control << 8 | target
};
__device__ inline void load_phase_gates(PhaseChunk& s, const QPhaseGate* gates, const float* __restrict__ params, int count) {
  __syncthreads();   // (the chunk before is read)
  if ((int)threadIdx.x < count) {
    const QPhaseGate g = gates[threadIdx.x];
    s.turns[threadIdx.x] = turns_of(params[g.param]);
    s.ct[threadIdx.x] = (uint32_t)g.c << 8 | (uint32_t)g.t;
  }
  __syncthreads();
}

// Phase-stage coefficients of the rounds in 32-bit fractions of a turn: alpha_q = -(1/2) sum_t
// theta_qt, beta_qq' = theta_qq' + theta_q'q (see QPhaseStage), formed in FP64 (all threads of a block).
__device__ inline void phase_entries(const QPlanDev* __restrict__ plan, const float* __restrict__ params, PhaseChunk& s,
                                     uint32_t* __restrict__ coef) {
  const int n = plan->n, nt = phase_terms(n), count = plan->n_phase_coef;
  const char* pb = reinterpret_cast<const char*>(plan);
  const QPhaseStage* stages = reinterpret_cast<const QPhaseStage*>(pb + plan->off_phase);
  const QPhaseGate* gates = reinterpret_cast<const QPhaseGate*>(pb + plan->off_phase_gates);
  for (int i0 = 0; i0 < count; i0 += kTabThreads) {
    const int i = i0 + (int)threadIdx.x < count ? i0 + (int)threadIdx.x : count - 1, last = min(i0 + kTabThreads, count) - 1;
    const QPhaseStage st = stages[i / nt], end = stages[last / nt];
    const int from = stages[i0 / nt].gate0, to = end.gate0 + end.ngates;   // gates of these entries
    const int e = i % nt;
    int qa = e, qb = -1;   // alpha_qa, or beta of the pair (qa, qb)
    if (e >= n) {
      int r = e - n;
      qa = 0;
      while (r >= n - 1 - qa) { r -= n - 1 - qa; ++qa; }
      qb = qa + 1 + r;
    }
    double turns = 0.0;
    for (int g0 = from; g0 < to; g0 += kTabThreads) {
      load_phase_gates(s, gates + g0, params, min(to - g0, kTabThreads));
      for (int g = max(st.gate0, g0); g < min(st.gate0 + st.ngates, g0 + kTabThreads); ++g) {
        const double th = s.turns[g - g0];
        const int c = (int)(s.ct[g - g0] >> 8), t = (int)(s.ct[g - g0] & 255u);
        if (qb < 0) {
          if (c == qa) turns -= 0.5 * th;
        } else if ((c == qa && t == qb) || (c == qb && t == qa)) {
          turns += th;
        }
      }
    }
    const double frac = turns - floor(turns);                 // [0, 1)
    if (i0 + (int)threadIdx.x < count) coef[st.coef_off + e] = (uint32_t)(unsigned long long)(frac * 4294967296.0);
  }
}

// Block blk of a circuit's tables (kTabThreads threads; all of them call this).  What bounds it is the chain
// of one wave's instructions, about 8 cycles each (a second pass over warm caches takes as long as the first).
// So everything that comes from the plan is fetched unconditionally and before anything is formed, the
// parameters beside it, choices are selected and not branched to, and gates, entries and the layer's rotations
// are different waves' (4 qubits, 2 layers: 5.3 -> 4.2 us; the bare gate matrices take 2.9).
// Every block forms the gates from its layer on, whose flips it needs: work grows with gates x layers, and
// from kFlipLayers layers on once more with every kFlipLayers (3 qubits, 600 layers of one rotation each: 81 us
// in front of a kernel of 937; 12 qubits, 700 layers of one gate: 507 us in front of 4165).
__device__ inline void sweep_tables(const SweepPlan& A, const float* __restrict__ params, const SweepTabs& T, int blk,
                                    int fp32) {
  __shared__ uint32_t flips[kFlipLayers];
  __shared__ double2 s_c[kMaxQubits], s_a[kMaxQubits];   // by the qubit's index bit, as the three below
  __shared__ double s_cos[kMaxQubits], s_t[kMaxQubits];
  __shared__ int s_flip[kMaxQubits];
  __shared__ double2 s_trig[kTabThreads];
  __shared__ float s_par[kTabThreads];
  __shared__ uint32_t s_x, s_xo;
  __shared__ PhaseChunk s_phase;
  const int tid = threadIdx.x;
  const QPlanDev* gplan = A.plan;
  CP<QPlanDev> plan = to_const(gplan);
  CP<char> pb = reinterpret_cast<CP<char>>(plan);
  const QFused* fused = reinterpret_cast<const QFused*>(reinterpret_cast<const char*>(gplan) + A.off_fused);
  CP<QSweep> sweeps = reinterpret_cast<CP<QSweep>>(pb + A.off_sweeps);
  const int n = A.n, F = A.n_fused, S = A.n_sweeps, L0 = A.sweep_first;
  const int cs = n > 8 ? n - 8 : 0;   // 2^cs blocks of kTabThreads entries per layer
  if (blk == 0) {
    for (int f = tid; f <= F; f += kTabThreads) gate_entry(gplan, params, f, fp32, T.gtab);
    return;
  }
  const int l = L0 + ((blk - 1) >> cs), chunk = (blk - 1) & ((1 << cs) - 1);   // l = S: behind the last layer
  if (l > S) {
    phase_entries(gplan, params, s_phase, reinterpret_cast<uint32_t*>(T.gtab + (size_t)(F + 1) * kGT));
    return;
  }
  // a thread per rotation takes its sine, then one per gate multiplies them up
  constexpr int kGates = kTabThreads / 3;
  const int rc = tid % 3, ti = tid - (kTabThreads - 64);
  // Everything is fetched unconditionally, from the plan's header where there is nothing (a circuit without
  // parameters has no gate and may have no parameter array): a condition would be a branch around each fetch,
  // or a wait for the one it depends on.
  const QFused* fsrc = F > 0 ? fused : reinterpret_cast<const QFused*>(gplan);
  const int fr0 = tid / 3 < F ? tid / 3 : 0;
  QFused fu = fsrc[tid < F ? tid : 0];
  int nc = fsrc[fr0].ncomp, pi = fsrc[fr0].param[rc];
  constexpr int kAhead = 4;
  const uint32_t* grows = S > 0 ? reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(gplan) + A.off_sweeps +
                                                                    offsetof(QSweep, arow))
                                : reinterpret_cast<const uint32_t*>(gplan);
  auto row_of = [&](int k) {   // (lanes 16.. repeat the rows; a layer out of range gives some row)
    k = k < S ? k : S - 1;
    return grows[(size_t)(k > 0 ? k : 0) * (sizeof(QSweep) / 4) + (tid & 15)];
  };
  uint32_t ahead[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) ahead[i] = row_of(S - 1 - i);
  const uint32_t row_l = row_of(l);
  CP<QSweep> L = sweeps + (l < S ? l : 0);
  const bool rot = ti >= 0 && ti < kPos && l < S;
  const int32_t* gl = reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(gplan) +
                                                       (rot ? A.off_sweeps + l * (int)sizeof(QSweep) : 0));
  const int gate_at = gl[rot ? ti : 0], bit_at = gl[rot ? offsetof(QSweep, tin) / 4 + ti : 0];
  // the parameters, fetched beside the plan that says which is whose, if there are no more than threads
  const bool few = A.n_params <= kTabThreads;
  const float par = (A.n_params > 0 ? params : reinterpret_cast<const float*>(gplan))[tid < A.n_params ? tid : 0];
  CP<int32_t> tin = reinterpret_cast<CP<int32_t>>(pb + (l < S ? A.off_sweeps + l * (int)sizeof(QSweep) + (int)offsetof(QSweep, tin)
                                                              : (int)offsetof(QPlanDev, ftpos)));
  int tb[kMaxQubits];   // index bit of each position of the mapping (0 behind the last)
#pragma unroll
  for (int k = 0; k < kMaxQubits; ++k) tb[k] = tin[k];
  int nterms = 0, phase = -1;
  uint32_t arow[kMaxQubits] = {};
  if (l < S) {
    nterms = L->nterms;
    phase = L->phase;
#pragma unroll
    for (int b = 0; b < kMaxQubits; ++b) arow[b] = L->arow[b];
  }
  // this thread's index in the layer's mapping, without the X mask, and where it was before the index map
  // (linear, so the mask's share is added later)
  // Up to 6 qubits the entries are one wave's, the third: the first has the gates and the masks.
  const bool apart = n <= 6;
  const int i = chunk * kTabThreads + (apart ? tid ^ 128 : tid);
  const uint32_t v = sweep_thread((uint32_t)i >> 3, n), r = (uint32_t)i & 7u;
  uint32_t ji = 0, joi = 0;
  if (i < (1 << n)) {
#pragma unroll
    for (int k = 0; k < kMaxQubits; ++k) ji ^= ((k < 3 ? r >> k : v >> (k - 3)) & 1u) << tb[k];
#pragma unroll
    for (int b = 0; b < kMaxQubits; ++b) joi |= ((uint32_t)__popc(arow[b] & ji) & 1u) << b;
  }
  asm volatile("" : "+v"(ji), "+v"(joi));   // (formed here: the mapping and the rows need not be kept)
  s_par[tid] = par;
  if (tid < kMaxQubits) {
    s_c[tid] = s_a[tid] = make_double2(1.0, 0.0);
    s_t[tid] = 0.0; s_cos[tid] = 1.0; s_flip[tid] = 0;
  }
  // Flips from layer l on, kFlipLayers layers at a time from the last one back; layer l's gates, and those
  // before it.
  auto first_gate = [&](int k) {
    int f = k < 0 ? 0 : F;
    if (k >= 0)
#pragma unroll
      for (int p = 0; p < kPos; ++p) {
        const int g = sweeps[k].gate[p];
        if (g >= 0 && g < f) f = g;
      }
    return f;
  };
  __syncthreads();
  float th = 0.f;
  if (F > 0) {
    const int at = rc < nc ? pi : 0;
    th = s_par[few ? at : 0];
    if (!few) th = params[at];
  }
  uint32_t x = 0;      // the X mask, carried back from the readout through the index maps (first wave)
  auto pass = [&](int hi, auto first) {
    constexpr bool FIRST = decltype(first)::value;   // (its gates and rows are fetched already)
    const int lo = hi - kFlipLayers > l ? hi - kFlipLayers : l;
    for (int k = lo + tid; k < hi; k += kTabThreads) flips[k - lo] = 0;
    if (F == 0) __syncthreads();
    int fa = 0, fb = F;   // the gates come layer by layer: from layer l - 1 on, and those of layers [lo, hi)
    if (F > kGates) {
      fa = first_gate(lo > l ? lo : l - 1) / kGates * kGates;
      if (hi < S) fb = first_gate(hi);
    }
    for (int f0 = fa; f0 < fb; f0 += kGates) {
      const int f = f0 + tid, fr = f0 + tid / 3;
      if (f0 || !FIRST) {
        fu = fused[f < F ? f : 0];
        nc = fused[fr < F ? fr : 0].ncomp, pi = fused[fr < F ? fr : 0].param[rc];
        th = params[rc < nc ? pi : 0];
      }
      if (tid < 3 * kGates && fr < F) {
        double sn, cn;
        if (fp32) {
          float sf, cf;
          sincosf(0.5f * th, &sf, &cf);
          sn = sf; cn = cf;
        } else {
          half_angle(th, &sn, &cn);
        }
        s_trig[tid] = make_double2(cn, sn);
      }
      __syncthreads();
      if (tid < kGates && f < F && !fu.head && fu.layer >= l - 1) {
        double2 u0 = make_double2(1.0, 0.0), u1 = make_double2(0.0, 0.0);   // first column: all the split needs
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double2 t = s_trig[3 * tid + k];
          if (k < fu.ncomp) column_rot(fu.kind[k], t.x, t.y, u0, u1);
        }
        const int b = n - 1 - fu.qubit, flip = zyz_flip(u0, u1);
        if (fu.layer >= lo && fu.layer < hi && flip) atomicOr(&flips[fu.layer - lo], 1u << b);
        if (fu.layer <= l) {
          const Zyz z = zyz_split(u0, u1);
          if (fu.layer == l) { s_c[b] = z.c; s_cos[b] = z.cosb; s_t[b] = z.t; }
          else { s_a[b] = z.a; s_flip[b] = flip; }
        }
      }
      __syncthreads();
    }
    if (tid < 64) {   // (ballots of row parities; rows and flips four layers at a time, for they are cold)
      auto steps = [&](int k0, const uint32_t (&rows)[kAhead]) {
        uint32_t fl[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) fl[i] = flips[k0 - i >= lo ? k0 - i - lo : 0];
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
          if (k0 - i >= lo) {
            x ^= __builtin_amdgcn_readfirstlane(fl[i]);
            if (k0 - i > l) x = (uint32_t)__ballot((int)(__popc(x & rows[i]) & 1u)) & 0xffffu;
          }
      };
      if constexpr (FIRST) steps(S - 1, ahead);
#pragma unroll 1
      for (int k0 = FIRST ? S - 1 - kAhead : hi - 1; k0 >= lo; k0 -= kAhead) {
        uint32_t rows[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) rows[i] = row_of(k0 - i);
        steps(k0, rows);
      }
    }
    return lo;
  };
  for (int hi = pass(S, std::true_type{}); hi > l;) {
    __syncthreads();   // the flips are read
    hi = pass(hi, std::false_type{});
  }
  if (tid < 64) {
    const uint32_t xo = l < S ? (uint32_t)__ballot((int)(__popc(x & row_l) & 1u)) & 0xffffu : x;   // before the index map
    if (tid == 0) {
      s_x = x;
      s_xo = xo;
      if (l == L0) T.xmask[S] = xo;   // the product state's (behind the opening layer, or in front of the first)
    }
  }
  double mag = 1.0;
#pragma unroll
  for (int b = 0; b < kMaxQubits; ++b) mag *= s_cos[b];
  __syncthreads();
  x = s_x;
  if (l == L0 && chunk == 0 && L0 > 0) {   // the opening layer: nothing is pulled back
    if (tid < kTC) T.tcoef[tid] = 0.f;
    if (tid == 0) { T.xmask[0] = s_xo; T.lscale[0] = 1.0; }
    for (int f = tid; f < F; f += kTabThreads) {
      if (F > kGates) fu = fused[f];   // (else each thread still has its gate)
      if (!fu.head) continue;
      double* g = T.gpar + (size_t)f * kGP;
      g[0] = 1.0; g[1] = 0.0; g[2] = 1.0;
      g[3] = ((s_xo >> (n - 1 - fu.qubit)) & 1u) ? -1.0 : 1.0;
    }
  }
  if (chunk == 0 && l < S && ti >= 0 && ti < kTC) {
    if (ti == 0) { T.xmask[l] = x; T.lscale[l] = mag * mag; }
    float t = 0.f;
    const int my_gate = rot ? gate_at : -1;
    if (my_gate >= 0) {
      // S_x, S_y: the cosines of the gates pulled back when they are taken (wave positions first,
      // then the swap slots, then the rest); S_z: of all
      double s7 = 1.0, s9 = 1.0;
#pragma unroll 1
      for (int p = 7; p < n; ++p) {
        const double c2 = s_cos[tin[p]] * s_cos[tin[p]];
        s7 *= c2;
        if (p >= 9) s9 *= c2;
      }
      const double sc = ti >= 9 ? s9 : (ti >= 7 ? s7 : mag * mag);
      const int b = bit_at;
      const bool neg = (x >> b) & 1u;   // X RY(b) X = RY(-b)
      t = (float)(neg ? -s_t[b] : s_t[b]);
      double* gp = T.gpar + (size_t)my_gate * kGP;
      gp[0] = s_c[b].x; gp[1] = s_c[b].y;
      gp[2] = sc;
      gp[3] = neg ? -mag * mag : mag * mag;
    }
    T.tcoef[(size_t)l * kTC + ti] = t;
  }
  const uint32_t j = ji ^ x, jo = l < S ? joi ^ s_xo : j;   // basis index of this entry, and before the index map
  double turn = 0.0;   // of the layer's CRZ gates, in units of pi
  if (l < S && phase >= 0) {
    CP<QPhaseStage> st = reinterpret_cast<CP<QPhaseStage>>(pb + plan->off_phase) + phase;
    const QPhaseGate* pg = reinterpret_cast<const QPhaseGate*>(reinterpret_cast<const char*>(gplan) + plan->off_phase_gates) + st->gate0;
    for (int g0 = 0, ng = st->ngates; g0 < ng; g0 += kTabThreads) {
      const int count = min(ng - g0, kTabThreads);
      load_phase_gates(s_phase, pg + g0, params, count);
      for (int g = 0; g < count; ++g) {
        const uint32_t ct = s_phase.ct[g];
        const double th = s_phase.turns[g];
        if ((j >> (n - 1 - (int)(ct >> 8))) & 1u) turn += ((j >> (n - 1 - (int)(ct & 255u))) & 1u) ? th : -th;
      }
    }
  }
  if (i >= (1 << n)) return;
  // two products, so that their chains overlap
  double2 ph = make_double2(mag, 0.0), pa = make_double2(1.0, 0.0);
  int half = 0;     // half turns
  const double2 one = make_double2(1.0, 0.0);
  for (int b0 = 0; b0 < n; b0 += 4) {
    double2 c[4], a[4];
    int fl[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) { c[b] = s_c[b0 + b]; a[b] = s_a[b0 + b]; fl[b] = s_flip[b0 + b]; }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const bool cb = (j >> (b0 + b)) & 1u, ab = (jo >> (b0 + b)) & 1u;
      ph = cmul(ph, cb ? c[b] : one);
      pa = cmul(pa, ab ? a[b] : one);
      half += ab ? 0 : fl[b];   // RY(pi) = diag(-1, 1) X
    }
  }
  ph = cmul(ph, pa);
  if (l < S) {
    CP<uint32_t> terms = reinterpret_cast<CP<uint32_t>>(pb + plan->off_terms) + 2 * L->term0;
    for (int t = 0; t < nterms; ++t) half += __popc(terms[2 * t] & j) & __popc(terms[2 * t + 1] & j) & 1;
    if (phase >= 0) {
      double2 e;
      sincospi(turn, &e.y, &e.x);
      ph = cmul(ph, e);
    }
  }
  if (half & 1) ph = make_double2(-ph.x, -ph.y);
  T.ptab[((size_t)(l - L0) << n) + i] = make_float2((float)ph.x, (float)ph.y);
}

}  // namespace qp

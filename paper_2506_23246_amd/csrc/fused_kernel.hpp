// Templates of the fused register/LDS kernel (included by the per-qubit-count units).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "const_dev.hpp"
#include "qp_internal.hpp"
#include "fused.hpp"

namespace qp {

__device__ __forceinline__ uint32_t parity(uint32_t x) { return __popc(x) & 1u; }

__device__ __forceinline__ uint32_t swz(uint32_t idx) { return lds_swizzle(idx); }

// Logical index bits of a thread in mapping tpos (v: the thread's index bits, see sweep_thread).
template <int N, typename TP>
__device__ __forceinline__ uint32_t deposit_thread(uint32_t v, TP tpos) {
  uint32_t j = 0;
#pragma unroll
  for (int k = 3; k < N; ++k) j |= ((v >> (k - 3)) & 1u) << tpos[k];
  return j;
}

__device__ __forceinline__ uint32_t reg_off(int r, uint32_t p0, uint32_t p1, uint32_t p2) {
  return ((uint32_t)(r & 1) << p0) | ((uint32_t)((r >> 1) & 1) << p1) |
         ((uint32_t)((r >> 2) & 1) << p2);
}

// Keeps the scheduler from interleaving what stands on its two sides: every side has independent work
// enough, and interleaved the live ranges exceed the 256 registers.
__device__ __forceinline__ void sched_cut() { __builtin_amdgcn_sched_barrier(0); }

template <typename V>
__device__ __forceinline__ void pin_sgpr(V& v) { asm volatile("" : "+s"(v)); }
template <typename V>
__device__ __forceinline__ void pin_vgpr(V& v) { asm volatile("" : "+v"(v)); }

// DPP permutation that brings the partner lane of thread bit K (lane XOR 1, 2, 7 or 8), as an operand
// modifier of the multiply-adds below.  They are written out because the compiler keeps the
// permutation as a move of its own (half the rate, and a register for every moved value: the Maxwell
// kernels spilled 700 and 1400 registers).  A VALU result may be read through DPP, or by a permlane
// swap, two wait states after it was written; the compiler does not see into the blocks, so each one
// starts (and, where it writes what a swap may read, ends) with that wait.  What a block writes is marked
// early-clobber: it is written before the last input is read, and an input that the compiler knows to hold
// the same value would else be given the same register.
#define QP_DPP_0 " quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
#define QP_DPP_1 " quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n"
#define QP_DPP_2 " row_half_mirror row_mask:0xf bank_mask:0xf\n"
#define QP_DPP_3 " row_ror:8 row_mask:0xf bank_mask:0xf\n"

// ---- one sweep layer's rotations ------------------------------------------------------------------
// RY(b) / cos(b/2): x0' = x0 - t x1, x1' = x1 + t x0 (t = tan(b/2), |t| <= 1).  One multiply-add per
// real number, against four for a general 2x2 gate; what bounds the kernels is VALU issue (see
// fused_tile), so the gates are kept in this form and everything diagonal goes into the tables.
// The coefficients sit in vector registers: a multiply-add with a scalar operand or a DPP permutation
// issues every 4 cycles, one with three vector operands every 2 to 3 (measured, 8 and 2 waves per
// SIMD).
template <int B, int S>
__device__ __forceinline__ void rot_reg(float (&sr)[8][8], float (&si)[8][8], float t) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (r & (1 << B)) continue;
    const int r1 = r | (1 << B);
    const float a = sr[S][r], b = sr[S][r1], c = si[S][r], d = si[S][r1];
    sr[S][r] = fmaf(-t, b, a); sr[S][r1] = fmaf(t, a, b);
    si[S][r] = fmaf(-t, d, c); si[S][r1] = fmaf(t, c, d);
  }
}
// The same on thread bit K; ts: +t in lanes whose bit is set, -t in the others.
#define QP_ROT_LANE(D)                                                                                        \
  asm("s_nop 1\n"                                                                                             \
      "v_fmac_f32_dpp %0, %0, %16" D "v_fmac_f32_dpp %1, %1, %16" D "v_fmac_f32_dpp %2, %2, %16" D             \
      "v_fmac_f32_dpp %3, %3, %16" D "v_fmac_f32_dpp %4, %4, %16" D "v_fmac_f32_dpp %5, %5, %16" D             \
      "v_fmac_f32_dpp %6, %6, %16" D "v_fmac_f32_dpp %7, %7, %16" D "v_fmac_f32_dpp %8, %8, %16" D             \
      "v_fmac_f32_dpp %9, %9, %16" D "v_fmac_f32_dpp %10, %10, %16" D "v_fmac_f32_dpp %11, %11, %16" D         \
      "v_fmac_f32_dpp %12, %12, %16" D "v_fmac_f32_dpp %13, %13, %16" D "v_fmac_f32_dpp %14, %14, %16" D       \
      "v_fmac_f32_dpp %15, %15, %16" D "s_nop 1"                                                              \
      : "+&v"(sr[S][0]), "+&v"(sr[S][1]), "+&v"(sr[S][2]), "+&v"(sr[S][3]), "+&v"(sr[S][4]), "+&v"(sr[S][5]), \
        "+&v"(sr[S][6]), "+&v"(sr[S][7]), "+&v"(si[S][0]), "+&v"(si[S][1]), "+&v"(si[S][2]), "+&v"(si[S][3]), \
        "+&v"(si[S][4]), "+&v"(si[S][5]), "+&v"(si[S][6]), "+&v"(si[S][7]) \
      : "v"(ts))
template <int K, int S>
__device__ __forceinline__ void rot_lane(float (&sr)[8][8], float (&si)[8][8], float ts) {
  if constexpr (K == 0) QP_ROT_LANE(QP_DPP_0);
  else if constexpr (K == 1) QP_ROT_LANE(QP_DPP_1);
  else if constexpr (K == 2) QP_ROT_LANE(QP_DPP_2);
  else QP_ROT_LANE(QP_DPP_3);
}

// Statistics of a statevector pair (x: lambda-family 4 + C, y: psi-family C):
//   S_x = sum Im(conj(x) y'), S_y = sum +-Re(conj(x) y') (+ where the bit is set), y' the amplitude with
// the gate's bit flipped.  Register bit B:
template <int B, int C, int X = 4 + C>
__device__ __forceinline__ void stat_reg(const float (&sr)[8][8], const float (&si)[8][8], float& sx, float& sy) {
  float a[2] = {0.f, 0.f}, b[2] = {0.f, 0.f};   // two partial sums: shorter dependent chains
  int np = 0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (r & (1 << B)) continue;
    const int r1 = r | (1 << B), h = np++ & 1;
    const float x0r = sr[X][r], x0i = si[X][r], x1r = sr[X][r1], x1i = si[X][r1];
    const float y0r = sr[C][r], y0i = si[C][r], y1r = sr[C][r1], y1i = si[C][r1];
    a[h] = fmaf(x0r, y1i, a[h]); a[h] = fmaf(-x0i, y1r, a[h]);
    a[h] = fmaf(x1r, y0i, a[h]); a[h] = fmaf(-x1i, y0r, a[h]);
    b[h] = fmaf(x1r, y0r, b[h]); b[h] = fmaf(x1i, y0i, b[h]);
    b[h] = fmaf(-x0r, y1r, b[h]); b[h] = fmaf(-x0i, y1i, b[h]);
  }
  sx += a[0] + a[1];
  sy += b[0] + b[1];
}
// Thread bit K (S_y without its lane sign, which the flush applies): a += Im(conj(x) y'),
// b += Re(conj(x) y') over registers R .. R + 3.
#define QP_STAT_LANE(D)                                                                                       \
  asm("s_nop 1\n"                                                                                             \
      "v_fmac_f32_dpp %0, %8, %12" D "v_fmac_f32_dpp %1, %4, %12" D                                            \
      "v_fmac_f32_dpp %2, %9, %13" D "v_fmac_f32_dpp %3, %5, %13" D                                            \
      "v_fmac_f32_dpp %0, -%4, %16" D "v_fmac_f32_dpp %1, %8, %16" D                                           \
      "v_fmac_f32_dpp %2, -%5, %17" D "v_fmac_f32_dpp %3, %9, %17" D                                           \
      "v_fmac_f32_dpp %0, %10, %14" D "v_fmac_f32_dpp %1, %6, %14" D                                           \
      "v_fmac_f32_dpp %2, %11, %15" D "v_fmac_f32_dpp %3, %7, %15" D                                           \
      "v_fmac_f32_dpp %0, -%6, %18" D "v_fmac_f32_dpp %1, %10, %18" D                                          \
      "v_fmac_f32_dpp %2, -%7, %19" D "v_fmac_f32_dpp %3, %11, %19" D                                          \
      : "+&v"(a0), "+&v"(b0), "+&v"(a1), "+&v"(b1) \
      : "v"(sr[C][R]), "v"(sr[C][R + 1]), "v"(sr[C][R + 2]), "v"(sr[C][R + 3]), "v"(si[C][R]),                 \
        "v"(si[C][R + 1]), "v"(si[C][R + 2]), "v"(si[C][R + 3]), "v"(sr[X][R]), "v"(sr[X][R + 1]),     \
        "v"(sr[X][R + 2]), "v"(sr[X][R + 3]), "v"(si[X][R]), "v"(si[X][R + 1]),                \
        "v"(si[X][R + 2]), "v"(si[X][R + 3]))
template <int K, int C, int X, int R>
__device__ __forceinline__ void stat_lane4(const float (&sr)[8][8], const float (&si)[8][8], float& a0, float& b0,
                                           float& a1, float& b1) {
  if constexpr (K == 0) QP_STAT_LANE(QP_DPP_0);
  else if constexpr (K == 1) QP_STAT_LANE(QP_DPP_1);
  else if constexpr (K == 2) QP_STAT_LANE(QP_DPP_2);
  else QP_STAT_LANE(QP_DPP_3);
}
template <int K, int C, int X = 4 + C>
__device__ __forceinline__ void stat_lane(const float (&sr)[8][8], const float (&si)[8][8], float& sx, float& sy) {
  float a0 = 0.f, b0 = 0.f, a1 = 0.f, b1 = 0.f;   // two partial sums: shorter dependent chains
  stat_lane4<K, C, X, 0>(sr, si, a0, b0, a1, b1);
  stat_lane4<K, C, X, 4>(sr, si, a0, b0, a1, b1);
  sx += a0 + a1;
  sy += b0 + b1;
}
// w_r += Im(conj(x_r) y_r): its signed sums are the S_z of every qubit and the moments of CRZ phases.
template <int C, int X = 4 + C>
__device__ __forceinline__ void stat_diag(const float (&sr)[8][8], const float (&si)[8][8], float (&w)[8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    w[r] = fmaf(sr[X][r], si[C][r], w[r]);
    w[r] = fmaf(-si[X][r], sr[C][r], w[r]);
  }
}

// Statevector S times the layer's table entries (CONJ: their conjugates).
template <int S, bool CONJ>
__device__ __forceinline__ void mul_phase(float (&sr)[8][8], float (&si)[8][8], const float (&pc)[8], const float (&ps)[8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const float c = pc[r], sn = CONJ ? -ps[r] : ps[r];
    const float a = sr[S][r], b = si[S][r];
    sr[S][r] = a * c - b * sn;
    si[S][r] = a * sn + b * c;
  }
}

template <int CTRL>
__device__ __forceinline__ float dppf(float v) {   // DPP lane permutation (row-local)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Reduce-scatter of four per-lane values over the wave: permlane32_swap pairs lanes l and l+32
// (entries split 2/2), permlane16_swap pairs rows 0/1 and 2/3 (1/1), then DPP row_ror:8,
// quad_perm xor 1, xor 2 and row_half_mirror sum the sixteen lanes of each row.  Lanes of row e
// end with entry e.  No LDS traffic.
__device__ __forceinline__ float wave_reduce_scatter4(const float* v) {
  float a[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(v[i]), __float_as_int(v[2 + i]), false, false);
    a[i] = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  }
  const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_int(a[0]), __float_as_int(a[1]), false, false);
  float c = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  c += dppf<0x128>(c);   // row_ror:8  (lane l <- l ^ 8 within a row)
  c += dppf<0xB1>(c);    // quad_perm [1,0,3,2]: xor 1
  c += dppf<0x4E>(c);    // quad_perm [2,3,0,1]: xor 2
  c += dppf<0x141>(c);   // row_half_mirror: lane l <- 7 - l within eight lanes
  return c;
}

// ---- register exchange through LDS ----------------------------------------------------------
// An exchange moves the statevectors from one layer's output mapping to the next layer's input
// mapping through the entanglers' index map A: logical index j of a point lives at LDS entry
// swz(pbase ^ M j), M an invertible GF(2) map chosen per exchange for conflict-free banks.  pbase is
// a multiple of 2^N and every index is below 2^N, so pbase + x equals pbase ^ x; M and the swizzle
// are linear over GF(2), so a register's entry is the thread's base XOR a uniform offset (woff for the
// writer, roff for the reader, which carries A).  Up to 9 qubits a point lives in one wave, whose LDS
// operations complete in order, so the exchange needs no barrier and one plane serves every
// statevector in turn.
template <int N>
__device__ __forceinline__ void point_fence() {   // before lanes of the point read what others wrote
  if (N >= 10) __syncthreads();
  else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

struct Addr {
  uint32_t w[8], r[8];   // byte offsets of the eight registers, writer and reader
};
__device__ __forceinline__ Addr xchg_addr(CP<uint32_t> wo, CP<uint32_t> ro, uint32_t wb, uint32_t rb) {
  Addr A;
#pragma unroll
  for (int r = 0; r < 8; ++r) { A.w[r] = wb ^ wo[r]; A.r[r] = rb ^ ro[r]; }
  return A;
}
template <int T, int S, int PL>
__device__ __forceinline__ void xwrite(const float (&sr)[8][8], const float (&si)[8][8], float2* __restrict__ buf,
                                       const uint32_t (&a)[8]) {
  char* b = reinterpret_cast<char*>(buf);
#pragma unroll
  for (int r = 0; r < 8; ++r)
    *reinterpret_cast<float2*>(b + a[r] + PL * (T * 64)) = make_float2(sr[S][r], si[S][r]);
}
template <int T, int S, int PL>
__device__ __forceinline__ void xread(float (&sr)[8][8], float (&si)[8][8], const float2* __restrict__ buf,
                                      const uint32_t (&a)[8]) {
  const char* b = reinterpret_cast<const char*>(buf);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const float2 v = *reinterpret_cast<const float2*>(b + a[r] + PL * (T * 64));
    sr[S][r] = v.x; si[S][r] = v.y;
  }
}
// In-wave exchange (up to 9 qubits) of statevectors [S, S + NV).
template <int T, int S, int NV>
__device__ __forceinline__ void exchange_wave(float (&sr)[8][8], float (&si)[8][8], float2* __restrict__ buf, const Addr& A) {
  if constexpr (NV > 0) {
    xwrite<T, S, 0>(sr, si, buf, A.w);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    xread<T, S, 0>(sr, si, buf, A.r);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    exchange_wave<T, S + 1, NV - 1>(sr, si, buf, A);
  }
}

// Wave exchange (10 qubits and more): register bits 0 .. NB-1 trade places with the wave bits of the
// point.  A plane holds [wave][register][lane]; wave w writes register r (low bits rl, high bits rh) as
// register (rh, w) of wave rl and reads its own eight back, so the addresses are two bases and
// constants.
template <int N, int T, int S, int PL>
__device__ __forceinline__ void wwrite(const float (&sr)[8][8], const float (&si)[8][8], float2* __restrict__ buf, uint32_t wbase) {
  constexpr int NB = sweep_wave(N);
  char* b = reinterpret_cast<char*>(buf) + wbase;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int rl = r & ((1 << NB) - 1), rh = r >> NB;
    *reinterpret_cast<float2*>(b + PL * (T * 64) + rl * 4096 + (rh << NB) * 512) = make_float2(sr[S][r], si[S][r]);
  }
}
template <int N, int T, int S, int PL>
__device__ __forceinline__ void wread(float (&sr)[8][8], float (&si)[8][8], const float2* __restrict__ buf, uint32_t rbase) {
  const char* b = reinterpret_cast<const char*>(buf) + rbase;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const float2 v = *reinterpret_cast<const float2*>(b + PL * (T * 64) + r * 512);
    sr[S][r] = v.x; si[S][r] = v.y;
  }
}

// Swap slot I of statevector S: register bit I trades places with lane bit 4 + I.  For each register
// pair (r, r | 2^I) a cross-lane swap exchanges odd rows of the first with even rows of the second
// (lane bit 4, permlane16_swap) or the upper half of the first with the lower half of the second
// (lane bit 5, permlane32_swap); the value at (register bit q', lane bit h') afterwards is the one
// that was at (q = h', h = q').  An involution.
template <int I, int S>
__device__ __forceinline__ void swap_slot(float (&sr)[8][8], float (&si)[8][8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (r & (1 << I)) continue;
    const int r1 = r | (1 << I);
    if (I == 0) {
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(sr[S][r]), __float_as_int(sr[S][r1]), false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(__float_as_int(si[S][r]), __float_as_int(si[S][r1]), false, false);
      sr[S][r] = __int_as_float(a[0]); sr[S][r1] = __int_as_float(a[1]);
      si[S][r] = __int_as_float(b[0]); si[S][r1] = __int_as_float(b[1]);
    } else {
      const auto a = __builtin_amdgcn_permlane32_swap(__float_as_int(sr[S][r]), __float_as_int(sr[S][r1]), false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(si[S][r]), __float_as_int(si[S][r1]), false, false);
      sr[S][r] = __int_as_float(a[0]); sr[S][r1] = __int_as_float(a[1]);
      si[S][r] = __int_as_float(b[0]); si[S][r1] = __int_as_float(b[1]);
    }
  }
}

// Adds v to a per-wave statistic slot in LDS with an LDS float add that returns nothing, so the
// wave does not wait for its outstanding LDS operations as a read-modify-write would.  Each slot
// belongs to one wave and receives one lane's value per flush, in program order, so the sums are
// those of the read-modify-write, bit for bit.
__device__ __forceinline__ void slot_add(float* p, float v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---- one layer's data -------------------------------------------------------------------------------
template <int N>
struct Coef {
  float t[N];   // tan(b/2) by position, lane positions with the lane's sign
};
template <int N, int P0 = 0, int P1 = N>   // positions [P0, P1)
__device__ __forceinline__ Coef<N> load_coef(CP<float> tc, uint32_t v, bool inverse) {
  Coef<N> K;
#pragma unroll
  for (int p = P0; p < P1; ++p) {
    float t = tc[p];
    if (inverse) t = -t;
    if (p >= 3 && p < 7) t = ((v >> (p - 3)) & 1u) ? t : -t;
    pin_vgpr(t);
    K.t[p] = t;
  }
  return K;
}
struct Phase {
  float c[8], s[8];
};
__device__ __forceinline__ Phase load_phase(const float4* __restrict__ tab) {   // the thread's eight entries
  Phase P;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 v = tab[i];
    P.c[2 * i] = v.x; P.s[2 * i] = v.y; P.c[2 * i + 1] = v.z; P.s[2 * i + 1] = v.w;
  }
  return P;
}

// Rotations of statevector S: the positions reached in place, then the swap slots.  has: the layer's flags (in
// the kernels of circuits that are not thin all positions, known to the compiler).
template <int N, int S>
__device__ __forceinline__ void rot_base(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K, int has) {
  rot_reg<0, S>(sr, si, K.t[0]);
  rot_reg<1, S>(sr, si, K.t[1]);
  rot_reg<2, S>(sr, si, K.t[2]);
  if (N > 3 && (has & kSweepLane0)) {
    if constexpr (N > 3) rot_lane<0, S>(sr, si, K.t[3]);
  }
  if (N > 4 && (has & kSweepLanes)) {
    if constexpr (N > 4) rot_lane<1, S>(sr, si, K.t[4]);
    if constexpr (N > 5) rot_lane<2, S>(sr, si, K.t[5]);
    if constexpr (N > 6) rot_lane<3, S>(sr, si, K.t[6]);
  }
}
template <int N, int S>
__device__ __forceinline__ void swap_all(float (&sr)[8][8], float (&si)[8][8]) {
  if constexpr (N > 7) swap_slot<0, S>(sr, si);
  if constexpr (N > 8) swap_slot<1, S>(sr, si);
}
template <int N, int S>
__device__ __forceinline__ void rot_slots(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K) {
  if constexpr (N > 7) rot_reg<0, S>(sr, si, K.t[7]);
  if constexpr (N > 8) rot_reg<1, S>(sr, si, K.t[8]);
}
template <int N, int S>
__device__ __forceinline__ void rot_wave(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K) {
  if constexpr (N > 9) rot_reg<0, S>(sr, si, K.t[9]);
  if constexpr (N > 10) rot_reg<1, S>(sr, si, K.t[10]);
  if constexpr (N > 11) rot_reg<2, S>(sr, si, K.t[11]);
}
// Forward: phase and rotations in place, then the swap slots (the state ends in the layer's mapping
// before the wave exchange).
template <int N, int S>
__device__ __forceinline__ void layer_fwd(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K, const Phase& P, int has) {
  mul_phase<S, false>(sr, si, P.c, P.s);
  rot_base<N, S>(sr, si, K, has);
  if (N > 7 && (has & kSweepSlots)) {
    swap_all<N, S>(sr, si);
    rot_slots<N, S>(sr, si, K);
  }
  sched_cut();
}

// Statistics of a layer by position: S_x, S_y, and the diagonal products.
template <int N>
struct Stats {
  float x[N], y[N], w[8];
};
template <int N, int P0 = 0, int P1 = N>
__device__ __forceinline__ void clear(Stats<N>& Q) {
#pragma unroll
  for (int p = P0; p < P1; ++p) Q.x[p] = Q.y[p] = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) Q.w[r] = 0.f;
}
// Marks the statistics as computed here: else the compiler sinks their multiply-adds into the flush,
// past the gates that overwrite the statevectors, and spills what they need.
template <int N, int P0, int P1>
__device__ __forceinline__ void pin_stats(Stats<N>& Q, bool w) {
#pragma unroll
  for (int p = P0; p < P1; ++p) { pin_vgpr(Q.x[p]); pin_vgpr(Q.y[p]); }
  if (w)
#pragma unroll
    for (int r = 0; r < 8; ++r) pin_vgpr(Q.w[r]);
}
// Adjoint of the wave positions on the pair (C, 4 + C): pull back, then the statistics.
template <int N, int C>
__device__ __forceinline__ void wave_rot(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K) {
  rot_wave<N, C>(sr, si, K); rot_wave<N, 4 + C>(sr, si, K);
}
template <int N, int C>
__device__ __forceinline__ void wave_stat(const float (&sr)[8][8], const float (&si)[8][8], Stats<N>& Q) {
  if constexpr (N > 9) stat_reg<0, C>(sr, si, Q.x[9], Q.y[9]);
  if constexpr (N > 10) stat_reg<1, C>(sr, si, Q.x[10], Q.y[10]);
  if constexpr (N > 11) stat_reg<2, C>(sr, si, Q.x[11], Q.y[11]);
  pin_stats<N, 9, N>(Q, false);
  sched_cut();
}
// Adjoint of the rest of a layer on the pair (unless PULL, of a layer folded into the encoding, whose
// statistics alone are taken): swap slots with their statistics, rotations in place; then the
// statistics of these, and the conjugate phase.  Gates of one layer act on different qubits and
// commute, so each statistic may be taken with any of the others pulled back or not; only the cosines
// left out so far scale it, which the gradient kernel puts back (gpar).
template <int N, int C, bool PULL>
__device__ __forceinline__ void adj_rot(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K, Stats<N>& Q, int has) {
  if (N > 7 && (has & kSweepSlots)) {
    if (PULL) { rot_slots<N, C>(sr, si, K); rot_slots<N, 4 + C>(sr, si, K); }
    if constexpr (N > 7) stat_reg<0, C>(sr, si, Q.x[7], Q.y[7]);
    if constexpr (N > 8) stat_reg<1, C>(sr, si, Q.x[8], Q.y[8]);
    if constexpr (N > 7) pin_stats<N, 7, N < 9 ? N : 9>(Q, false);
    swap_all<N, C>(sr, si); swap_all<N, 4 + C>(sr, si);
  }
  sched_cut();
  if (PULL) { rot_base<N, C>(sr, si, K, has); rot_base<N, 4 + C>(sr, si, K, has); }
  sched_cut();
}
template <int N, int C, bool PULL>
__device__ __forceinline__ void adj_stat(float (&sr)[8][8], float (&si)[8][8], const Phase& P, Stats<N>& Q, int has) {
  stat_reg<0, C>(sr, si, Q.x[0], Q.y[0]);
  stat_reg<1, C>(sr, si, Q.x[1], Q.y[1]);
  stat_reg<2, C>(sr, si, Q.x[2], Q.y[2]);
  sched_cut();
  if (N > 3 && (has & kSweepLane0)) {
    if constexpr (N > 3) stat_lane<0, C>(sr, si, Q.x[3], Q.y[3]);
  }
  if (N > 4 && (has & kSweepLanes)) {
    if constexpr (N > 4) stat_lane<1, C>(sr, si, Q.x[4], Q.y[4]);
    if constexpr (N > 5) stat_lane<2, C>(sr, si, Q.x[5], Q.y[5]);
    if constexpr (N > 6) stat_lane<3, C>(sr, si, Q.x[6], Q.y[6]);
  }
  stat_diag<C>(sr, si, Q.w);
  pin_stats<N, 0, N < 7 ? N : 7>(Q, true);
  sched_cut();
  if (PULL) { mul_phase<C, true>(sr, si, P.c, P.s); mul_phase<4 + C, true>(sr, si, P.c, P.s); }
  sched_cut();
}
template <int N, int C, bool PULL>
__device__ __forceinline__ void layer_adj(float (&sr)[8][8], float (&si)[8][8], const Coef<N>& K, const Phase& P, Stats<N>& Q,
                                          int has) {
  adj_rot<N, C, PULL>(sr, si, K, Q, has);
  adj_stat<N, C, PULL>(sr, si, P, Q, has);
}

// Adds the S_x and S_y of positions [P0, P1) to the wave's slots (two gates per reduction).
template <int N, int P0, int P1, bool THIN>
__device__ __forceinline__ void flush_xy(CP<QSweep> L, const Stats<N>& Q, uint32_t v, float* __restrict__ slots, int F,
                                         int wave, int lane) {
#pragma unroll
  for (int p = P0; p < P1; p += 2) {
    const int q = p + 1 < P1 ? p + 1 : p;
    if (THIN && L->gate[p] < 0 && L->gate[q] < 0) continue;
    auto ys = [&](int k) { return k >= 3 && k < 7 && !((v >> (k - 3)) & 1u) ? -Q.y[k] : Q.y[k]; };
    const float v4[4] = {Q.x[p], ys(p), Q.x[q], ys(q)};
    const float s = wave_reduce_scatter4(v4);
    const int g = lane < 32 ? L->gate[p] : (q > p ? L->gate[q] : -1);
    if (g >= 0 && (lane & 15) == 0) slot_add(slots + (wave * F + g) * kGS + ((lane >> 4) & 1), s);
  }
}
// Signed sums of w over the wave: S_z of every position, and with a CRZ phase in front of the layer
// (mslots) the first- and second-order parity sums W_q, W_qq' its gradient needs.
template <int N>
__device__ __forceinline__ void flush_z(CP<QSweep> L, const float (&w)[8], uint32_t v, float* __restrict__ slots,
                                        float* __restrict__ mom, int F, int wave, int lane) {
  float W[8];   // Walsh transform over the register bits: W[s] = sum_r (-1)^(s.r) w_r
#pragma unroll
  for (int r = 0; r < 8; ++r) W[r] = w[r];
#pragma unroll
  for (int b = 1; b < 8; b <<= 1)
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (!(r & b)) { const float x = W[r], y = W[r | b]; W[r] = x + y; W[r | b] = x - y; }
  auto flip = [&](float x, int p) { return ((v >> (p - 3)) & 1u) ? -x : x; };   // times (-1)^bit of thread position p
  float z[N];
#pragma unroll
  for (int p = 0; p < N; ++p) z[p] = p < 3 ? W[1 << p] : flip(W[0], p);
#pragma unroll
  for (int p = 0; p < N; p += 4) {
    float v4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v4[i] = p + i < N ? z[p + i < N ? p + i : 0] : 0.f;
    const float s = wave_reduce_scatter4(v4);
    const int row = lane >> 4;
    int g = -1, t = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (p + i < N && row == i) { g = L->gate[p + i < N ? p + i : 0]; t = L->tin[p + i < N ? p + i : 0]; }
    if ((lane & 15) == 0 && p + row < N) {
      if (g >= 0) slot_add(slots + (wave * F + g) * kGS + 2, s);
      if (mom) slot_add(mom + (N - 1 - t), s);
    }
  }
  if (mom) {
#pragma unroll
    for (int p = 0; p < N; ++p) {
#pragma unroll
      for (int q0 = p + 1; q0 < N; q0 += 4) {
        float v4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = q0 + i;
          float x = 0.f;
          if (q < N) {
            if (q < 3) x = W[(1 << p) | (1 << (q < 3 ? q : 0))];
            else x = flip(p < 3 ? W[1 << (p < 3 ? p : 0)] : flip(W[0], p), q);
          }
          v4[i] = x;
        }
        const float s = wave_reduce_scatter4(v4);
        const int row = lane >> 4;
        int t = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (q0 + i < N && row == i) t = L->tin[q0 + i < N ? q0 + i : 0];
        const int a = N - 1 - L->tin[p], b = N - 1 - t;
        if ((lane & 15) == 0 && q0 + row < N)
          slot_add(mom + N + phase_pair_index(N, a < b ? a : b, a < b ? b : a), s);
      }
    }
  }
}

// ---- forward by rounds ------------------------------------------------------------------------------
// The kernels that return a loss (and the fields the total loss is formed from) run the forward on the
// fused 2x2 gates as they are, in rounds of three register-bit gates and up to two swap slots (QRound),
// with the roundings and the summation order in which their FP64 losses have always been formed; only
// the adjoint, and calls that return no loss, run the sweep layers.
//
// Single-qubit gate on register bit B for statevectors [S0, S0 + NS).
// u: u00r,u00i,u01r,u01i,u10r,u10i,u11r,u11i.  Each lane applies the gate to its own amplitude
// pairs on the matrix cores: v_mfma_f32_4x4x1f32 treats the wave as 16 blocks of 4 lanes,
// C[m][n] += A[m] B[n] with A[m] from lane 4b + m, B[n] from lane 4b + n and C[m][n] in register m
// of lane 4b + n.  With lane 4b + m holding row m of the gate's real 4x4 form M (acting on
// (re x, im x, re y, im y)) as A, and every lane its own pair component k as B, four such steps
// (k = 0..3) leave M (x, y) of each lane's pair in its four C registers.  The 2x2 products thus
// leave the vector ALU (no gain in rate: the two share the FP32 pipe; one instruction does the work of
// four).  Called in wave-uniform control flow only: a lane's result depends on the A operands of the other three
// lanes of its block, so all 64 lanes must be active.
template <int B, int S0, int NS>
__device__ __forceinline__ void apply_gate(float (&sr)[8][8], float (&si)[8][8], const float* u) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const uint32_t q = threadIdx.x & 3u;   // row m of M held by this lane
  const bool lo = q < 2, odd = q & 1u;
  // M rows: (u00r, -u00i, u01r, -u01i), (u00i, u00r, u01i, u01r), (u10r, -u10i, u11r, -u11i),
  // (u10i, u10r, u11i, u11r); column k of row q.  (u points at pinned coefficients: selects
  // between the elements of a plain local array would become a per-lane indexed scratch load.)
  const float e0 = lo ? u[0] : u[4], e1 = lo ? u[1] : u[5], e2 = lo ? u[2] : u[6], e3 = lo ? u[3] : u[7];
  const float k0 = odd ? e1 : e0;
  const float k1 = odd ? e0 : -e1;
  const float k2 = odd ? e3 : e2;
  const float k3 = odd ? e2 : -e3;
#pragma unroll
  for (int s = S0; s < S0 + NS; ++s) {
    // the four pairs' chains interleaved step by step (independent MFMAs between dependent ones)
    f32x4 c[4];
    int rr[4], r1s[4];
    int np = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (r & (1 << B)) continue;
      rr[np] = r; r1s[np] = r | (1 << B); ++np;
    }
    // Raised wave priority while this wave issues its matrix-core chains: the SIMD's other wave
    // (statistics, exchanges) fills the issue slots between them instead of delaying the next
    // link of a chain (12-qubit step 322 -> 298 ms).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(k0, sr[s][rr[i]], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(k1, si[s][rr[i]], c[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(k2, sr[s][r1s[i]], c[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(k3, si[s][r1s[i]], c[i], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sr[s][rr[i]] = c[i][0]; si[s][rr[i]] = c[i][1]; sr[s][r1s[i]] = c[i][2]; si[s][r1s[i]] = c[i][3];
    }
  }
}

// Marks statevector S as computed at this point of the instruction stream: keeps the compiler
// from sinking a group's gate arithmetic past the following barrier, which would undo the
// overlap of that group's arithmetic with another group's LDS traffic.
template <int S>
__device__ __forceinline__ void pin_sv(float (&sr)[8][8], float (&si)[8][8]) {
#pragma unroll
  for (int r = 0; r < 8; ++r) asm volatile("" : "+v"(sr[S][r]), "+v"(si[S][r]));
}

struct RoundCoef {
  float c[40];   // gate b's 2x2 matrix at c[8b .. 8b+7]; b = 3, 4: swap slots
};

template <int NS>
__device__ __forceinline__ RoundCoef load_round(CP<QRound> rk, CP<float> gtab, int F) {
  RoundCoef R;
#pragma unroll
  for (int b = 0; b < 3 + NS; ++b) {
    const int g = b < 3 ? rk->gate[b] : rk->sgate[b - 3];
    const int gi = g >= 0 ? g : F;
#pragma unroll
    for (int e = 0; e < 8; ++e) R.c[8 * b + e] = gtab[gi * kGT + e];
  }
#pragma unroll
  for (int i = 0; i < 8 * (3 + NS); ++i) pin_sgpr(R.c[i]);
  return R;
}

struct Offs {
  uint32_t o[8];
};

__device__ __forceinline__ Offs load_offs(CP<uint32_t> p) {
  Offs O;
#pragma unroll
  for (int r = 0; r < 8; ++r) { O.o[r] = p[r]; pin_sgpr(O.o[r]); }
  return O;
}

// Per exchange a lane needs three words: its writer and reader byte bases and the sign bits of
// its eight reads (the planner tabulates them per thread of a point: QLane); each access then
// costs one XOR.
struct XLane {
  uint32_t wb, rb, sgn;
};

// The lane words of exchange k for thread u of the point whose swizzled base is pb8 = 8 swz(pbase): one 16-byte vector load from the plan's lane table
// (vector loads use their own wait counter, so a load issued early does not hold up LDS waits).
__device__ __forceinline__ XLane lane_words(const QLane* __restrict__ lanes, int k, int TPn, uint32_t u,
                                            uint32_t pb8) {
  const QLane L = lanes[(size_t)k * TPn + u];
  XLane x;
  x.wb = L.wb ^ pb8;
  x.rb = L.rb ^ pb8;
  x.sgn = L.sgn;
  return x;
}

// Writes statevectors SV0 and SV1 to LDS planes PL and PL + 1 in the writer mapping wr.
template <int T, int SV0, int SV1, int PL>
__device__ __forceinline__ void rwrite(const float (&sr)[8][8], const float (&si)[8][8], float2* __restrict__ buf,
                                       const Offs& wo, uint32_t wb) {
  constexpr uint32_t PLANE = T * 8 * 8;   // bytes; a power of two above every in-plane offset
  char* b = reinterpret_cast<char*>(buf);
  const uint32_t base = wb | (PL * PLANE);   // plane PL folded into the base: one XOR per access
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t o = base ^ wo.o[r];
    *reinterpret_cast<float2*>(b + o) = make_float2(sr[SV0][r], si[SV0][r]);
    *reinterpret_cast<float2*>(b + PLANE + o) = make_float2(sr[SV1][r], si[SV1][r]);
  }
}

// Reads statevectors SV0 and SV1 back from planes PL, PL + 1 through the descriptor X.
template <int T, int SV0, int SV1, int PL>
__device__ __forceinline__ void rread(float (&sr)[8][8], float (&si)[8][8], const float2* __restrict__ buf,
                                      const Offs& ro, bool signs, uint32_t rb, uint32_t sgn) {
  // SV0 is read completely before SV1, so the gates on SV0 can start while SV1 is in flight.
  constexpr uint32_t PLANE = T * 8 * 8;   // bytes; a power of two above every in-plane offset
  const char* b = reinterpret_cast<const char*>(buf);
  const uint32_t base = rb | (PL * PLANE);   // plane PL folded into the base: one XOR per access
  // raised wave priority while issuing the reads (as for the matrix-core chains): after a
  // barrier the wave's reads go out ahead of the other wave's arithmetic (12-qubit step 298 ->
  // 284 ms)
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t o = base ^ ro.o[r];
      const float2 v = *reinterpret_cast<const float2*>(b + h * PLANE + o);
      if (h == 0) { sr[SV0][r] = v.x; si[SV0][r] = v.y; } else { sr[SV1][r] = v.x; si[SV1][r] = v.y; }
    }
  __builtin_amdgcn_s_setprio(0);
  if (signs) {   // a CZ stage: negate the amplitudes whose sign bit is set (uniform branch)
    // The empty volatile asm keeps this a branch: merged into the unconditional path, the flips
    // would cost two XORs per amplitude on every exchange and consume the loaded values at once,
    // which forces the LDS reads to complete before any independent work can cover them.
    asm volatile("");
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t flip = ((sgn >> r) & 1u) << 31;   // negate by flipping the sign bits
      sr[SV0][r] = __uint_as_float(__float_as_uint(sr[SV0][r]) ^ flip);
      si[SV0][r] = __uint_as_float(__float_as_uint(si[SV0][r]) ^ flip);
      sr[SV1][r] = __uint_as_float(__float_as_uint(sr[SV1][r]) ^ flip);
      si[SV1][r] = __uint_as_float(__float_as_uint(si[SV1][r]) ^ flip);
    }
  }
}

// The exchange of the four statevectors, pair by pair through planes 0 and 1 (up to 9 qubits inside a
// wave; from 10 where the LDS holds only two planes per workgroup).
template <int N, int T>
__device__ __forceinline__ void rexchange(float (&sr)[8][8], float (&si)[8][8], float2* __restrict__ buf,
                                          CP<QXchg> X, const XLane& x) {
  const Offs wo = load_offs(X->woff), ro = load_offs(X->roff);
  const bool sg = X->nterms != 0;
  rwrite<T, 0, 1, 0>(sr, si, buf, wo, x.wb);
  point_fence<N>();
  rread<T, 0, 1, 0>(sr, si, buf, ro, sg, x.rb, x.sgn);
  point_fence<N>();
  rwrite<T, 2, 3, 0>(sr, si, buf, wo, x.wb);
  point_fence<N>();
  rread<T, 2, 3, 0>(sr, si, buf, ro, sg, x.rb, x.sgn);
  point_fence<N>();
}

// Forward gates of a round on statevectors S0, S0 + 1 (an absent gate is the identity entry):
// gates01 applies the gates on register bits 0 and 1, gate2 the gate on bit 2 (gates on
// different qubits commute, so the split point is free).
template <int S0>
__device__ __forceinline__ void gates01(float (&sr)[8][8], float (&si)[8][8], const RoundCoef& R) {
  apply_gate<0, S0, 1>(sr, si, R.c); apply_gate<1, S0, 1>(sr, si, R.c + 8);
  apply_gate<0, S0 + 1, 1>(sr, si, R.c); apply_gate<1, S0 + 1, 1>(sr, si, R.c + 8);
}
template <int S0>
__device__ __forceinline__ void gate2(float (&sr)[8][8], float (&si)[8][8], const RoundCoef& R) {
  apply_gate<2, S0, 1>(sr, si, R.c + 16); apply_gate<2, S0 + 1, 1>(sr, si, R.c + 16);
}
// The rest of a round after the bit-0/1 gates: the bit-2 gate, then the swap slots with their gates
// (the statevectors end in the round's output mapping).
template <int S0, int NS>
__device__ __forceinline__ void finish(float (&sr)[8][8], float (&si)[8][8], const RoundCoef& R) {
  gate2<S0>(sr, si, R);
  if (NS > 0) {
    swap_slot<0, S0>(sr, si); swap_slot<0, S0 + 1>(sr, si);
    apply_gate<0, S0, 1>(sr, si, R.c + 24); apply_gate<0, S0 + 1, 1>(sr, si, R.c + 24);
  }
  if (NS > 1) {
    swap_slot<1, S0>(sr, si); swap_slot<1, S0 + 1>(sr, si);
    apply_gate<1, S0, 1>(sr, si, R.c + 32); apply_gate<1, S0 + 1, 1>(sr, si, R.c + 32);
  }
}
template <int S0, int NS>
__device__ __forceinline__ void round_fwd(float (&sr)[8][8], float (&si)[8][8], const RoundCoef& R) {
  gates01<S0>(sr, si, R);
  finish<S0, NS>(sr, si, R);
}

// Phase stages (CRZ runs).
// In a round's input mapping, slot k (register bit k < 3, thread bit k - 3 otherwise) holds the
// index bit of qubit N - 1 - tpos[k].  phi(j) = sum_q alpha_q b_q + sum_(q<q') beta_qq' b_q b_q' is
// split into the thread's part and per-register terms; all sums are unsigned 32-bit fractions of a
// turn, so they are exact modulo 2 pi, and only the final angle of each amplitude is rounded.
template <int N>
__device__ __forceinline__ uint32_t phase_beta(CP<uint32_t> coef, int a, int b) {
  return a < b ? coef[N + phase_pair_index(N, a, b)] : coef[N + phase_pair_index(N, b, a)];
}

template <int N>
__device__ __forceinline__ void phase_factors(CP<QRound> rk, CP<uint32_t> coef, uint32_t u, float (&pc)[8],
                                              float (&ps)[8]) {
  int qk[N];
#pragma unroll
  for (int k = 0; k < N; ++k) qk[k] = N - 1 - rk->tpos[k];
  uint32_t th = 0, g0 = coef[qk[0]], g1 = coef[qk[1]], g2 = coef[qk[2]];
#pragma unroll
  for (int k = 3; k < N; ++k) {
    const uint32_t bk = (u >> (k - 3)) & 1u;
    uint32_t t = coef[qk[k]];
#pragma unroll
    for (int k2 = k + 1; k2 < N; ++k2) t += ((u >> (k2 - 3)) & 1u) * phase_beta<N>(coef, qk[k], qk[k2]);
    th += bk * t;
    g0 += bk * phase_beta<N>(coef, qk[0], qk[k]);
    g1 += bk * phase_beta<N>(coef, qk[1], qk[k]);
    g2 += bk * phase_beta<N>(coef, qk[2], qk[k]);
  }
  const uint32_t d01 = phase_beta<N>(coef, qk[0], qk[1]);
  const uint32_t d02 = phase_beta<N>(coef, qk[0], qk[2]);
  const uint32_t d12 = phase_beta<N>(coef, qk[1], qk[2]);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    uint32_t ph = th;
    if (r & 1) ph += g0;
    if (r & 2) ph += g1;
    if (r & 4) ph += g2;
    if ((r & 3) == 3) ph += d01;
    if ((r & 5) == 5) ph += d02;
    if ((r & 6) == 6) ph += d12;
    // angle = 2 pi ph / 2^32 = pi x with x = (signed) ph / 2^31 in [-1, 1)
    sincospif((float)(int32_t)ph * 4.656612873077392578125e-10f, &ps[r], &pc[r]);
  }
}

template <int I>
struct IntC {
  static constexpr int value = I;
};

// ---- angle encoding of one qubit ------------------------------------------------------------
// Embedded single-qubit state e(b) (b = 0, 1) and its angle derivative d(b) for qubit q, with the
// Jacobian d theta_q / d(t, x, y).  RY: e = (cos, sin), RX: e = (cos, -i sin), of theta/2.  When the
// circuit opens with a rotation stage, the qubit's gate U of that stage is applied here (e <- U e,
// d <- U d): the stage acts on the product state, so the state after it is still a product.  (The
// rounds fold the stage's rounds but the circuit's last, the sweeps always the whole stage.)
struct QEnc {
  float e0r, e0i, e1r, e1i, d0r, d0i, d1r, d1i, j[3];
};

template <int N>
__device__ __forceinline__ QEnc encode_qubit(CP<QPlanDev> plan, CP<float> gtab, const FusedArgs& a, long long pt,
                                             bool valid, const float* p3, int q, uint32_t x, bool rounds) {
  float c, s, j0 = 0.f, j1 = 0.f, j2 = 0.f;
  if (plan->enc_kind == QP_ENC_CYCLE) {
    const int cc = plan->coord_of_qubit[q];
    const float x = cc == 0 ? p3[0] : (cc == 1 ? p3[1] : p3[2]);
    float jv;
    const int sc = plan->enc_scale;
    if (sc == QP_SCALE_PI) {           // theta/2 = pi x/2
      sincospif(0.5f * x, &s, &c);
      jv = 3.14159265358979323846f;
    } else if (sc == QP_SCALE_BIAS) {  // theta/2 = pi (x+1)/4
      sincospif(0.25f * (x + 1.f), &s, &c);
      jv = 1.57079632679489661923f;
    } else if (sc == QP_SCALE_NONE) {
      sincosf(0.5f * x, &s, &c);
      jv = 1.f;
    } else {
      const float xx = fminf(fmaxf(x, -1.f), 1.f);
      const float th = (sc == QP_SCALE_ASIN) ? asinf(xx) + 1.57079632679489661923f : acosf(xx);
      sincosf(0.5f * th, &s, &c);
      const float rs = 1.f / sqrtf(fmaxf(1.f - xx * xx, 0.f));
      jv = (sc == QP_SCALE_ASIN) ? rs : -rs;
    }
    j0 = cc == 0 ? jv : 0.f;
    j1 = cc == 1 ? jv : 0.f;
    j2 = cc == 2 ? jv : 0.f;
  } else {   // angles given per point (QP_ENC_ANGLES, or random Fourier features formed beforehand)
    float th = 0.f;
    if (valid) {
      th = a.angles[pt * N + q];
      j0 = a.jac[(pt * N + q) * 3 + 0];
      j1 = a.jac[(pt * N + q) * 3 + 1];
      j2 = a.jac[(pt * N + q) * 3 + 2];
    }
    sincosf(0.5f * th, &s, &c);
  }
  QEnc E;
  E.e0r = c; E.e0i = 0.f;
  E.d0r = -0.5f * s; E.d0i = 0.f;
  if (plan->enc_gate == QP_ENC_RY) {
    E.e1r = s; E.e1i = 0.f; E.d1r = 0.5f * c; E.d1i = 0.f;
  } else {   // RX|0> = (cos, -i sin)
    E.e1r = 0.f; E.e1i = -s; E.d1r = 0.f; E.d1i = -0.5f * c;
  }
  const int hg = rounds ? plan->head_gate[q] : plan->hgate[q];
  if (hg >= 0) {
    CP<float> g = gtab + hg * kGT;   // U: u00r, u00i, u01r, u01i, u10r, u10i, u11r, u11i
    const float xr = E.e0r, xi = E.e0i, yr = E.e1r, yi = E.e1i;
    E.e0r = g[0] * xr - g[1] * xi + g[2] * yr - g[3] * yi;
    E.e0i = g[0] * xi + g[1] * xr + g[2] * yi + g[3] * yr;
    E.e1r = g[4] * xr - g[5] * xi + g[6] * yr - g[7] * yi;
    E.e1i = g[4] * xi + g[5] * xr + g[6] * yi + g[7] * yr;
    const float ar = E.d0r, ai = E.d0i, br = E.d1r, bi = E.d1i;
    E.d0r = g[0] * ar - g[1] * ai + g[2] * br - g[3] * bi;
    E.d0i = g[0] * ai + g[1] * ar + g[2] * bi + g[3] * br;
    E.d1r = g[4] * ar - g[5] * ai + g[6] * br - g[7] * bi;
    E.d1i = g[4] * ai + g[5] * ar + g[6] * bi + g[7] * br;
  }
  E.j[0] = j0; E.j[1] = j1; E.j[2] = j2;
  if (!rounds && ((x >> (N - 1 - q)) & 1u)) {   // the sweeps' X mask in front of the first layer
    const QEnc D = E;
    E.e0r = D.e1r; E.e0i = D.e1i; E.e1r = D.e0r; E.e1i = D.e0i;
    E.d0r = D.d1r; E.d0i = D.d1i; E.d1r = D.d0r; E.d1i = D.d0i;
  }
  return E;
}

// The embedded qubits of a point, spread over the lanes of its wave that hold the point: lane u forms
// the qubits at positions u, u + LP, .. of the mapping emap (packed: of the four slots' points in turn),
// and every lane takes each from the lane that has it.  Else every lane would evaluate the sines of
// every qubit, and the kernel would hold a copy of that code per qubit, which a small call fetches once
// from a cold instruction cache (simulate, 4 qubits, 64 points: 15.1 -> 14.0 us; forward and backward,
// 7 qubits, 64000 points: 833 -> 788 us; outputs only, 10 qubits, 20000 points: 240 -> 175 us).
template <int N, int M>
struct Encodings {
  static constexpr int LP = N < 9 ? 1 << (N - 3) : 64;   // a point's lanes in a wave
  static constexpr int IT = (M + LP - 1) / LP;
  QEnc E[IT];

  __device__ __forceinline__ void form(CP<QPlanDev> plan, CP<float> gtab, const FusedArgs& a, long long pt, CP<int32_t> emap,
                                       uint32_t x, bool rounds) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      int k = (int)(threadIdx.x % LP) + i * LP;
      if (M % LP != 0 && k >= M) k = M - 1;
      const long long p = M > N ? pt + k / N : pt;
      const bool valid = p < a.P;
      float p3[3] = {0.f, 0.f, 0.f};
      if (valid && a.points && plan->enc_kind != QP_ENC_ANGLES) {
        p3[0] = a.points[p * 3 + 0];
        p3[1] = a.points[p * 3 + 1];
        p3[2] = a.points[p * 3 + 2];
      }
      E[i] = encode_qubit<N>(plan, gtab, a, p, valid, p3, N - 1 - emap[M > N ? k % N : k], x, rounds);
    }
  }
  template <int K>
  static __device__ __forceinline__ float lane(float v) {
    const int b = __float_as_int(v);
    if constexpr (LP == 1) return v;
    else if constexpr (LP == 64) return __int_as_float(__builtin_amdgcn_readlane(b, K));
    else return __int_as_float(__builtin_amdgcn_ds_swizzle(b, (K << 5) | (32 - LP)));   // lane (l & -LP) | K
  }
  template <int I>
  __device__ __forceinline__ QEnc get() const {
    constexpr int K = I % LP;
    const QEnc& e = E[I / LP];
    QEnc o;
    o.e0r = lane<K>(e.e0r); o.e0i = lane<K>(e.e0i); o.e1r = lane<K>(e.e1r); o.e1i = lane<K>(e.e1i);
    if (M == N) {
      o.d0r = lane<K>(e.d0r); o.d0i = lane<K>(e.d0i); o.d1r = lane<K>(e.d1r); o.d1i = lane<K>(e.d1i);
#pragma unroll
      for (int c = 0; c < 3; ++c) o.j[c] = lane<K>(e.j[c]);
    }
    return o;
  }
};

// Calls f(IntC<I0>), .., f(IntC<I1 - 1>).
template <int I0, int I1, typename Fn>
__device__ __forceinline__ void static_for(const Fn& f) {
  if constexpr (I0 < I1) {
    f(IntC<I0>{});
    static_for<I0 + 1, I1>(f);
  }
}

// ---- gradients with respect to the per-point angles and their Jacobian ------------------------
// The embedding rotation of qubit q has generator G_q (Y for RY, X for RX): d psi_0/d theta_q =
// -(i/2) G_q psi_0, and the tangents are dpsi_c,0 = sum_q J_qc (-(i/2) G_q) psi_0, so (the G's of
// different qubits commute) d dpsi_c,0/d theta_q = -(i/2) G_q dpsi_c,0.  With lambda, mu_c the
// adjoints pulled back to the embedded state,
//   dL/d theta_q = Im <lambda|G_q|psi> + sum_c Im <mu_c|G_q|dpsi_c>,   dL/d J_qc = Im <mu_c|G_q|psi>,
// the same Pauli statistics the adjoint takes for every gate, but per point.  When the circuit's
// opening rotation stage is folded into the encoding, the sweep ends at that stage's output, and
// G_q is replaced by U_q G_q U_q^H (U_q the stage's gate on qubit q), which the statistics
// contract with as an axis (n_x, n_y, n_z).  At the end of the sweep the statevectors sit in mapping
// gtpos.
template <int N, int T>
__device__ __forceinline__ float enc_pair(float nx, float ny, float nz, float sb, float xr, float xi, float yor,
                                          float yoi, float2 yp) {
  const float im_p = xr * yp.y - xi * yp.x;    // Im(conj(x) y_partner)
  const float re_p = xr * yp.x + xi * yp.y;    // Re(conj(x) y_partner)
  const float im_o = xr * yoi - xi * yor;      // Im(conj(x) y_own)
  return nx * im_p + sb * (ny * re_p - nz * im_o);
}

// Axis (n_x, n_y, n_z) of U G U^H (U: the opening-stage gate on q, identity if none; G = X or Y).
__device__ __forceinline__ void enc_axis(CP<QPlanDev> plan, CP<float> gtab, int q, float& nx, float& ny, float& nz) {
  const bool rx = plan->enc_gate == QP_ENC_RX;
  float u8[8] = {1.f, 0.f, 0.f, 0.f, 0.f, 0.f, 1.f, 0.f};
  const int hg = plan->hgate[q];
  if (hg >= 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) u8[i] = gtab[hg * kGT + i];
  }
  // W = U G: X swaps U's columns; Y gives [[i u01, -i u00], [i u11, -i u10]]
  float w00r, w00i, w01r, w01i;
  if (rx) {
    w00r = u8[2]; w00i = u8[3]; w01r = u8[0]; w01i = u8[1];
  } else {
    w00r = -u8[3]; w00i = u8[2]; w01r = u8[1]; w01i = -u8[0];
  }
  // M = W U^H: M00 = W00 conj(u00) + W01 conj(u01), M01 = W00 conj(u10) + W01 conj(u11)
  const float m00r = w00r * u8[0] + w00i * u8[1] + w01r * u8[2] + w01i * u8[3];
  const float m01r = w00r * u8[4] + w00i * u8[5] + w01r * u8[6] + w01i * u8[7];
  const float m01i = w00i * u8[4] - w00r * u8[5] + w01i * u8[6] - w01r * u8[7];
  nx = m01r; ny = -m01i; nz = m00r;
}

// Sum over the point's lanes (up to 9 qubits), in all of them.
template <int N>
__device__ __forceinline__ float point_sum(float v) {
  if constexpr (N > 3) v += dppf<0xB1>(v);    // lane ^ 1
  if constexpr (N > 4) v += dppf<0x4E>(v);    // lane ^ 2
  if constexpr (N > 5) v += dppf<0x141>(v);   // the other four of eight lanes
  if constexpr (N > 6) v += dppf<0x128>(v);   // lane ^ 8
  if constexpr (N > 7) {
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
    v = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  }
  if constexpr (N > 8) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
    v = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  }
  return v;
}

// Up to 9 qubits a point's lanes are in one wave, and the sums are those of a layer's statistics, per
// point and contracted with the axis: G = 0 of all pairs (in Q already if the circuit opens with
// rotations, whose statistics are taken of the same statevectors), G = 1 .. 3 of psi with mu_(G-1).
// (Forward and backward at 7 qubits, 64000 points: 738 us with the staging below, 663 so.)
template <int N, int C, int X>
__device__ __forceinline__ void enc_stat(const float (&sr)[8][8], const float (&si)[8][8], Stats<N>& Q) {
  stat_reg<0, C, X>(sr, si, Q.x[0], Q.y[0]);
  stat_reg<1, C, X>(sr, si, Q.x[1], Q.y[1]);
  stat_reg<2, C, X>(sr, si, Q.x[2], Q.y[2]);
  if constexpr (N > 3) stat_lane<0, C, X>(sr, si, Q.x[3], Q.y[3]);
  if constexpr (N > 4) stat_lane<1, C, X>(sr, si, Q.x[4], Q.y[4]);
  if constexpr (N > 5) stat_lane<2, C, X>(sr, si, Q.x[5], Q.y[5]);
  if constexpr (N > 6) stat_lane<3, C, X>(sr, si, Q.x[6], Q.y[6]);
  stat_diag<C, X>(sr, si, Q.w);
}
template <int N, int C, int X>
__device__ __forceinline__ void enc_stat_slots(const float (&sr)[8][8], const float (&si)[8][8], Stats<N>& Q) {
  if constexpr (N > 7) stat_reg<0, C, X>(sr, si, Q.x[7], Q.y[7]);
  if constexpr (N > 8) stat_reg<1, C, X>(sr, si, Q.x[8], Q.y[8]);
}
template <int N, int P0, int P1>
__device__ __forceinline__ void enc_write(const Stats<N>& Q, CP<QPlanDev> plan, CP<float> gtab, uint32_t x, uint32_t v,
                                          float* __restrict__ out, int stride, bool first) {
  float w0 = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) w0 += Q.w[r];
#pragma unroll
  for (int p = P0; p < P1; ++p) {
    const int b = plan->gtpos[p], q = N - 1 - b;
    float nx, ny, nz;
    enc_axis(plan, gtab, q, nx, ny, nz);
    float y = Q.y[p], z = 0.f;
    if (p < 3) {
#pragma unroll
      for (int r = 0; r < 8; ++r) z += ((r >> (p < 3 ? p : 0)) & 1) ? -Q.w[r] : Q.w[r];
    } else {
      const bool set = (v >> (p - 3)) & 1u;
      z = set ? -w0 : w0;
      if (p < 7) y = set ? y : -y;
    }
    const float yz = ny * y + nz * z;
    const float s = point_sum<N>(nx * Q.x[p] + (((x >> b) & 1u) ? -yz : yz));
    if (first) out[(long long)q * stride] = s;
  }
}
template <int N>
__device__ __forceinline__ void encoding_grads_wave(float (&sr)[8][8], float (&si)[8][8], Stats<N>& Q, CP<QPlanDev> plan,
                                                    CP<float> gtab, const FusedArgs& a, long long pt, bool first, uint32_t v) {
  constexpr int NB = N < 7 ? N : 7;   // positions in place; the rest in the swap slots
  const uint32_t x = to_const(a.xmask)[plan->n_sweeps];
  float* da = a.d_angles + pt * N;
  float* dj = a.d_jac + pt * N * 3;
  const bool head = plan->sweep_first > 0;
  if (a.d_angles) {
    if (!head) {
      clear(Q);
      enc_stat<N, 0, 4>(sr, si, Q); enc_stat<N, 1, 5>(sr, si, Q); enc_stat<N, 2, 6>(sr, si, Q); enc_stat<N, 3, 7>(sr, si, Q);
    }
    enc_write<N, 0, NB>(Q, plan, gtab, x, v, da, 1, first);
    if (N > 7 && head) enc_write<N, NB, N>(Q, plan, gtab, x, v, da, 1, first);
  }
  float w[4][8];   // the diagonal products, kept for the swap slots
#pragma unroll
  for (int r = 0; r < 8; ++r) w[0][r] = Q.w[r];
  auto jac = [&](auto c) {
    constexpr int G = decltype(c)::value;
    clear(Q);
    enc_stat<N, 0, 4 + G>(sr, si, Q);
    enc_write<N, 0, NB>(Q, plan, gtab, x, v, dj + G - 1, 3, first);
#pragma unroll
    for (int r = 0; r < 8; ++r) w[G][r] = Q.w[r];
  };
  if (a.d_jac) { jac(IntC<1>{}); jac(IntC<2>{}); jac(IntC<3>{}); }
  if constexpr (N > 7) {
    static_for<0, 8>([&](auto c) { swap_all<N, decltype(c)::value>(sr, si); });
    auto slots = [&](auto c) {
      constexpr int G = decltype(c)::value;
      clear<N, 7, N>(Q);
      if constexpr (G == 0) {
        enc_stat_slots<N, 0, 4>(sr, si, Q); enc_stat_slots<N, 1, 5>(sr, si, Q);
        enc_stat_slots<N, 2, 6>(sr, si, Q); enc_stat_slots<N, 3, 7>(sr, si, Q);
      } else {
        enc_stat_slots<N, 0, 4 + G>(sr, si, Q);
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) Q.w[r] = w[G][r];
      enc_write<N, NB, N>(Q, plan, gtab, x, v, G == 0 ? da : dj + G - 1, G == 0 ? 1 : 3, first);
    };
    if (a.d_angles && !head) slots(IntC<0>{});
    if (a.d_jac) { slots(IntC<1>{}); slots(IntC<2>{}); slots(IntC<3>{}); }
  }
}

// From 10 qubits on the partner amplitude of a pair (index bit of qubit q flipped) is read back from the
// LDS planes, where the psi-family is staged two statevectors at a time.  One of two passes (PASS 0: partners of psi and dpsi_t; PASS 1: of dpsi_x and dpsi_y).  The
// qubits are taken one at a time (a loop, so no per-qubit register arrays), each qubit's sums are
// reduced over the point's threads at once, and the point's first thread writes them (PASS 0) or
// adds its share (PASS 1).
template <int N, int T, int PASS>
__device__ __forceinline__ void enc_grad_pass(const float (&sr)[8][8], const float (&si)[8][8],
                                              float2* __restrict__ buf, float* __restrict__ red, CP<QPlanDev> plan,
                                              CP<float> gtab, uint32_t jl, const FusedArgs& a,
                                              long long pt, bool valid, uint32_t u) {
  constexpr int PLANE = T * 8;
  constexpr int TP = 1 << (N - 3);
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  CP<int32_t> gt = plan->gtpos;
  const uint32_t l0 = gt[0], l1 = gt[1], l2 = gt[2];
  point_fence<N>();   // the planes are free (every wave of the point is past its last read of the sweep)
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const uint32_t e = tid * 8 + (r ^ (tid & 7));
    buf[e] = make_float2(sr[2 * PASS][r], si[2 * PASS][r]);
    buf[PLANE + e] = make_float2(sr[2 * PASS + 1][r], si[2 * PASS + 1][r]);
  }
  point_fence<N>();
#pragma unroll 1
  for (int q = 0; q < N; ++q) {
    const int pos = N - 1 - q;
    uint32_t rmask = 0, tmask = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (gt[k] == pos) {
        if (k < 3) rmask = 1u << k;
        else tmask = sweep_xor(k - 3);
      }
    }
    float nx, ny, nz;
    enc_axis(plan, gtab, q, nx, ny, nz);
    const uint32_t ptid = tid ^ tmask;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t j = jl ^ reg_off(r, l0, l1, l2);
      const float sb = ((j >> pos) & 1u) ? 1.f : -1.f;
      const uint32_t e = ptid * 8 + (((uint32_t)r ^ rmask) ^ (ptid & 7));
      const float2 y0 = buf[e];
      const float2 y1 = buf[PLANE + e];
      if (PASS == 0) {   // partners of psi and dpsi_t
        s0 += enc_pair<N, T>(nx, ny, nz, sb, sr[4][r], si[4][r], sr[0][r], si[0][r], y0);
        s0 += enc_pair<N, T>(nx, ny, nz, sb, sr[5][r], si[5][r], sr[1][r], si[1][r], y1);
        s1 += enc_pair<N, T>(nx, ny, nz, sb, sr[5][r], si[5][r], sr[0][r], si[0][r], y0);
        s2 += enc_pair<N, T>(nx, ny, nz, sb, sr[6][r], si[6][r], sr[0][r], si[0][r], y0);
        s3 += enc_pair<N, T>(nx, ny, nz, sb, sr[7][r], si[7][r], sr[0][r], si[0][r], y0);
      } else {           // partners of dpsi_x and dpsi_y
        s0 += enc_pair<N, T>(nx, ny, nz, sb, sr[6][r], si[6][r], sr[2][r], si[2][r], y0);
        s0 += enc_pair<N, T>(nx, ny, nz, sb, sr[7][r], si[7][r], sr[3][r], si[3][r], y1);
      }
    }
    // sum over the point's threads
#pragma unroll
    for (int off = 1; off < (TP < 64 ? TP : 64); off <<= 1) {
      s0 += __shfl_xor(s0, off);
      if (PASS == 0) {
        s1 += __shfl_xor(s1, off);
        s2 += __shfl_xor(s2, off);
        s3 += __shfl_xor(s3, off);
      }
    }
    if (TP > 64) {   // the point spans TP / 64 waves: combine them through the scratch slots
      constexpr int WPP = TP > 64 ? TP / 64 : 1;
      if (lane == 0) {
        red[wave * 40 + 0] = s0;
        red[wave * 40 + 1] = s1;
        red[wave * 40 + 2] = s2;
        red[wave * 40 + 3] = s3;
      }
      __syncthreads();
      const int w0 = (wave / WPP) * WPP;
      float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
      for (int w = 0; w < WPP; ++w) {
        t0 += red[(w0 + w) * 40 + 0];
        t1 += red[(w0 + w) * 40 + 1];
        t2 += red[(w0 + w) * 40 + 2];
        t3 += red[(w0 + w) * 40 + 3];
      }
      s0 = t0; s1 = t1; s2 = t2; s3 = t3;
      __syncthreads();
    }
    if (valid && u == 0) {
      if (PASS == 0) {
        if (a.d_angles) a.d_angles[pt * N + q] = s0;
        if (a.d_jac) {
          a.d_jac[(pt * N + q) * 3 + 0] = s1;
          a.d_jac[(pt * N + q) * 3 + 1] = s2;
          a.d_jac[(pt * N + q) * 3 + 2] = s3;
        }
      } else if (a.d_angles) {
        a.d_angles[pt * N + q] += s0;
      }
    }
  }
}

template <int N, int T>
__device__ __forceinline__ void encoding_grads(const float (&sr)[8][8], const float (&si)[8][8],
                                               float2* __restrict__ buf, float* __restrict__ red, CP<QPlanDev> plan,
                                               CP<float> gtab, const FusedArgs& a, long long pt,
                                               bool valid, uint32_t u) {
  const uint32_t jl = deposit_thread<N>(sweep_thread(u, N), plan->gtpos) ^ to_const(a.xmask)[plan->n_sweeps];
  enc_grad_pass<N, T, 0>(sr, si, buf, red, plan, gtab, jl, a, pt, valid, u);
  enc_grad_pass<N, T, 1>(sr, si, buf, red, plan, gtab, jl, a, pt, valid, u);
  point_fence<N>();   // the next tile's first exchange writes the planes
}

// Packed modes: the product state of point pt0 + SL in statevector slot SL (no input tangents; an
// out-of-range point gives the zero state).
template <int N, int SL>
__device__ __forceinline__ void packed_state(float (&sr)[8][8], float (&si)[8][8], const Encodings<N, 4 * N>& enc, bool vs,
                                             uint32_t v) {
  float Pr = vs ? 1.f : 0.f, Pi = 0.f;
  static_for<3, N>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    const QEnc E = enc.template get<SL * N + k>();
    const bool bit = (v >> (k - 3)) & 1u;
    const float er = bit ? E.e1r : E.e0r, ei = bit ? E.e1i : E.e0i;
    const float npr = Pr * er - Pi * ei, npi = Pr * ei + Pi * er;
    Pr = npr; Pi = npi;
  });
  const QEnc Q[3] = {enc.template get<SL * N>(), enc.template get<SL * N + 1>(), enc.template get<SL * N + 2>()};
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float pr = Pr, pi = Pi;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const bool b = (r >> i) & 1;
      const float er = b ? Q[i].e1r : Q[i].e0r, ei = b ? Q[i].e1i : Q[i].e0i;
      const float npr = pr * er - pi * ei, npi = pr * ei + pi * er;
      pr = npr; pi = npi;
    }
    sr[SL][r] = pr; si[SL][r] = pi;
  }
}

// ---- one tile of PPW points: forward, readout, seeds, adjoint --------------------------------
// buf: exchange planes (one up to 9 qubits, two with the forward by rounds; else EXS); slots: per-wave
// gate statistics [WAVES][F][kGS]; mslots: per-wave parity sums of CRZ layers; red: [WAVES][40].
//
// What bounds it: VALU issue.  Per amplitude and layer a statevector costs N multiply-adds per real
// number and one complex product, the statistics of a gate 4 multiply-adds per amplitude and
// statevector pair for each of S_x and S_y, and S_z of all gates together 2; LDS moves every
// statevector once per layer (twice from 10 qubits, where the wave bits are brought into registers
// through it).  Against 2x2 products both ways, an exchange per round of three to five gates and three
// sums per gate: 12 qubits x 8 layers, 262144 points, 284 -> 229 ms (layers in the adjoint alone; 194 ms
// both ways, not run: see the forward by rounds); forward and backward of 7 qubits x 4 layers, 64000
// points, layers both ways, 1424 -> 833 us.
template <int N, int T, int EXS, int MODE, bool EG = false, bool THIN = false>
__device__ __forceinline__ void fused_tile(const FusedArgs& a, int tile, float2* __restrict__ buf,
                                           float* __restrict__ slots, float* __restrict__ mslots,
                                           float* __restrict__ red, float& lacc) {
  constexpr int TP = 1 << (N - 3);         // threads per point
  constexpr int PPW = T / TP;              // points per workgroup tile (x4 in the packed modes)
  constexpr int DIM = 1 << N;
  constexpr bool PK = mode_packed(MODE);
  constexpr bool RND = mode_rounds(MODE);  // forward by rounds (see there), else by sweep layers
  static_assert(PPW >= 1, "tile too small");
  static_assert(!(PK && EG), "the packed modes carry no input gradients");
  CP<QPlanDev> plan = to_const(a.plan);
  CP<char> pb = reinterpret_cast<CP<char>>(plan);
  CP<QSweep> sweeps = reinterpret_cast<CP<QSweep>>(pb + plan->off_sweeps);
  const uint4* __restrict__ slanes =
      reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.plan) + plan->off_slanes);
  CP<float> gtab = to_const(a.gtab);
  CP<QRound> rounds = reinterpret_cast<CP<QRound>>(pb + plan->off_rounds);
  CP<float> tcoef = to_const(a.tcoef);
  const int L0 = plan->sweep_first, L1 = plan->n_sweeps;
  const int m = plan->n_out;
  const int F = a.n_fused;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int ps = tid / TP;
  const uint32_t u = (uint32_t)(tid % TP);
  const uint32_t v = sweep_thread(u, N);   // the thread's index bits
  const uint32_t pbase = (uint32_t)ps * DIM;
  const uint32_t pb8 = swz(pbase) * 8u;
  // wave exchange: bases of the thread's writes and reads (see wwrite)
  constexpr int WPP = TP > 64 ? TP / 64 : 1;
  const uint32_t wvb = (uint32_t)((wave / WPP) * WPP * 4096 + (wave % WPP) * 512 + lane * 8);
  const uint32_t rvb = (uint32_t)(wave * 4096 + lane * 8);
  const float4* __restrict__ ptab = reinterpret_cast<const float4*>(a.ptab) + u * 4;   // this thread's entries, per layer
  auto phase_of = [&](int l) { return load_phase(ptab + (size_t)(l - L0) * (DIM / 2)); };
  auto positions = [&](CP<QSweep> L) { return THIN ? L->flags : L->flags | kSweepAll; };
  auto lane_of = [&](int l) { return slanes[(size_t)l * TP + u]; };
  // loss weights: 1/P for the mean over all points, 1/N_vac and 1/N_diel for the split loss
  float w_all = 1.f, w_vac = 1.f, w_diel = 1.f;
  if ((MODE == kModeMaxwell || MODE == kModeTotal) && !a.loss_sum) {
    w_all = a.P > 0 ? 1.f / (float)a.P : 0.f;
    if (a.loss_kind == QP_LOSS_DIEL_SPLIT) {
      const int nv = a.counts[0], nd = a.counts[1];
      w_vac = nv > 0 ? 1.f / (float)nv : 0.f;
      w_diel = nd > 0 ? 1.f / (float)nd : 0.f;
    }
  }
  float sr[8][8], si[8][8];
  {
    // packed modes: slot s of the thread group holds point pt0 + s
    const long long pt = PK ? ((long long)tile * PPW + ps) * 4 : (long long)tile * PPW + ps;
    const long long pt0 = pt;
    const bool valid = pt < a.P;

    // ---------------- encoding and product state -------------------------------------------
    // An opening rotation stage is folded into the product state, which is formed in that layer's
    // output mapping.
    const int H = plan->n_head;
    CP<int32_t> emap = !RND ? plan->etpos : (H > 0 ? rounds[H - 1].tpost : rounds[0].tpos);
    const uint32_t ve = RND ? u : v, xe = to_const(a.xmask)[L1];   // thread bits of the mapping; X mask of the product state
    if constexpr (PK) {
      // four product states, one per slot (no tangents)
      Encodings<N, 4 * N> enc;
      enc.form(plan, gtab, a, pt0, emap, xe, RND);
      packed_state<N, 0>(sr, si, enc, pt0 + 0 < a.P, ve);
      packed_state<N, 1>(sr, si, enc, pt0 + 1 < a.P, ve);
      packed_state<N, 2>(sr, si, enc, pt0 + 2 < a.P, ve);
      packed_state<N, 3>(sr, si, enc, pt0 + 3 < a.P, ve);
    } else {
      Encodings<N, N> enc;
      enc.form(plan, gtab, a, pt, emap, xe, RND);
      // thread part: (P, D_c) by the product rule over the thread qubits
      float Pr = valid ? 1.f : 0.f, Pi = 0.f;
      float Dr[3] = {0.f, 0.f, 0.f}, Di[3] = {0.f, 0.f, 0.f};
      static_for<3, N>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        const QEnc E = enc.template get<k>();
        const bool bit = (ve >> (k - 3)) & 1u;
        const float er = bit ? E.e1r : E.e0r, ei = bit ? E.e1i : E.e0i;
        const float dr = bit ? E.d1r : E.d0r, di = bit ? E.d1i : E.d0i;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float nr = Dr[c] * er - Di[c] * ei + E.j[c] * (Pr * dr - Pi * di);
          const float ni = Dr[c] * ei + Di[c] * er + E.j[c] * (Pr * di + Pi * dr);
          Dr[c] = nr; Di[c] = ni;
        }
        const float npr = Pr * er - Pi * ei, npi = Pr * ei + Pi * er;
        Pr = npr; Pi = npi;
      });
      const QEnc Q[3] = {enc.template get<0>(), enc.template get<1>(), enc.template get<2>()};
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float pr = Pr, pi = Pi, dr[3] = {Dr[0], Dr[1], Dr[2]}, di[3] = {Di[0], Di[1], Di[2]};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const bool b = (r >> i) & 1;
          const float er = b ? Q[i].e1r : Q[i].e0r, ei = b ? Q[i].e1i : Q[i].e0i;
          const float ddr = b ? Q[i].d1r : Q[i].d0r, ddi = b ? Q[i].d1i : Q[i].d0i;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const float nr = dr[c] * er - di[c] * ei + Q[i].j[c] * (pr * ddr - pi * ddi);
            const float ni = dr[c] * ei + di[c] * er + Q[i].j[c] * (pr * ddi + pi * ddr);
            dr[c] = nr; di[c] = ni;
          }
          const float npr = pr * er - pi * ei, npi = pr * ei + pi * er;
          pr = npr; pi = npi;
        }
        sr[0][r] = pr; si[0][r] = pi;
#pragma unroll
        for (int c = 0; c < 3; ++c) { sr[1 + c][r] = dr[c]; si[1 + c][r] = di[c]; }
      }
    }
    // ---------------- forward ----------------------------------------------------------------
    if constexpr (RND) {
      constexpr int NS = swap_slots(N);
      CP<QXchg> xf = reinterpret_cast<CP<QXchg>>(pb + plan->off_xf);
      const QLane* __restrict__ lanes =
          reinterpret_cast<const QLane*>(reinterpret_cast<const char*>(a.plan) + plan->off_lanes);
      const int R = plan->n_rounds;
      if constexpr (N >= 10 && EXS == 4) {
        // Software-pipelined: group A = statevectors {0, 1} (planes 0, 1), group B = {2, 3} (planes 2, 3).
        // Each slot reads one group, finishes the other group's round (its bit-2 gate and swap slots)
        // and writes it, then runs the bit-0/1 gates of the group just read: the finishing work covers
        // the read latency and the writes drain under the following gates.  Every barrier separates a
        // plane pair's reads from its next writes.
        // All four statevectors complete in round k0 - 1's output mapping: the encoding leaves them
        // there when the opening stage is folded (k0 = H); otherwise round 0 runs here (k0 = 1).
        int k0 = H;
        RoundCoef Rc = load_round<NS>(rounds + (H > 0 ? H - 1 : 0), gtab, a.n_gates);
        if (k0 == 0) {
          round_fwd<0, NS>(sr, si, Rc);
          round_fwd<2, NS>(sr, si, Rc);
          k0 = 1;
        }
        if (k0 < R) {
          Offs wo = load_offs(xf[k0].woff);
          // lane words of the current exchange as scalars (updated inside the lambda below)
          uint32_t xwb, xrb, xsg;
          {
            const XLane x0 = lane_words(lanes, k0, TP, u, pb8);
            xwb = x0.wb; xrb = x0.rb; xsg = x0.sgn;
          }
          rwrite<T, 0, 1, 0>(sr, si, buf, wo, xwb);
          // Iteration k: group A is read and runs round k; group B lags by half a round (it finishes
          // round k - 1 while A's read is in flight, except in the first iteration, where it is
          // complete).  The first iteration is peeled so that neither copy has a branch around
          // group B's work.
          auto iter = [&](int k, auto lag) {
            constexpr bool LAG = decltype(lag)::value != 0;
            CP<QRound> rk = rounds + k;
            const RoundCoef Rk = load_round<NS>(rk, gtab, a.n_gates);
            const Offs ro = load_offs(xf[k].roff);
            const bool sg = xf[k].nterms != 0;
            // the next exchange's lane words: a vector load issued a whole round ahead of its use
            XLane xn{xwb, xrb, xsg};
            if (k + 1 < R) xn = lane_words(lanes, k + 1, TP, u, pb8);
            __syncthreads();
            rread<T, 0, 1, 0>(sr, si, buf, ro, sg, xrb, xsg);
            if (LAG) finish<2, NS>(sr, si, Rc);          // group B finishes round k - 1
            rwrite<T, 2, 3, 2>(sr, si, buf, wo, xwb);
            gates01<0>(sr, si, Rk);
            pin_sv<0>(sr, si); pin_sv<1>(sr, si);
            // The next exchange's write offsets, loaded before the barrier: scalar loads share the
            // wait counter with LDS operations, and waiting here costs nothing.
            if (k + 1 < R) wo = load_offs(xf[k + 1].woff);
            __syncthreads();
            rread<T, 2, 3, 2>(sr, si, buf, ro, sg, xrb, xsg);
            finish<0, NS>(sr, si, Rk);                   // group A finishes round k
            if (k + 1 < R) rwrite<T, 0, 1, 0>(sr, si, buf, wo, xn.wb);
            gates01<2>(sr, si, Rk);
            pin_sv<2>(sr, si); pin_sv<3>(sr, si);
            xwb = xn.wb; xrb = xn.rb; xsg = xn.sgn;
            Rc = Rk;
          };
          iter(k0, IntC<0>{});
          for (int k = k0 + 1; k < R; ++k) iter(k, IntC<1>{});
          __syncthreads();
          finish<2, NS>(sr, si, Rc);                     // group B finishes the last round
        }
      } else {
        CP<uint32_t> pcoef = reinterpret_cast<CP<uint32_t>>(gtab + (a.n_gates + 1) * kGT);
        const QPhaseStage* pstages =
            reinterpret_cast<const QPhaseStage*>(reinterpret_cast<const char*>(a.plan) + plan->off_phase);
        for (int k = H; k < R; ++k) {
          CP<QRound> rk = rounds + k;
          if (k > 0) rexchange<N, T>(sr, si, buf, xf + k, lane_words(lanes, k, TP, u, pb8));
          if (rk->phase >= 0) {   // CRZ phase stage after the exchange
            float pc[8], ps[8];
            phase_factors<N>(rk, pcoef + to_const(pstages)[rk->phase].coef_off, u, pc, ps);
            mul_phase<0, false>(sr, si, pc, ps); mul_phase<1, false>(sr, si, pc, ps);
            mul_phase<2, false>(sr, si, pc, ps); mul_phase<3, false>(sr, si, pc, ps);
          }
          const RoundCoef Rk = load_round<NS>(rk, gtab, a.n_gates);
          round_fwd<0, NS>(sr, si, Rk);
          round_fwd<2, NS>(sr, si, Rk);
        }
      }
    } else if constexpr (N < 10) {
      for (int l = L0; l < L1; ++l) {
        CP<QSweep> L = sweeps + l;
        const Phase P = phase_of(l);
        const Coef<N> K = load_coef<N>(tcoef + l * kTC, v, false);
        if (L->flags & kSweepXchg) {
          const uint4 w = lane_of(l);
          const Addr A = xchg_addr(L->woff, L->roff, w.x ^ pb8, w.y ^ pb8);
          exchange_wave<T, 0, 4>(sr, si, buf, A);
        }
        const int has = positions(L);
        layer_fwd<N, 0>(sr, si, K, P, has);
        layer_fwd<N, 1>(sr, si, K, P, has);
        layer_fwd<N, 2>(sr, si, K, P, has);
        layer_fwd<N, 3>(sr, si, K, P, has);
      }
    } else if constexpr (EXS == 4) {
      // Statevectors {0, 1} go through planes 0 and 1, {2, 3} through planes 2 and 3: between two
      // barriers one group is read and rotated while the other is written, so every barrier
      // separates a plane's reads from its next writes.
      Addr A;
      auto addr = [&](int l) {
        const uint4 w = lane_of(l);
        A = xchg_addr(sweeps[l].woff, sweeps[l].roff, w.x ^ pb8, w.y ^ pb8);
      };
      if (L0 < L1 && (sweeps[L0].flags & kSweepXchg)) {
        addr(L0);
        xwrite<T, 0, 0>(sr, si, buf, A.w); xwrite<T, 1, 1>(sr, si, buf, A.w);
      }
      for (int l = L0; l < L1; ++l) {
        CP<QSweep> L = sweeps + l;
        const int has = positions(L);
        const bool moves = has & kSweepXchg, wave_bits = has & kSweepWave;
        const Phase P = phase_of(l);
        const Coef<N> K = load_coef<N>(tcoef + l * kTC, v, false);
        if (moves) {
          __syncthreads();
          xread<T, 0, 0>(sr, si, buf, A.r); xread<T, 1, 1>(sr, si, buf, A.r);
          xwrite<T, 2, 2>(sr, si, buf, A.w); xwrite<T, 3, 3>(sr, si, buf, A.w);
        }
        layer_fwd<N, 0>(sr, si, K, P, has);
        layer_fwd<N, 1>(sr, si, K, P, has);
        if (moves) {
          __syncthreads();
          xread<T, 2, 2>(sr, si, buf, A.r); xread<T, 3, 3>(sr, si, buf, A.r);
        }
        if (wave_bits) {
          wwrite<N, T, 0, 0>(sr, si, buf, wvb); wwrite<N, T, 1, 1>(sr, si, buf, wvb);
        }
        layer_fwd<N, 2>(sr, si, K, P, has);
        layer_fwd<N, 3>(sr, si, K, P, has);
        if (wave_bits) {
          __syncthreads();
          wread<N, T, 0, 0>(sr, si, buf, rvb); wread<N, T, 1, 1>(sr, si, buf, rvb);
          wwrite<N, T, 2, 2>(sr, si, buf, wvb); wwrite<N, T, 3, 3>(sr, si, buf, wvb);
          rot_wave<N, 0>(sr, si, K); rot_wave<N, 1>(sr, si, K);
          __syncthreads();
          wread<N, T, 2, 2>(sr, si, buf, rvb); wread<N, T, 3, 3>(sr, si, buf, rvb);
        }
        if (l + 1 < L1 && (sweeps[l + 1].flags & kSweepXchg)) {
          addr(l + 1);
          xwrite<T, 0, 0>(sr, si, buf, A.w); xwrite<T, 1, 1>(sr, si, buf, A.w);
        }
        if (wave_bits) { rot_wave<N, 2>(sr, si, K); rot_wave<N, 3>(sr, si, K); }
      }
    } else {
      for (int l = L0; l < L1; ++l) {
        CP<QSweep> L = sweeps + l;
        const Phase P = phase_of(l);
        const Coef<N> K = load_coef<N>(tcoef + l * kTC, v, false);
        const int has = positions(L);
        const bool moves = has & kSweepXchg;
        const uint4 w = lane_of(l);
        const Addr A = xchg_addr(L->woff, L->roff, w.x ^ pb8, w.y ^ pb8);
        auto pair = [&](auto c) {
          constexpr int S = decltype(c)::value;
          if (moves) {
            xwrite<T, S, 0>(sr, si, buf, A.w); xwrite<T, S + 1, 1>(sr, si, buf, A.w);
            __syncthreads();
            xread<T, S, 0>(sr, si, buf, A.r); xread<T, S + 1, 1>(sr, si, buf, A.r);
            __syncthreads();
          }
          layer_fwd<N, S>(sr, si, K, P, has);
          layer_fwd<N, S + 1>(sr, si, K, P, has);
          if (has & kSweepWave) {
            wwrite<N, T, S, 0>(sr, si, buf, wvb); wwrite<N, T, S + 1, 1>(sr, si, buf, wvb);
            __syncthreads();
            wread<N, T, S, 0>(sr, si, buf, rvb); wread<N, T, S + 1, 1>(sr, si, buf, rvb);
            __syncthreads();
            rot_wave<N, S>(sr, si, K); rot_wave<N, S + 1>(sr, si, K);
          }
        };
        pair(IntC<0>{});
        pair(IntC<2>{});
      }
    }
    // ---------------- readout ----------------------------------------------------------------
    CP<int32_t> ft = RND ? rounds[plan->n_rounds - 1].tpost : plan->ftpos;
    uint32_t jl = deposit_thread<N>(RND ? u : v, ft);
    uint32_t l0 = ft[0], l1 = ft[1], l2 = ft[2];
    float acc[kMaxOut * 4];
#pragma unroll
    for (int i = 0; i < kMaxOut * 4; ++i) acc[i] = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t j = jl ^ reg_off(r, l0, l1, l2);
      // per output: <Z> and its three input tangents, or (packed) <Z> of the four slots' points
      const float p2 = sr[0][r] * sr[0][r] + si[0][r] * si[0][r];
      float gc[3];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        gc[c] = PK ? sr[1 + c][r] * sr[1 + c][r] + si[1 + c][r] * si[1 + c][r]
                   : 2.f * (sr[0][r] * sr[1 + c][r] + si[0][r] * si[1 + c][r]);
#pragma unroll
      for (int i = 0; i < kMaxOut; ++i) {
        if (i < m) {
          const float z = parity(plan->zmask[i] & j) ? -1.f : 1.f;
          acc[i * 4 + 0] += z * p2;
          acc[i * 4 + 1] += z * gc[0];
          acc[i * 4 + 2] += z * gc[1];
          acc[i * 4 + 3] += z * gc[2];
        }
      }
    }
    // all-reduce over the point's thread group
    if (TP <= 64) {
#pragma unroll
      for (int off = 1; off < (TP < 64 ? TP : 64); off <<= 1)
#pragma unroll
        for (int i = 0; i < kMaxOut * 4; ++i)
          if (i < 4 * m) acc[i] += __shfl_xor(acc[i], off);
    } else {
#pragma unroll
      for (int off = 1; off < 64; off <<= 1)
#pragma unroll
        for (int i = 0; i < kMaxOut * 4; ++i)
          if (i < 4 * m) acc[i] += __shfl_xor(acc[i], off);
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < kMaxOut * 4; ++i)
          if (i < 4 * m) red[wave * 40 + i] = acc[i];
      }
      __syncthreads();
      constexpr int WPP = TP / 64;   // waves per point
      const int w0 = (wave / WPP) * WPP;
#pragma unroll
      for (int i = 0; i < kMaxOut * 4; ++i) {
        if (i < 4 * m) {
          float s = 0.f;
          for (int w = 0; w < WPP; ++w) s += red[(w0 + w) * 40 + i];
          acc[i] = s;
        }
      }
      __syncthreads();
    }
    if (PK && u == 0 && a.out) {
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        if (pt0 + sl >= a.P) break;
#pragma unroll
        for (int i = 0; i < kMaxOut; ++i) {
          if (i >= m) break;
          a.out[(pt0 + sl) * m + i] = acc[i * 4 + sl];
        }
      }
    }
    if (!PK && valid && u == 0) {
#pragma unroll
      for (int i = 0; i < kMaxOut; ++i) {
        if (i >= m) break;
        if (a.out) a.out[pt * m + i] = acc[i * 4];
        if (a.tan) {
          a.tan[(pt * m + i) * 3 + 0] = acc[i * 4 + 1];
          a.tan[(pt * m + i) * 3 + 1] = acc[i * 4 + 2];
          a.tan[(pt * m + i) * 3 + 2] = acc[i * 4 + 3];
        }
      }
    }
    if constexpr (mode_fwd_only(MODE)) return;

    // ---------------- seeds -----------------------------------------------------------------
    float Wv[kMaxOut][3], Vv[kMaxOut];
#pragma unroll
    for (int i = 0; i < kMaxOut; ++i) { Vv[i] = 0.f; Wv[i][0] = Wv[i][1] = Wv[i][2] = 0.f; }
    if (MODE == kModeMaxwell || MODE == kModeTotal) {
      if (valid) {
        const float gEt = acc[1], gEx = acc[2], gEy = acc[3];
        const float gXt = acc[5], gXy = acc[7];
        const float gYt = acc[9], gYx = acc[10];
        float eps = 1.f, w1 = w_all;
        if (a.loss_kind != QP_LOSS_VACUUM) {
          const float x = a.points[pt * 3 + 1];
          const bool diel = x >= a.x_if;
          eps = diel ? a.eps_r : 1.f;
          if (a.loss_kind == QP_LOSS_DIEL_SPLIT) w1 = diel ? w_diel : w_vac;
        }
        const float ie = 1.f / eps;
        const float r1 = gEt - (gYx - gXy) * ie;
        const float r2 = gXt + gEy;
        const float r3 = gYt - gEx;
        const float w = w_all;
        lacc += (u == 0) ? (w1 * r1 * r1 + w * (r2 * r2 + r3 * r3)) : 0.f;
        const float A = 2.f * w1 * r1, Bq = 2.f * w * r2, C = 2.f * w * r3;
        Wv[0][0] = A;  Wv[2][1] = -A * ie;  Wv[1][2] = A * ie;
        Wv[1][0] = Bq; Wv[0][2] += Bq;
        Wv[2][0] = C;  Wv[0][1] += -C;
        if constexpr (MODE == kModeTotal) {
          // the energy term, mean square of the local Poynting residual e (eq. energy_loss), and
          // this point's share of the symmetry term (eq. 2D_symLoss) against its mirror images
          const float E = acc[0], Hx = acc[4], Hy = acc[8];
          const float e = eps * E * gEt + Hx * gXt + Hy * gYt - (gEx * Hy + E * gYx) + (gEy * Hx + E * gXy);
          const float k = a.w_energy * 2.f * e * w;
          Vv[0] += k * (eps * gEt - gYx + gXy);
          Vv[1] += k * (gXt + gEy);
          Vv[2] += k * (gYt - gEx);
          Wv[0][0] += k * eps * E; Wv[0][1] += -k * Hy; Wv[0][2] += k * Hx;
          Wv[1][0] += k * Hx;      Wv[1][2] += k * E;
          Wv[2][0] += k * Hy;      Wv[2][1] += -k * E;
          const float ks = a.w_sym * 2.f * w;
          for (int j = 0; j < a.n_mir; ++j) {   // parities: y-mirror (+, -, +), x-mirror (+, +, -)
            const float* fm = a.f_mir + ((long long)j * a.P + pt) * m;
            Vv[0] += ks * (E - fm[0]);
            Vv[1] += ks * (j == 0 ? Hx + fm[1] : Hx - fm[1]);
            Vv[2] += ks * (j == 0 ? Hy - fm[2] : Hy + fm[2]);
          }
        }
      }
    } else if (PK) {   // output seeds of the four slots' points: slot 0 in Vv, slot c + 1 in Wv[.][c]
      if (a.d_out) {
#pragma unroll
        for (int i = 0; i < kMaxOut; ++i) {
          if (i >= m) break;
          if (pt0 < a.P) Vv[i] = a.d_out[pt0 * m + i];
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (pt0 + 1 + c < a.P) Wv[i][c] = a.d_out[(pt0 + 1 + c) * m + i];
        }
      }
    } else {   // VJP seeds
      if (valid) {
#pragma unroll
        for (int i = 0; i < kMaxOut; ++i) {
          if (i >= m) break;
          if (a.d_out) Vv[i] = a.d_out[pt * m + i];
          if (a.d_tan) {
            Wv[i][0] = a.d_tan[(pt * m + i) * 3 + 0];
            Wv[i][1] = a.d_tan[(pt * m + i) * 3 + 1];
            Wv[i][2] = a.d_tan[(pt * m + i) * 3 + 2];
          }
        }
      }
    }
    if constexpr (RND) {
      // From the rounds' mapping to the sweeps', and behind the last layer's diagonal part (which the
      // readout does not see): an exchange and a phase.
      CP<QTurn> turn = reinterpret_cast<CP<QTurn>>(pb + plan->off_turn);
      const uint2 w = reinterpret_cast<const uint2*>(reinterpret_cast<const char*>(a.plan) + plan->off_tlanes)[u];
      const Addr A = xchg_addr(turn->woff, turn->roff, w.x ^ pb8, w.y ^ pb8);
      const Phase P = phase_of(L1);
      if constexpr (N < 10) {
        exchange_wave<T, 0, 4>(sr, si, buf, A);
      } else {
        __syncthreads();
        xwrite<T, 0, 0>(sr, si, buf, A.w); xwrite<T, 1, 1>(sr, si, buf, A.w);
        __syncthreads();
        xread<T, 0, 0>(sr, si, buf, A.r); xread<T, 1, 1>(sr, si, buf, A.r);
        __syncthreads();
        xwrite<T, 2, 0>(sr, si, buf, A.w); xwrite<T, 3, 1>(sr, si, buf, A.w);
        __syncthreads();
        xread<T, 2, 0>(sr, si, buf, A.r); xread<T, 3, 1>(sr, si, buf, A.r);
        __syncthreads();
      }
      mul_phase<0, true>(sr, si, P.c, P.s); mul_phase<1, true>(sr, si, P.c, P.s);
      mul_phase<2, true>(sr, si, P.c, P.s); mul_phase<3, true>(sr, si, P.c, P.s);
      CP<int32_t> f2 = plan->ftpos;
      jl = deposit_thread<N>(v, f2);
      l0 = f2[0]; l1 = f2[1]; l2 = f2[2];
    }
    // lambda = Df psi + sum_c D_c dpsi_c, mu_c = D_c psi (D real diagonal in the final basis)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t j = jl ^ reg_off(r, l0, l1, l2);
      float Df = 0.f, D0 = 0.f, D1 = 0.f, D2 = 0.f;
#pragma unroll
      for (int i = 0; i < kMaxOut; ++i) {
        if (i < m) {
          const float z = parity(plan->zmask[i] & j) ? -1.f : 1.f;
          Df += z * Vv[i];
          D0 += z * Wv[i][0];
          D1 += z * Wv[i][1];
          D2 += z * Wv[i][2];
        }
      }
      if (PK) {   // lambda of each slot's point, paired with that slot's psi
        sr[4][r] = Df * sr[0][r]; si[4][r] = Df * si[0][r];
        sr[5][r] = D0 * sr[1][r]; si[5][r] = D0 * si[1][r];
        sr[6][r] = D1 * sr[2][r]; si[6][r] = D1 * si[2][r];
        sr[7][r] = D2 * sr[3][r]; si[7][r] = D2 * si[3][r];
      } else {
        sr[4][r] = Df * sr[0][r] + D0 * sr[1][r] + D1 * sr[2][r] + D2 * sr[3][r];
        si[4][r] = Df * si[0][r] + D0 * si[1][r] + D1 * si[2][r] + D2 * si[3][r];
        sr[5][r] = D0 * sr[0][r]; si[5][r] = D0 * si[0][r];
        sr[6][r] = D1 * sr[0][r]; si[6][r] = D1 * si[0][r];
        sr[7][r] = D2 * sr[0][r]; si[7][r] = D2 * si[0][r];
      }
    }
    // ---------------- adjoint sweep with uncompute -----------------------------------------
    // Per layer in reverse: psi-family (uncompute) and lambda-family through the inverse rotations, gate
    // statistics, conjugate phase, inverse exchange.  The pair (psi_c, lambda_c) for c = 0..3 is a
    // self-contained group (its gates and its share of the statistics need no other statevector).
    // Layers below L0 (the opening layer, folded into the encoding) only take their statistics.
    Stats<N> Q;
    auto mom_of = [&](CP<QSweep> L) -> float* {
      return L->phase >= 0 ? mslots + wave * a.n_mom + L->phase * phase_terms(N) : nullptr;
    };
    if constexpr (N < 10) {
      auto layer = [&](int l, auto pull) {
        constexpr bool PULL = decltype(pull)::value != 0;
        CP<QSweep> L = sweeps + l;
        Phase P{};
        if (PULL) P = phase_of(l);
        const Coef<N> K = load_coef<N>(tcoef + l * kTC, v, true);
        clear(Q);
        const int has = positions(L);
        layer_adj<N, 0, PULL>(sr, si, K, P, Q, has);
        layer_adj<N, 1, PULL>(sr, si, K, P, Q, has);
        layer_adj<N, 2, PULL>(sr, si, K, P, Q, has);
        layer_adj<N, 3, PULL>(sr, si, K, P, Q, has);
        flush_xy<N, 0, N, THIN>(L, Q, v, slots, F, wave, lane);
        flush_z<N>(L, Q.w, v, slots, mom_of(L), F, wave, lane);
        if (PULL && (L->flags & kSweepXchg) && (l > 0 || EG)) {   // (nothing follows the first layer else)
          const uint4 w = lane_of(l);
          const Addr A = xchg_addr(L->bwoff, L->broff, w.z ^ pb8, w.w ^ pb8);
          exchange_wave<T, 0, 8>(sr, si, buf, A);
        }
      };
      for (int l = L1 - 1; l >= L0; --l) layer(l, IntC<1>{});
      if (L0 > 0) layer(0, IntC<0>{});
    } else if constexpr (EXS == 4) {
      // Pair c goes through planes 2 (c & 1) and 2 (c & 1) + 1.  Between two barriers one pair is read,
      // the next one written, and the pair just read rotated and its statistics taken.  A layer takes
      // two such passes: the wave positions (behind the index-map exchange of the layer above, if it
      // has one), then, behind the wave exchange, the rest.  The statistics of a pass are flushed at
      // its end, and the first pair of an index-map exchange is written after that: with both live the
      // kernel spilled.
      auto wpair = [&](auto c) {   // wave exchange, writes
        constexpr int C = decltype(c)::value, PL = 2 * (C & 1);
        wwrite<N, T, C, PL>(sr, si, buf, wvb); wwrite<N, T, 4 + C, PL + 1>(sr, si, buf, wvb);
      };
      Addr A;
      auto xpair = [&](auto c) {   // index-map exchange, writes
        constexpr int C = decltype(c)::value, PL = 2 * (C & 1);
        xwrite<T, C, PL>(sr, si, buf, A.w); xwrite<T, 4 + C, PL + 1>(sr, si, buf, A.w);
      };
      auto xstep = [&](auto c) {
        constexpr int C = decltype(c)::value, PL = 2 * (C & 1);
        __syncthreads();
        xread<T, C, PL>(sr, si, buf, A.r); xread<T, 4 + C, PL + 1>(sr, si, buf, A.r);
        if constexpr (C < 3) xpair(IntC<C + 1>{});
      };
      bool moves = false;          // the layer above ended with its index-map exchange's first write
      auto enter = [&](int l, auto pull) {
        constexpr bool PULL = decltype(pull)::value != 0;
        const Coef<N> K = load_coef<N, 9, N>(tcoef + l * kTC, v, true);
        const bool wave_bits = positions(sweeps + l) & kSweepWave;
        clear<N, 9, N>(Q);
        auto step = [&](auto c) {
          constexpr int C = decltype(c)::value;
          if (moves) xstep(c);
          if (!wave_bits) return;
          if (PULL) wave_rot<N, C>(sr, si, K);
          wave_stat<N, C>(sr, si, Q);
          if constexpr (C == 3) wpair(IntC<0>{});
        };
        step(IntC<0>{}); step(IntC<1>{}); step(IntC<2>{}); step(IntC<3>{});
        flush_xy<N, 9, N, THIN>(sweeps + l, Q, v, slots, F, wave, lane);
      };
      auto rest = [&](int l, auto pull) {
        constexpr bool PULL = decltype(pull)::value != 0;
        CP<QSweep> L = sweeps + l;
        Phase P{};
        if (PULL) P = phase_of(l);
        const Coef<N> K = load_coef<N, 0, 9>(tcoef + l * kTC, v, true);
        const int has = positions(L);
        clear<N, 0, 9>(Q);
        auto step = [&](auto c) {
          constexpr int C = decltype(c)::value, PL = 2 * (C & 1);
          if (has & kSweepWave) {
            __syncthreads();
            wread<N, T, C, PL>(sr, si, buf, rvb); wread<N, T, 4 + C, PL + 1>(sr, si, buf, rvb);
            if constexpr (C < 3) wpair(IntC<C + 1>{});
          }
          layer_adj<N, C, PULL>(sr, si, K, P, Q, has);
        };
        step(IntC<0>{}); step(IntC<1>{}); step(IntC<2>{}); step(IntC<3>{});
        flush_xy<N, 0, 9, THIN>(L, Q, v, slots, F, wave, lane);
        flush_z<N>(L, Q.w, v, slots, mom_of(L), F, wave, lane);
        moves = PULL && (L->flags & kSweepXchg) && (l > 0 || EG);
        if (moves) {
          const uint4 w = lane_of(l);
          A = xchg_addr(L->bwoff, L->broff, w.z ^ pb8, w.w ^ pb8);
          xpair(IntC<0>{});
        }
      };
      for (int l = L1 - 1; l >= L0; --l) {
        enter(l, IntC<1>{});
        rest(l, IntC<1>{});
      }
      if (L0 > 0) {
        enter(0, IntC<0>{});
        rest(0, IntC<0>{});
      } else if (EG && moves) {
        xstep(IntC<0>{}); xstep(IntC<1>{}); xstep(IntC<2>{}); xstep(IntC<3>{});
      }
      __syncthreads();
    } else {
      auto layer = [&](int l, auto pull) {
        constexpr bool PULL = decltype(pull)::value != 0;
        CP<QSweep> L = sweeps + l;
        Phase P{};
        if (PULL) P = phase_of(l);
        const Coef<N> K = load_coef<N>(tcoef + l * kTC, v, true);
        const int has = positions(L);
        const bool moves = PULL && (has & kSweepXchg) && (l > 0 || EG);
        const uint4 w = lane_of(l);
        const Addr A = xchg_addr(L->bwoff, L->broff, w.z ^ pb8, w.w ^ pb8);
        clear(Q);
        auto pair = [&](auto c) {
          constexpr int C = decltype(c)::value;
          if (has & kSweepWave) {
            if (PULL) wave_rot<N, C>(sr, si, K);
            wave_stat<N, C>(sr, si, Q);
            wwrite<N, T, C, 0>(sr, si, buf, wvb); wwrite<N, T, 4 + C, 1>(sr, si, buf, wvb);
            __syncthreads();
            wread<N, T, C, 0>(sr, si, buf, rvb); wread<N, T, 4 + C, 1>(sr, si, buf, rvb);
            __syncthreads();
          }
          layer_adj<N, C, PULL>(sr, si, K, P, Q, has);
          if (moves) {
            xwrite<T, C, 0>(sr, si, buf, A.w); xwrite<T, 4 + C, 1>(sr, si, buf, A.w);
            __syncthreads();
            xread<T, C, 0>(sr, si, buf, A.r); xread<T, 4 + C, 1>(sr, si, buf, A.r);
            __syncthreads();
          }
        };
        pair(IntC<0>{}); pair(IntC<1>{}); pair(IntC<2>{}); pair(IntC<3>{});
        flush_xy<N, 0, N, THIN>(L, Q, v, slots, F, wave, lane);
        flush_z<N>(L, Q.w, v, slots, mom_of(L), F, wave, lane);
      };
      for (int l = L1 - 1; l >= L0; --l) layer(l, IntC<1>{});
      if (L0 > 0) layer(0, IntC<0>{});
    }
    if constexpr (EG) {
      // the point index again, from an opaque copy of the thread index: keeping pt and valid live
      // through the adjoint sweep would cost registers there
      uint32_t t2 = threadIdx.x;
      asm volatile("" : "+v"(t2));
      const long long pt2 = PK ? 0 : (long long)tile * PPW + (long long)(t2 / TP);
      if constexpr (N < 10) encoding_grads_wave<N>(sr, si, Q, plan, gtab, a, pt2, pt2 < a.P && u == 0, v);
      else encoding_grads<N, T>(sr, si, buf, red, plan, gtab, a, pt2, pt2 < a.P, u);
    }
  }
}

// ---- the fused kernel: a persistent grid walks the tiles ------------------------------------
template <int N, int T, int EXS, int MODE, bool EG = false, bool THIN = false>
__global__ __launch_bounds__(T, mode_fwd_only(MODE) ? fwd_waves(N, EXS, MODE) : 2) void k_fused(FusedArgs a) {
  constexpr int WAVES = T / 64;
  constexpr int PLANE = T * 8;
  // Exchange planes in static LDS (their address is a link-time constant, so every access is
  // one XOR of a byte offset); gate statistics and readout scratch in the dynamic part.
  __shared__ float4 planes[sweep_planes(N, EXS, mode_rounds(MODE)) * PLANE / 2];
  extern __shared__ float4 smem4[];
  float2* buf = reinterpret_cast<float2*>(planes);
  float* slots = reinterpret_cast<float*>(smem4);                   // [WAVES][F][kGS]
  float* mslots = slots + WAVES * a.n_fused * kGS;                   // [WAVES][n_mom] phase moments
  float* red = mslots + WAVES * a.n_mom;                             // [WAVES][40]
  const int F = a.n_fused;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  if (!mode_fwd_only(MODE)) {
    for (int i = tid; i < WAVES * (F * kGS + a.n_mom); i += T) slots[i] = 0.f;
  }
  __syncthreads();
  float lacc = 0.f;
  // XCD-aware tile order: workgroups are dealt round-robin to the 8 XCDs (blockIdx % 8), so each
  // XCD walks one contiguous range of tiles and neighbouring points' output lines are written
  // through one L2 instead of eight.
  constexpr int kXcd = 8;
  int t_begin = blockIdx.x, t_end = a.ntiles, t_step = gridDim.x;
  if (gridDim.x % kXcd == 0) {
    const int chunk = (a.ntiles + kXcd - 1) / kXcd;
    t_begin = (blockIdx.x % kXcd) * chunk + blockIdx.x / kXcd;
    t_end = min(a.ntiles, (int)(blockIdx.x % kXcd) * chunk + chunk);
    t_step = gridDim.x / kXcd;
  }
  for (int tile = t_begin; tile < t_end; tile += t_step)
    fused_tile<N, T, EXS, MODE, EG, THIN>(a, tile, buf, slots, mslots, red, lacc);
  if (mode_fwd_only(MODE)) return;
  // ---------------- per-workgroup partials (fixed order) -----------------------------------
  __syncthreads();
  const int ncol = F * kGS + a.n_mom;
  for (int i = tid; i < F * kGS; i += T) {
    float s = 0.f;
    for (int w = 0; w < WAVES; ++w) s += slots[w * F * kGS + i];
    a.mpart[(long long)blockIdx.x * ncol + i] = s;
  }
  for (int i = tid; i < a.n_mom; i += T) {
    float s = 0.f;
    for (int w = 0; w < WAVES; ++w) s += mslots[w * a.n_mom + i];
    a.mpart[(long long)blockIdx.x * ncol + F * kGS + i] = s;
  }
  if (MODE == kModeMaxwell) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) lacc += __shfl_xor(lacc, off);
    __syncthreads();
    if (lane == 0) red[wave * 40] = lacc;
    __syncthreads();
    if (tid == 0) {
      float s = 0.f;
      for (int w = 0; w < WAVES; ++w) s += red[w * 40];
      a.lpart[blockIdx.x] = s;
    }
  }
}


template <int N, int EXS, int MODE, bool EG, bool THIN>
hipError_t launch_one(const FusedArgs& a, int grid, size_t dyn, hipStream_t st) {
  constexpr int T = fused_wg_threads(N);
  auto kern = k_fused<N, T, EXS, MODE, EG, THIN>;
  // the attribute is set once per device (and raised when a larger size comes)
  static size_t attr_bytes[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (dyn > 0 && dyn > attr_bytes[dev]) {
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) return e;
    attr_bytes[dev] = dyn;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(T), dyn, st, a);
  return hipGetLastError();
}

// Entry point of one per-N unit.  exs: exchange planes (2 or 4) from 10 qubits on; below, an exchange
// stays inside a wave and one kernel serves both.  Thin circuits have kernels of their own, with branches around
// what a layer leaves out (24 layers, adjoint: 3 of 9 qubits rotated 806 -> 412 us, 3 of 11 1007 -> 454, 4 of 12 1111 -> 599);
// in one kernel with the rest, the branches cost full layers 1 to 6 % from 7 qubits on.
// Input gradients take two planes (4 layers, 2^23 amplitudes, adjoint: 10 qubits 1140 us with four planes, 997 with
// two; 11: 1230, 1053; 12: 1278, 1181; with the loss 1251 and 1217, 1330 and 1227, 1506 and 1397; 32 points 126 and
// 119, 135 and 125, 170 and 166): with four planes their kernels spill 160 to 330 registers.
template <int N, int EXS, int MODE, bool EG>
hipError_t launch_kind(const FusedArgs& a, int grid, size_t dyn, hipStream_t st) {
  constexpr bool kThin = N >= kThinQubits && MODE != kModeFieldsPk;   // (kModeFieldsPk runs no layers)
  if constexpr (kThin) {
    if (a.thin) return launch_one<N, EXS, MODE, EG, true>(a, grid, dyn, st);
  }
  return launch_one<N, EXS, MODE, EG, false>(a, grid, dyn, st);
}
template <int N, int MODE, bool EG = false>
hipError_t launch_mode(const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st) {
  if constexpr (N >= 10 && !EG) {
    if (exs == 4) return launch_kind<N, 4, MODE, EG>(a, grid, dyn, st);
  }
  return launch_kind<N, 2, MODE, EG>(a, grid, dyn, st);
}
template <int N>
hipError_t launch_fused_n(int mode, const FusedArgs& a, int grid, int exs, size_t dyn, hipStream_t st) {
  const bool eg = a.d_angles || a.d_jac;   // per-point input gradients
  switch (mode) {
    case kModeFwd: return launch_mode<N, kModeFwd>(a, grid, exs, dyn, st);
    case kModeFwdPk: return launch_mode<N, kModeFwdPk>(a, grid, exs, dyn, st);
    case kModeFieldsPk: return launch_mode<N, kModeFieldsPk>(a, grid, exs, dyn, st);
    case kModeTotal: return launch_mode<N, kModeTotal>(a, grid, exs, dyn, st);
    case kModeVjpPk: return launch_mode<N, kModeVjpPk>(a, grid, exs, dyn, st);
    case kModeMaxwell:
      return eg ? launch_mode<N, kModeMaxwell, true>(a, grid, exs, dyn, st) : launch_mode<N, kModeMaxwell>(a, grid, exs, dyn, st);
    default:
      return eg ? launch_mode<N, kModeVjp, true>(a, grid, exs, dyn, st) : launch_mode<N, kModeVjp>(a, grid, exs, dyn, st);
  }
}

}  // namespace qp

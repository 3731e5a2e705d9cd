// Internal types shared by the planner (host C++) and the gfx950 kernels.
//
// All fields are 32-bit so that the kernels read them with scalar loads.
//
// Index conventions: a basis index j of an n-qubit state has qubit q in bit (n-1-q), so
// qubit 0 is the most significant bit.  "Logical" index = the index of the state the circuit
// defines.  In the fused kernels a thread owns 8 amplitudes of each statevector: its three
// "register" bits r0,r1,r2 plus n-3 "thread" bits u.  A round's mapping tpos[k] gives the
// logical index-bit position of physical bit k (k = 0..2 register bits, k >= 3 thread bit k-3).
#pragma once
#include <cstdint>

#if defined(__HIPCC__) || defined(__HIP__)
#define QP_HD __host__ __device__
#else
#define QP_HD
#endif

namespace qp {

// LDS index swizzle of the fused kernels: XOR the low nibble with the fold of all higher
// nibbles.  A bijection, and linear over GF(2): swz(a ^ b) = swz(a) ^ swz(b).
QP_HD inline constexpr uint32_t lds_swizzle(uint32_t idx) {
  return idx ^ (((idx >> 4) ^ (idx >> 8) ^ (idx >> 12) ^ (idx >> 16)) & 15u);
}

constexpr int kMaxQubits = 12;     // fused register/LDS kernels
constexpr int kMaxDevices = 64;    // per-device host-side state (launch attributes, scratch addresses)
constexpr int kMaxQubitsPlain = 14;
constexpr int kMaxOut = 8;
constexpr int kMaxTerms = 32;      // sign terms of one entangler stage
constexpr int kRegBits = 3;        // 8 amplitudes per thread per statevector
// Per fused gate the adjoint sweep accumulates S_k = Im <lambda|sigma_k|psi> (k = x, y, z) over
// all points and statevector pairs, stored as kGS floats/doubles per gate (the last unused).
constexpr int kGS = 4;
// Gate-table entry: U, 8 floats, row-major complex.
constexpr int kGT = 8;

// Swap slots of a round: after its three register-bit gates, register bit i (i < swap_slots(n))
// trades places with thread bit 4 + i (lane bit 4 or 5 of the wave, by a cross-lane swap of
// register pairs), and gate sgate[i] acts on the qubit brought in.  They are used where they turn
// a rotation stage into fewer rounds without identity slots (8 qubits: 4 + 4; 10 qubits: 5 + 5
// instead of 3 + 3 + 3 + 1; 12 qubits: 4 + 4 + 4 instead of 3 + 3 + 3 + 3).  At 6 and 9 qubits
// three-gate rounds are already full and at 11 a slot would stay empty; at 12, two swap slots
// (5 + 5 + 2) were slower than none.
QP_HD inline constexpr int swap_slots(int n) { return n == 10 ? 2 : ((n == 8 || n == 12) ? 1 : 0); }

// Threads per workgroup of the fused kernels (a thread holds 8 amplitudes of each statevector).
QP_HD inline constexpr int fused_wg_threads(int n) { return n == 12 ? 512 : 256; }

struct alignas(16) QRound {
  int32_t gate[3];    // fused-gate id applied on register bit b in the round's input mapping (-1: none)
  int32_t phase;      // phase stage applied after the exchange into this round (-1: none)
  int32_t sgate[2];   // fused-gate id applied on register bit i after swap slot i (-1: none)
  int32_t pad1[2];
  int32_t tpos[16];   // input mapping: logical index-bit position of physical bit k
  int32_t tpost[16];  // output mapping (tpos with the swap slots applied)
};
// One direction of the register exchange that precedes a round.  Reader thread (u, r) in the
// read mapping holds logical index jn = base(u) ^ jr(r); it takes the amplitude stored at
// src = A jn (A over GF(2), given by its columns), times (-1)^Q(x), where x = jn (sign in the
// destination coordinates) or x = src (sign in the source coordinates) and
// Q(x) = XOR_t parity(qu[t] & x) * parity(qv[t] & x).
struct alignas(16) QXchg {
  uint32_t acol[16];
  uint32_t src_r[8];  // A jr(r): uniform part of the source index
  uint32_t qu[kMaxTerms];
  uint32_t qv[kMaxTerms];
  uint32_t ue[3];     // bit t: parity(qu[t] & x_e(i)) for register basis i (uniform)
  uint32_t ve[3];
  uint32_t nterms;
  uint32_t sign_at_src;
  uint32_t qsign_r;   // bit r: Q(x_r) for the uniform part x_r
  uint32_t identity;  // A = I and no sign terms
  uint32_t pad1[2];
  // LDS layout of the exchange: logical index j sits at entry swz(pbase ^ M j), M an invertible
  // GF(2) map of the n index bits (columns mcol) that the planner chooses per exchange so that
  // every group of 16 lanes hits 16 distinct banks when writing and when reading.
  uint32_t roff[8];   // 8 swz(M A jr(r)): register r's uniform source offset in bytes, reader side
  uint32_t woff[8];   // 8 swz(M jr(r)): register r's offset in the writer's mapping, in bytes
  uint32_t mcol[16];
};
static_assert(sizeof(QXchg) == 528, "QXchg layout");

// Per-lane words of one exchange for the thread u of a point (u < 2^(n-3)): the writer's and the
// reader's LDS byte bases 8 swz(thread part of the index) in their mappings (the reader's through
// the index map A), and bit r set where register r's amplitude changes sign.  A point's base
// index pbase enters as 8 swz(pbase), XORed into both bases (swz is linear over GF(2)).
struct alignas(16) QLane {
  uint32_t wb, rb, sgn, pad;
};
static_assert(sizeof(QRound) == 160, "QRound layout");

// Fused single-qubit gate: U = R_{c-1} ... R_1 R_0 (component 0 acts first).  stat_out: the
// gate belongs to the leading rotation stage, which acts on the product state and is folded into
// the encoding; its statistic is taken at the gate output instead of the input.
struct alignas(16) QFused {
  int32_t qubit;
  int32_t ncomp;
  int32_t kind[3];
  int32_t param[3];
  int32_t stat_out;
  int32_t layer;   // sweep layer that applies the gate (index into the QSweep array)
  int32_t head;    // 1: the gate belongs to the opening layer folded into the encoding
  int32_t pad;
};
static_assert(sizeof(QFused) == 48, "QFused layout");

// ---- sweep layers: what the fused kernels execute ------------------------------------------------
// Every fused gate is split as U = e^{i g} RZ(a) RY(b) RZ(c).  The RZ factors of a rotation stage and
// the CZ and CRZ gates between two stages are all diagonal, so everything diagonal between one
// stage's RYs and the next one's is a single phase per basis index, tabulated once per call
// (k_sweep_tables); what is left of a stage is one real rotation per qubit, applied as
// x0' = x0 - t x1, x1' = x1 + t x0 with t = tan(b/2) and its cosine folded into the table.  Where
// |tan| would exceed one, RY(b) = RY(pi) RY(b - pi) and RY(pi) is an X and a sign: the X is not
// applied but carried along as a mask x (statevector index i stands for basis index i ^ x; the mask is
// zero at the readout), the sign goes into the next table.
//
// A layer is one rotation stage with the entanglers before it: an index-map exchange (xchg), the
// table's phase, then the RYs.  Physical bit k of an index: 0..2 register bits, 3..6 lane bits whose
// partner lane a DPP permutation reaches, 7..8 the lane bits 4 and 5 (swapped with register bits 0
// and 1 by permlane swaps), 9..11 the wave bits (swapped with register bits through LDS).  A gate at
// a position 7.. runs on the register bit it was swapped into, so the layer starts in mapping tin
// and ends in mapping tout.  Lane bits are counted in the basis 1, 2, 7, 8, 16, 32 of lane XORs (a
// half-row mirror flips lane bits 0..2 together): see sweep_thread.
constexpr int kPos = 12;
struct alignas(16) QSweep {
  int32_t gate[kPos];       // fused gate at each position (-1: none)
  int32_t flags;            // kSweepXchg: an index-map exchange comes first; kSweepPos ..: positions of gates
  int32_t phase;            // CRZ phase stage in front of the layer, or -1
  int32_t term0, nterms;    // CZ terms in front of the layer: masks [term0, term0 + nterms) of the term list
  int32_t tin[16], tout[16];
  uint32_t woff[8], roff[8];     // forward exchange: LDS byte offsets of the registers, writer and reader
  uint32_t bwoff[8], broff[8];   // reverse exchange
  uint32_t arow[16];        // index map: new index j takes the amplitude of old index A j (rows of A)
};
static_assert(sizeof(QSweep) == 384, "QSweep layout");
constexpr int kSweepXchg = 1;
// Thin circuits (QPlanDev::thin): positions a layer has gates at.  The others are neither rotated nor summed,
// and slots or wave bits with no gate at all are not swapped.  Any other circuit has all of them set.
constexpr int kThinQubits = 5;   // fewest qubits of a thin circuit
constexpr int kSweepPos = 256;   // position 0; 1 .. follow
constexpr int kSweepLane0 = kSweepPos << 3, kSweepLanes = 7 * (kSweepPos << 4), kSweepSlots = 3 * (kSweepPos << 7),
              kSweepWave = 7 * (kSweepPos << 9), kSweepAll = 0xfff * kSweepPos;
// Per thread of a point and layer: LDS byte bases of the forward and reverse exchange.
struct alignas(16) QSweepLane {
  uint32_t fwb, frb, bwb, brb;
};
// The exchange from the rounds' mapping at the readout to the sweeps' (ftpos): register offsets, and per
// thread of a point the writer's and the reader's base.
struct alignas(16) QTurn {
  uint32_t woff[8], roff[8];
};
// Lane bits reached by DPP, permlane swap slots and wave bits at n qubits.
QP_HD inline constexpr int sweep_dpp(int n) { return n < 7 ? n - 3 : 4; }
QP_HD inline constexpr int sweep_slots(int n) { return n < 8 ? 0 : (n < 9 ? 1 : 2); }
QP_HD inline constexpr int sweep_wave(int n) { return n < 10 ? 0 : n - 9; }
// Index bits of thread u of a point in the lane basis above (1 and 2 as they are, 7 for bit 2).
QP_HD inline constexpr uint32_t sweep_thread(uint32_t u, int n) { return n >= 6 ? u ^ (((u >> 2) & 1u) * 3u) : u; }
// Lane XOR that flips thread bit k.
QP_HD inline constexpr uint32_t sweep_xor(int k) { return k == 2 ? 7u : 1u << k; }
// Exchange planes a fused kernel allocates: up to 9 qubits an exchange stays inside a wave and one
// plane serves all statevectors (two: the rounds' exchange, which hands two over at a time); else exs.
QP_HD inline constexpr int sweep_planes(int n, int exs, bool two) { return n >= 10 ? exs : (two ? 2 : 1); }
constexpr int kTC = 16;            // floats per layer of the coefficient table (kPos used)
constexpr int kGP = 4;             // doubles per gate: cos c, sin c, scale of S_x and S_y, scale of S_z (sign: X mask)

// Phase stage: a run of CRZ gates (with any CZ of the same stage), all diagonal, applied as one
// phase e^{i phi(j)} per basis index after the exchange that precedes a round.  With
// CRZ(c, t)(theta) = |0><0|_c (x) I + |1><1|_c (x) RZ_t(theta),
//   phi(j) = sum_(c,t) theta_ct (-1/2) b_c(j) (1 - 2 b_t(j)) = sum_q alpha_q b_q + sum_(q<q') beta_qq' b_q b_q',
//   alpha_q = -(1/2) sum_t theta_qt,  beta_qq' = theta_qq' + theta_q'q.
// The kernels take phi from the layer's table (QSweep).  The adjoint accumulates the parity sums
// W_q = sum_j w_j z_q and W_qq' = sum_j w_j z_q z_q', z_q = (-1)^{b_q}, of
// w_j = Im(conj(lambda_j) psi_j) + sum_c Im(conj(mu_c,j) dpsi_c,j) (n of the first, then the n(n-1)/2
// of the second, pairs q < q' in row order, at mom_off among the moments), and
// dL/dtheta_ct = sum_j w_j b_c z_t = (W_t - W_ct) / 2.
struct alignas(16) QPhaseStage {
  int32_t gate0, ngates;  // range in the QPhaseGate array
  int32_t coef_off;       // first coefficient alpha, beta of the stage (n + n(n-1)/2 per stage)
  int32_t mom_off;        // first moment among the phase moments
};
struct alignas(16) QPhaseGate {
  int32_t c, t, param, layer;   // control and target qubits, parameter index, sweep layer behind the stage
};
QP_HD inline constexpr int phase_pair_index(int n, int a, int b) {   // a < b
  return a * n - a * (a + 1) / 2 + (b - a - 1);
}
QP_HD inline constexpr int phase_terms(int n) { return n + n * (n - 1) / 2; }

// Fused-kernel modes.  The packed modes carry no input tangents: the four statevector slots of a
// thread group hold four consecutive points (forward: outputs only; VJP: output seeds only, the
// adjoint slots holding each point's lambda), so a point costs a quarter of a tangent-carrying one.
// kModeTotal: the Maxwell step of the paper's total loss over the collocation points (residual,
// energy and symmetry seeds formed in the kernel; the mirror images' outputs come from memory).
// kModeFieldsPk: the packed forward of the total loss's mirror and initial-condition points.
enum Mode : int { kModeFwd = 0, kModeMaxwell = 1, kModeVjp = 2, kModeFwdPk = 3, kModeVjpPk = 4, kModeTotal = 5, kModeFieldsPk = 6 };
QP_HD inline constexpr bool mode_packed(int mode) { return mode == kModeFwdPk || mode == kModeVjpPk || mode == kModeFieldsPk; }
QP_HD inline constexpr bool mode_fwd_only(int mode) { return mode == kModeFwd || mode == kModeFwdPk || mode == kModeFieldsPk; }
// Waves per SIMD of the forward-only kernels: half the statevectors of an adjoint, so more waves fit.  2^24
// amplitudes, 4 layers, us at 2, 3 and 4 waves: states of 3 qubits 164, 134, 126; 4: 182, 151, 146; 5: 209, 174, 167;
// 6: 227, 187, 180; 7: 264, 209, 199; 8: 288, 238, 229; 9: 321, 283, 269.  Outputs alone (at 128 registers they
// spill 11 to 37, at 168 none): 3 qubits 71, 64, 63; 4: 64, 54, 53; 5: 64, 53, 62; 6: 66, 54, 58; 7: 73, 59, 60; 8:
// 78, 64, 65; 9: 89, 72, 76.  That is 2048 tiles, three generations at three waves and two at four; over 8 to 4000
// tiles and 1 to 10 layers three waves take 0.66 to 0.97 of the time of four at 5 qubits, but up to 1.07 at 6, 1.10
// at 7, 1.17 at 8 (900 tiles, 1 layer: 19.1 us at four, 22.4 at three) and 1.09 at 9, where the tiles fill a
// generation of four waves and spill over one of three.  By rounds, within a total loss of 2^23 amplitudes: 3 qubits
// 249, 236, 240; 4: 250, 238, 254; 5: 246, 238, 266; 6: 254, 247, 267; 7: 298, 283, 302; 8: 306, 293, 301; 9: 343,
// 327, 342; over 500 to 4000 tiles three waves take 0.87 to 1.00 of the time of four from 4 qubits on, at 3 up to
// 1.02.  10 and 11 qubits, states: 395 and 409 at 2 waves with 4 exchange planes, 419 and 429 with 2, 348 and 357 at
// 3 waves; outputs alone 103 and 108, 112 and 114, 88 and 90.  At 12 qubits a workgroup is 2 waves per SIMD, and two
// of them leave 128 registers, where the kernel spills 200.
QP_HD inline constexpr int fwd_waves(int n, int exs, int mode) {
  if (n >= 10) return n < 12 && exs == 2 ? 3 : 2;
  return (mode == kModeFieldsPk && n >= 4) || (mode == kModeFwdPk && n == 5) ? 3 : 4;
}
// Modes whose results enter an FP64 loss: their forward runs the rounds.
QP_HD inline constexpr bool mode_rounds(int mode) { return mode == kModeMaxwell || mode == kModeTotal || mode == kModeFieldsPk; }

// Dense 2^5 blocks (MFMA path): a contiguous run of gates acting on at most five qubits.
constexpr int kDenseK = 5;
struct alignas(16) QDenseGate {
  int32_t kind, lq0, lq1, param;   // local qubit bits inside the block (0..4)
};
struct alignas(16) QDenseGroup {
  int32_t pos[kDenseK];   // logical index-bit position of block bit i
  int32_t gate0, ngates;  // range in the QDenseGate array
  int32_t pad;
};

// Plan header uploaded to the device (followed by the arrays at the given byte offsets).
struct alignas(16) QPlanDev {
  int32_t n, n_params, n_out, n_fused, n_rounds;
  int32_t enc_kind, enc_gate, enc_scale, n_feat;
  int32_t coord_of_qubit[16];
  uint32_t zmask[kMaxOut];          // readout parity mask of output i (trailing entangler folded)
  int32_t off_rounds;               // QRound[n_rounds]
  int32_t off_xf;                   // QXchg[n_rounds]  forward exchange before round k (k>=1)
  int32_t off_xb;                   // QXchg[n_rounds]  inverse exchange after round k (k>=1); qp_plan_image only
  int32_t off_fused;                // QFused[n_fused]
  int32_t off_csr_ptr;              // int32[n_params+1]
  int32_t off_csr_idx;              // int32[nnz]: fused*4 + component
  int32_t off_rff_B;                // float[F][3]
  int32_t off_rff_W;                // float[n][2F]
  int32_t bytes;
  int32_t n_dgroups;                // dense groups (0: no dense plan)
  int32_t off_dgroups;              // QDenseGroup[n_dgroups]
  int32_t off_dgates;               // QDenseGate[...]
  int32_t n_docc;                   // parametrised gates inside dense groups
  int32_t off_docc;                 // int32[n_docc][2]: group, gate index
  int32_t off_dcsr_ptr;             // int32[n_params+1] over the occurrences
  int32_t off_dcsr_idx;             // int32[n_docc]
  uint32_t zplain[kMaxOut];         // readout parity mask of output i without folding
  int32_t n_head;                   // leading rounds folded into the encoding (rounds 0 .. n_head-1; < n_rounds)
  int32_t head_gate[16];            // per qubit: fused gate of the leading stage, -1 if none
  int32_t off_lanes;                // QLane[2][n_rounds][2^(n-3)]: forward (0) and reverse (1) exchanges (the kernels' image: forward only)
  int32_t n_phase;                  // phase stages (CRZ runs)
  int32_t off_phase;                // QPhaseStage[n_phase]
  int32_t off_phase_gates;          // QPhaseGate[...]
  int32_t n_phase_coef;             // coefficients of the phase stages (n_phase * phase_terms(n))
  int32_t n_moments;                // phase moments accumulated by the adjoint (same count)
  int32_t off_pcsr_ptr;             // int32[n_params+1]: parameter -> CRZ occurrences
  int32_t off_pcsr_idx;             // int32[...]: phase-gate index
  int32_t n_sweeps;                 // sweep layers, the folded opening layer included
  int32_t sweep_first;              // 1: layer 0 is the opening layer folded into the encoding
  int32_t off_sweeps;               // QSweep[n_sweeps]
  int32_t off_slanes;               // QSweepLane[n_sweeps][2^(n-3)]
  int32_t off_terms;                // uint32[][2]: CZ terms of the sweep layers
  int32_t hgate[16];                // per qubit: gate of the folded opening layer, -1 if none
  int32_t etpos[16];                // mapping in which the product state is formed
  int32_t ftpos[16];                // mapping at the readout
  int32_t gtpos[16];                // mapping at the end of the adjoint
  int32_t off_turn;                 // QTurn
  int32_t off_tlanes;               // uint32[2^(n-3)][2]
  int32_t thin;                     // 1: layers leave positions out (kernels of their own)
};

}  // namespace qp

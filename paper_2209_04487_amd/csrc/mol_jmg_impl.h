// The molecular step in the rotational basis |j, m>, 2 <= j_max <= 5, with
// all three field components: one workgroup per molecule, (j_max + 1)^2
// lines per electronic state.  The coupling is the exact exponential on the
// truncated basis, applied as a rotation of the (g, e) parts of pairs of
// eigenvectors of the direction cosine along the field (the construction is
// described at jmg_couple, the tables in mol_jmg.h).
//
// Work decomposition: the line layout and the kinetic half-steps are those
// of the m = 0 step (R2 lanes per line, R1 values per lane, in-wave
// four-step FFT).  The lines, times e^{i m alpha}, go through LDS in SP rounds of
// radial points; in each round the coupling replaces them by their increments
// (matrix cores), and every lane adds those, times e^{-i m alpha}, to the values it
// kept in registers (the increment form: rounding errors scale with the change,
// not with psi).
//
// What bounds it: the latency of the phases of a molecule in a row, with one
// workgroup per CU at j_max >= 4 (registers).  At n_r = 256, j_max = 5, complex64,
// of 49 us per molecule and CU the transforms take 12, the dipole 7, the coupling
// about 8 and the wavepacket's loads and stores 8 (30,000 molecules: 8.85 GB, 1.8 ms
// at a copy's rate).
#pragma once

#include "mol_impl.h"
#include "mol_jmg.h"

namespace msqd {

// Even and odd states of the basis and the pairs of eigenvectors (see below):
// NE states with even j, NO with odd j, P pairs.  A set of up to 16 rows takes
// steps(n) K instructions; row 4 i + kk belongs to lane group kk, element i (the
// four rows that an instruction reads are neighbouring lines, on distinct banks).
// The odd states of j_max = 5 (21) take a second set of rows.
template <int JM>
struct JmgPairs {
  static constexpr int count(int parity) {
    int n = 0;
    for (int j = parity; j <= JM; j += 2) n += 2 * j + 1;
    return n;
  }
  static constexpr int pairs_of(int a) { return (JM + 1 - a) / 2; }   // of the block |m'| = a
  static constexpr int count_pairs() {
    int n = pairs_of(0);
    for (int a = 1; a <= JM; ++a) n += 2 * pairs_of(a);
    return n;
  }
  static constexpr int steps(int n) { return (n + 3) / 4; }
  static constexpr int NE = count(0), NO = count(1), P = count_pairs();
  static constexpr int NO1 = NO < 16 ? NO : 16, NO2 = NO - NO1;
  static constexpr int SE = steps(NE), S1 = steps(NO1), S2 = steps(NO2), SP = steps(P);
  static constexpr int PST = P | 1;   // row stride of W in LDS
  static_assert(NE <= 16 && NO2 <= 16 && P <= 16, "rows of one matrix-core tile");
  // The state j^2 + m + j of row r of the even or the odd states, and its j
  __device__ static __forceinline__ int even_j(int r) { return r < 1 ? 0 : (r < 6 ? 2 : 4); }
  __device__ static __forceinline__ int even_b(int r) { return r < 1 ? 0 : (r < 6 ? r + 3 : r + 10); }
  __device__ static __forceinline__ int odd_j(int r) { return r < 3 ? 1 : (r < 10 ? 3 : 5); }
  __device__ static __forceinline__ int odd_b(int r) { return r < 3 ? r + 1 : (r < 10 ? r + 6 : r + 15); }
};

// LDS of the per-molecule coupling tables: the phases e^{i m alpha}; W and the
// scaled nodes; and the workgroup reduction scratch.
template <typename T, int JM>
struct JmgTabShape {
  static constexpr size_t a16(size_t b) { return (b + 15) / 16 * 16; }
  static constexpr JmgTab tab = jmg_tab(JM);
  typedef JmgPairs<JM> PR;
  static constexpr int n_w = (PR::NE + PR::NO) * PR::PST;
  static constexpr size_t ph_bytes = a16(sizeof(cx<T>) * (2 * JM + 1));
  static constexpr size_t mt_bytes = a16(sizeof(T) * static_cast<size_t>(n_w + 16));
  static constexpr size_t red_bytes = 6 * 16 * sizeof(double);
  static constexpr size_t bytes = ph_bytes + mt_bytes + red_bytes;
};

// Wide lines (mol_impl.h) at n_r = 256 in complex64: us per step, 8 lanes per line /
// 16: j_max = 4, 30,000 molecules 4523 / 3850, three steps 9369 / 7985; j_max = 3 1831 /
// 1729, 4332 / 3879, 100 molecules 35.7 / 27.9.  At j_max = 2 the five wavefronts of a
// workgroup leave a CU room for two (40,000: 1721 / 2010), at j_max = 5 they would need
// 1,152 threads.
template <typename T, int NR, int JM>
constexpr int jmg_wide() { return wide_lines<T, NR>() && (JM == 3 || JM == 4) ? 2 : 1; }

// Radial rounds of the line exchange.  Complex64 workgroups for j_max >= 4
// hold one molecule per CU whatever their LDS (their registers exclude a
// second), so they exchange all radial points in one round when the LDS
// allows it: half the barriers per step and twice the tasks per stage.  The
// others use the rounds of the m = 0 step, which keep the LDS of a
// workgroup small enough for several per CU.
template <typename T, int NR, int JM>
struct JmgSplit {
  static constexpr int W = jmg_wide<T, NR, JM>(), R2 = FftShape<NR, T, W>::R2, L = 2 * (JM + 1) * (JM + 1);
  static constexpr size_t one_round = StagedTables<NR, T, true, false, W>::bytes +
                                      JmgTabShape<T, JM>::a16(sizeof(cx<T>) * static_cast<size_t>(lds_line_start(
                                                                                   L, NR + R2, sizeof(cx<T>)))) +
                                      JmgTabShape<T, JM>::bytes;
  static constexpr int value = (sizeof(T) == 4 && JM >= 4 && one_round <= 160 * 1024) ? 1 : fwd_split<NR, T, W>();
};

template <typename T, int NR, int JM>
struct JmgShape : JmgTabShape<T, JM> {
  typedef JmgTabShape<T, JM> TS;
  static constexpr int W = jmg_wide<T, NR, JM>();
  static constexpr int R1 = FftShape<NR, T, W>::R1, R2 = FftShape<NR, T, W>::R2;
  static constexpr int NB = (JM + 1) * (JM + 1), L = 2 * NB, threads = L * R2;
  static constexpr int SP = JmgSplit<T, NR, JM>::value, NRH = NR / SP;
  static constexpr int LS = NRH + R2;   // line stride (elements) of the LDS rows
  typedef StagedTables<NR, T, true, false, W> TBL;
  static constexpr size_t rows_bytes =
      TS::a16(sizeof(cx<T>) * static_cast<size_t>(lds_line_start(L, LS, sizeof(cx<T>))));
  static constexpr size_t bytes = TBL::bytes + rows_bytes + TS::bytes;
  static constexpr bool fits = threads <= 1024 && bytes <= 160 * 1024;
};

// Start (elements) of line `line` in the LDS rows.
template <typename T, int NR, int JM>
__device__ __forceinline__ int jmg_row(int line) {
  return lds_line_start(line, JmgShape<T, NR, JM>::LS, static_cast<int>(sizeof(cx<T>)));
}

// ------------------------------------------------------------- coupling
// The coupling's increments in LDS, in place: psi_b -> sum over the pairs p of
// W_bp dchi_p, both states, all radial points of a round.
//
// In the field frame cos(theta) only joins states of neighbouring j, so that its
// eigenvalues come in pairs +-x (or are zero, with no increment) and the two
// eigenvectors of a pair share their even-j part and, but for the sign, their
// odd-j part.  With W_bp = sqrt(2) d^j_{m m'}(beta) Q^{|m'|}_{j k} (p: m' and an
// eigenvalue x_k > 0) and u_b = e^{i m alpha} psi_b, the coupling acts on
//   a_p = sum_{even b} W_bp u_b and b_p = sum_{odd b} W_bp u_b
// of the two electronic states s, s' as
//   da_s = -vers a_s + i sin b_s',   db_s' = -vers b_s' + i sin a_s,
// vers = 1 - cos, of the angle mu12 dt |E| x_p: 15 angles and 15 x 36
// coefficients at j_max = 5 for 36 states, where the rotation to the field frame
// and the transforms of every m' block take 34 angles and 286 + 144, in three
// stages with a barrier after each.  One step, those stages on the vector units ->
// this, complex64: 7.18 -> 6.00 ms (30,000 molecules, n_r = 256, j_max = 5), 5.91 ->
// 4.69 (j_max = 4), 1.91 -> 1.84 (j_max = 3), 1.83 -> 1.83 (40,000, j_max = 2), 3.78
// -> 3.23 (30,000, n_r = 128, j_max = 5), 2.28 -> 1.92 (10,000, n_r = 512, j_max =
// 3); three steps at n_r = 256, j_max = 3: 6.08 -> 4.40.  complex128: 2.00 -> 1.47
// (10,000, n_r = 256, j_max = 3), 1.61 -> 1.04 (j_max = 2), 1.95 -> 1.30 (n_r = 128,
// j_max = 4), 2.94 -> 2.81 (j_max = 5), 2.88 -> 1.90 (20,000, n_r = 64, j_max = 5)
// (with JmgOcc's bound 1.24, 0.98, 1.10, 2.73, 1.78).
//
// A task is 16 radial points with the even states of one electronic state and the
// odd states of the other; its four products are chains of 16x16x4 matrix-core
// instructions whose output rows are the next one's operand rows (MfmaK4), so
// nothing passes between lanes.  (a re, b im) and (a im, b re) are taken in turn.
// Every task reads and writes its own elements only.
template <typename T>
__device__ __forceinline__ int jmg_slot_row(int slot, int S) {
  // the row whose product comes out in row `slot` of a tile; -1: none
  const int kk = sizeof(T) == 4 ? slot >> 2 : slot & 3, i = sizeof(T) == 4 ? slot & 3 : slot >> 2;
  return i < S ? 4 * i + kk : -1;
}

// A lane's part of the coupling in every task: its states' LDS rows (of the two
// electronic states, 16 bits each), the operands of
// W^T (fw: row = pair, K = state) and of W (row = state, K = pair), its pairs' nodes.
template <typename T, int NR, int JM>
struct JmgOps {
  typedef JmgPairs<JM> PR;
  static constexpr int SE = PR::SE, S1 = PR::S1, S2 = PR::S2, SP = PR::SP, NI = SE + S1 + S2;
  unsigned row[NI];
  bool in[NI];   // whether there is such a state
  T fw[NI], be[SP], bo[SP], b2[SP], xk[4];

  __device__ __forceinline__ JmgOps(const T* W, const T* xe) {
    constexpr int NE = PR::NE, NO1 = PR::NO1, NO = PR::NO, P = PR::P, PST = PR::PST;
    const int lane = fresh_lane();
    const int col = lane & 15, kk = lane >> 4;
    const int pr = jmg_slot_row<T>(col, SP);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bool even = i < SE;
      int r = even ? 4 * i + kk : (i < SE + S1 ? 4 * (i - SE) + kk : NO1 + 4 * (i - SE - S1) + kk);
      in[i] = r < (even ? NE : (i < SE + S1 ? NO1 : NO));
      r = in[i] ? r : 0;   // W is zero for the rows past the last; any state will do
      const int b = even ? PR::even_b(r) : PR::odd_b(r);
      static_assert(JmgShape<T, NR, JM>::rows_bytes / sizeof(cx<T>) < 65536, "16-bit rows");
      row[i] = jmg_row<T, NR, JM>(b) | jmg_row<T, NR, JM>(JmgShape<T, NR, JM>::NB + b) << 16;
      const bool ok = in[i] && pr >= 0 && pr < P;
      const T w = W[ok ? (even ? r : NE + r) * PST + pr : 0];
      fw[i] = ok ? w : T(0);
    }
    const int re = jmg_slot_row<T>(col, SE), r1 = jmg_slot_row<T>(col, S1), r2 = jmg_slot_row<T>(col, S2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = 4 * i + kk;
      const bool ok = i < SP && p < P;
      xk[i] = ok ? xe[p] : T(0);
      if (i < SP) {
        const bool oke = ok && re >= 0 && re < NE, ok1 = ok && r1 >= 0 && r1 < NO1;
        const bool ok2 = S2 > 0 && ok && r2 >= 0 && NO1 + r2 < NO;
        const T we = W[oke ? re * PST + p : 0], w1 = W[ok1 ? (NE + r1) * PST + p : 0];
        be[i < SP ? i : 0] = oke ? we : T(0);
        bo[i < SP ? i : 0] = ok1 ? w1 : T(0);
        if constexpr (S2 > 0) {
          const T w2 = W[ok2 ? (NE + NO1 + r2) * PST + p : 0];
          b2[i < SP ? i : 0] = ok2 ? w2 : T(0);
        }
      }
    }
  }
};

// Run task(t), t < nt, on the workgroup's whole wavefronts.  Workgroups of more than
// four wavefronts put more of them on some execution units than on others, and with a
// fixed share of the tasks those would set the pace: their wavefronts take the next
// task from an LDS counter (zero on entry).  The tasks' outputs are their own.
template <typename T, int NR, int JM, typename F>
__device__ __forceinline__ void jmg_tasks(int nt, int* ctr, F&& task) {
  constexpr int NW = JmgShape<T, NR, JM>::threads / 64;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  if (wave >= NW) return;
  if constexpr (NW > 4) {
    for (;;) {
      int t = 0;
      if (fresh_lane() == 0) t = atomicAdd(ctr, 1);
      t = __builtin_amdgcn_readfirstlane(t);
      if (t >= nt) break;
      task(t);
    }
  } else {
#pragma unroll 1
    for (int t = wave; t < nt; t += NW) task(t);
  }
}

template <typename T, int NR, int JM>
__device__ __forceinline__ void jmg_couple(cx<T>* sh, const JmgOps<T, NR, JM>& o, const T* mudt_h, int* ctr) {
  typedef JmgShape<T, NR, JM> S;
  typedef JmgOps<T, NR, JM> O;
  typedef MfmaK4<T> MK;
  typedef typename MK::acc acc_t;
  constexpr int SE = O::SE, S1 = O::S1, S2 = O::S2, SP = O::SP, NI = O::NI;
  constexpr int NT = 2 * S::NRH / 16;   // tasks
  const int col = fresh_lane() & 15;
  const acc_t z = {T(0), T(0), T(0), T(0)};
  auto task = [&](int t) {
    const int s = t & 1, rl = (t >> 1) * 16 + col;
    T sn[4], vs[4];
    sin_vers_tile<NR>(mudt_h[rl], o.xk, sn, vs);
    T* at[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
      at[i] = reinterpret_cast<T*>(sh + ((o.row[i] >> (((i < SE) == (s == 0)) ? 0 : 16)) & 0xffffu) + rl);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      // c = 0: (a re, b im); c = 1: (a im, b re)
      acc_t A = z, B = z;
#pragma unroll
      for (int i = 0; i < SE; ++i) A = MK::mma(o.fw[i], at[i][c], A);
#pragma unroll
      for (int i = SE; i < NI; ++i) B = MK::mma(o.fw[i], at[i][1 - c], B);
      if constexpr (sizeof(T) == 8) MK::settle(A, B);
#pragma unroll
      for (int i = 0; i < SP; ++i) {
        const T sg = c == 0 ? sn[i] : -sn[i];
        const T a = A[i], b = B[i];
        A[i] = -vs[i] * a - sg * b;
        B[i] = -vs[i] * b + sg * a;
      }
      acc_t oe = z, o1 = z, o2 = z;
#pragma unroll
      for (int i = 0; i < SP; ++i) {
        oe = MK::mma(o.be[i], A[i], oe);
        o1 = MK::mma(o.bo[i], B[i], o1);
        if constexpr (S2 > 0) o2 = MK::mma(o.b2[i], B[i], o2);
      }
      if constexpr (sizeof(T) == 8) {
        MK::settle(oe, o1);
        if constexpr (S2 > 0) MK::settle(o2, o2);
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (o.in[i]) at[i][i < SE ? c : 1 - c] = i < SE ? oe[i & 3] : (i < SE + S1 ? o1[(i - SE) & 3] : o2[(i - SE - S1) & 3]);
    }
  };
  jmg_tasks<T, NR, JM>(NT, ctr, task);
}

// The terms of the dipole vector at radial point rl from the basis states of
// one j (FP64): Re<g|D_z|e>, and P = <g|D_+|e>, P' = <e|D_+|g> with
// D_+ = D_x + i D_y, from which Re<g|D_x|e> = (Re P + Re P') / 2 and
// Re<g|D_y|e> = (Im P + Im P') / 2.  Summed over j they give the dipole.
template <typename T, int NR, int JM>
__device__ __forceinline__ void jmg_dipole_point(const cx<T>* sh, const double* dip, int j, int rl, double* tx,
                                                 double* ty, double* tz) {
  constexpr int NB = (JM + 1) * (JM + 1);
  auto ld = [&](int line) {
    const cx<T> v = sh[jmg_row<T, NR, JM>(line) + rl];
    return cx<double>{static_cast<double>(v.x), static_cast<double>(v.y)};
  };
  double z = 0.0, pr = 0.0, pi = 0.0;
  constexpr int kUnroll = sizeof(T) == 4 ? 2 : 1;   // complex128 spilled with two
#pragma unroll kUnroll
  for (int m = -j; m <= j; ++m) {
    const int b = j * j + m + j;
    const cx<double> gb = ld(b), eb = ld(NB + b);
    if (j < JM) {
      const int bz = (j + 1) * (j + 1) + m + j + 1;        // (j+1, m)
      const int bp = bz + 1;                               // (j+1, m+1)
      const cx<double> gz = ld(bz), ez = ld(NB + bz);
      z += dip[3 * b] * ((gz.x * eb.x + gz.y * eb.y) + (gb.x * ez.x + gb.y * ez.y));
      const cx<double> gp = ld(bp), ep = ld(NB + bp);
      const double c = dip[3 * b + 1];
      // conj(g_p) e_b + conj(e_p) g_b
      pr += c * ((gp.x * eb.x + gp.y * eb.y) + (ep.x * gb.x + ep.y * gb.y));
      pi += c * ((gp.x * eb.y - gp.y * eb.x) + (ep.x * gb.y - ep.y * gb.x));
    }
    if (m + 1 <= j - 1) {
      const int bm = (j - 1) * (j - 1) + m + 1 + j - 1;    // (j-1, m+1)
      const cx<double> gm = ld(bm), em = ld(NB + bm);
      const double c = dip[3 * b + 2];
      pr += c * ((gm.x * eb.x + gm.y * eb.y) + (em.x * gb.x + em.y * gb.y));
      pi += c * ((gm.x * eb.y - gm.y * eb.x) + (em.x * gb.y - em.y * gb.x));
    }
  }
  *tx = 0.5 * pr;
  *ty = 0.5 * pi;
  *tz = z;
}

// ---------------------------------------------------------------- kernel
// Waves per SIMD the register allocation targets (complex64): three where
// that fits more workgroups on a CU than two does (a seven-wave workgroup gets one
// per CU either way, so it keeps two waves per SIMD and the registers that come with
// them); four with wide lines.
template <typename T, int NR, int JM>
struct JmgOcc {
  static constexpr int wg_waves = (JmgShape<T, NR, JM>::threads + 63) / 64;
  static constexpr int waves =
      sizeof(T) == 8 ? (NR >= 128 ? 2 : 1) : (jmg_wide<T, NR, JM>() > 1 ? 4 : ((12 / wg_waves) > (8 / wg_waves) ? 3 : 2));
  // The bound from above: complex128 from n_r = 128 on and complex64 from n_r = 256 on
  // are told that more will not do, or the scheduler spreads the phase table's loads
  // out to keep registers free (complex128, n_r = 128, j_max = 3, 10,000 molecules: 829
  // -> 530 us; complex64, n_r = 256, j_max = 2, 40,000: 1685 -> 1630, j_max = 5, 30,000:
  // 5655 -> 5622, n_r = 512, j_max = 3, 10,000: 1872 -> 1813).  On smaller grids
  // aiming at more is right (complex64, n_r = 128, j_max = 3, 50,000: 1407 / 1618 us;
  // n_r = 64, j_max = 2, 60,000: 624 / 789).
  static constexpr int most = sizeof(T) == 8 ? (NR >= 128 ? 2 : 8) : (NR >= 256 ? waves : 8);
};

template <typename T, int NR, int JM, bool ONE>
__global__ __launch_bounds__((JmgShape<T, NR, JM>::threads)) __attribute__((amdgpu_waves_per_eu(JmgOcc<T, NR, JM>::waves, JmgOcc<T, NR, JM>::most)))
void mol_jmg_kernel(MolArgs a) {
  typedef JmgShape<T, NR, JM> S;
  constexpr int R1 = S::R1, R2 = S::R2, NB = S::NB, SP = S::SP, PH = R1 / SP, NRH = S::NRH;
  constexpr JmgTab TB = S::tab;
  typedef typename S::TBL TBL;
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* kin_s = reinterpret_cast<cx<T>*>(smem);
  cx<T>* tw_s = kin_s + NR;
  T* mask_s = reinterpret_cast<T*>(tw_s + TBL::tw_elems);
  cx<T>* sh = reinterpret_cast<cx<T>*>(smem + TBL::bytes);
  cx<T>* ph = reinterpret_cast<cx<T>*>(smem + TBL::bytes + S::rows_bytes);
  T* W = reinterpret_cast<T*>(smem + TBL::bytes + S::rows_bytes + S::ph_bytes);
  T* xe = W + S::n_w;
  double* red = reinterpret_cast<double*>(smem + TBL::bytes + S::rows_bytes + S::ph_bytes + S::mt_bytes);
  // the coupling's task counter lives in the reduction area, which is used
  // only after the last round
  int* ctr = reinterpret_cast<int*>(red);

  const int mol = blockIdx.x;
  const int tid = threadIdx.x;
  constexpr int nthr = S::threads;
  const int line = tid / R2;
  const int q = tid - line * R2;
  const int st = line / NB, b = line - st * NB;
  int jl = 0;
  while ((jl + 1) * (jl + 1) <= b) ++jl;

  const char* ws = a.ws;
  const bool dbl = sizeof(T) == 8;
  const cx<T>* kin_g = reinterpret_cast<const cx<T>*>(ws + (dbl ? a.lay.kin_d : a.lay.kin_f));
  const cx<T>* tw_g = reinterpret_cast<const cx<T>*>(ws + (dbl ? a.lay.tw_d : tw_scaled<NR, T>() ? a.lay.tw_fs : a.lay.tw_f));
  const cx<T>* vph_g = reinterpret_cast<const cx<T>*>(ws + (dbl ? a.lay.vph_d : a.lay.vph_f));
  const T* mudt = reinterpret_cast<const T*>(ws + (dbl ? a.lay.mudt_d : a.lay.mudt_f));
  const T* mask_g = reinterpret_cast<const T*>(ws + (dbl ? a.lay.mask_d : a.lay.mask_f));
  const double* mu = reinterpret_cast<const double*>(ws + a.lay.mu_d);
  const double* tg = reinterpret_cast<const double*>(ws + a.lay.total);

  // the coupling's host tables, one entry per thread, ahead of the wavepacket's
  // loads: what is formed from them is formed while those are in flight
  constexpr int NTAB = TB.n_jx + TB.n_q + TB.n_x;
  static_assert(NTAB <= nthr && TB.jx == 0 && TB.q == TB.n_jx && TB.x == TB.n_jx + TB.n_q, "one entry per thread");
  const double tab_e = tg[tid < NTAB ? tid : 0];

  // field at the molecule (each component at its own edge of the cell)
  double E3[3];
  if (a.Ex != nullptr) {
    const int c = a.cell_of_mol[mol];
    const void* f3[3] = {a.Ex, a.Ey, a.Ez};
#pragma unroll
    for (int k = 0; k < 3; ++k)
      E3[k] = (a.ex_is_float ? static_cast<double>(static_cast<const float*>(f3[k])[c])
                             : static_cast<const double*>(f3[k])[c]) * a.inv_eau;
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) E3[k] = a.E_mol[3 * mol + k];
  }
  if (a.E_out != nullptr && tid == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a.E_out[3 * mol + k] = E3[k];
  }

  cx<T>* psi = reinterpret_cast<cx<T>*>(a.psi) + static_cast<size_t>(mol) * S::L * NR;
  cx<T>* slot = sh + jmg_row<T, NR, JM>(line);
  const int loff = line * NR + q;
  const int voff = (st * a.nj + jl) * NR + q;   // potential phases depend on (state, j)
  cx<T> vv[R1];
  if constexpr (stage_tables<NR, T>()) stage_tables_to_lds<NR, T, true, S::W>(kin_s, tw_s, mask_s, kin_g, tw_g, mask_g);
  // The wavepacket's loads: ahead of the coupling tables' arithmetic, which other
  // workgroups' loads would otherwise wait behind; after it for the complex64 forms
  // of one exchange round (ms, after / ahead: n_r = 256, j_max = 3, 30,000 molecules 1.72 /
  // 1.86; n_r = 64, j_max = 2, 60,000 0.62 / 0.71, j_max = 5, 20,000 1.39 / 1.41; n_r =
  // 128, j_max = 5, 20,000 2.12 / 2.15; n_r = 256, j_max = 4 and 5, 30,000 within 2%:
  // 3.75 / 3.69, 5.65 / 5.61).
  constexpr bool LATE = sizeof(T) == 4 && SP == 1;
  if constexpr (!LATE) {
#pragma unroll
    for (int p = 0; p < R1; ++p) vv[p] = psi[loff + R2 * p];
  }

  // per-molecule coupling tables: the field frame (alpha, beta) and |E|; the LDS
  // rows, which are not in use yet, hold the host tables and d^j(beta)
  {
    double* tl = reinterpret_cast<double*>(sh);
    double* dj = tl + NTAB;
    static_assert((NTAB + TB.n_jx) * sizeof(double) <= S::rows_bytes, "scratch in the rows");
    if (tid < NTAB) tl[tid] = tab_e;
    const double en = sqrt(E3[0] * E3[0] + E3[1] * E3[1] + E3[2] * E3[2]);
    const double rho = sqrt(E3[0] * E3[0] + E3[1] * E3[1]);
    const double ca = rho > 0.0 ? E3[0] / rho : 1.0, sa = rho > 0.0 ? E3[1] / rho : 0.0;
    const double cb = en > 0.0 ? E3[2] / en : 1.0, sb = en > 0.0 ? rho / en : 0.0;
    if (tid < 2 * JM + 1) {
      const int m = tid - JM, am = m < 0 ? -m : m;
      double px = 1.0, py = 0.0;
      for (int k = 0; k < am; ++k) {
        const double nx = px * ca - py * sa;
        py = px * sa + py * ca;
        px = nx;
      }
      ph[tid] = {static_cast<T>(px), static_cast<T>(m < 0 ? -py : py)};
    }
    // d^j_{m m'}(beta) = sum_k O_{m k} O_{m' k} cos(pi/2 (m' - m) - beta mu_k),
    // mu_k = k - j: ra, rc are the rows of m and m' in O
    auto wigner_d = [&](int j, int ra, int rc) {
      const int n = 2 * j + 1;
      const double* O = tl + TB.jx + jmg_jx_off(j);
      // cos(pi/2 (m' - m) - beta mu) = cA cos(mu beta) + sA sin(mu beta)
      const int dq = (rc - ra) & 3;
      const double cA = dq == 0 ? 1.0 : (dq == 2 ? -1.0 : 0.0);
      const double sA = dq == 1 ? 1.0 : (dq == 3 ? -1.0 : 0.0);
      double acc = O[ra * n + j] * O[rc * n + j] * cA;
      double wc = 1.0, wsn = 0.0;   // cos(mu beta), sin(mu beta)
      for (int mu_ = 1; mu_ <= j; ++mu_) {
        const double nc = wc * cb - wsn * sb;
        wsn = wc * sb + wsn * cb;
        wc = nc;
        acc += O[ra * n + j + mu_] * O[rc * n + j + mu_] * (cA * wc + sA * wsn) +
               O[ra * n + j - mu_] * O[rc * n + j - mu_] * (cA * wc - sA * wsn);
      }
      return acc;
    };
    __syncthreads();
    for (int t = tid; t < TB.n_jx; t += nthr) {
      int j = 0;
      while (t >= jmg_jx_off(j + 1)) ++j;
      const int n = 2 * j + 1, o = t - jmg_jx_off(j), r = o / n;
      dj[t] = wigner_d(j, r, o - r * n);
    }
    __syncthreads();
    typedef JmgPairs<JM> PR;
    for (int t = tid; t < (PR::NE + PR::NO) * PR::P; t += nthr) {
      const int r = t / PR::P;
      int p = t - r * PR::P;
      const bool even = r < PR::NE;
      const int j = even ? PR::even_j(r) : PR::odd_j(r - PR::NE);
      const int b = even ? PR::even_b(r) : PR::odd_b(r - PR::NE);
      const int m = b - j * j - j;
      // pair p: m' = 0, 1, -1, 2, -2, ..., the positive eigenvalues of each in order
      const int pw = r * PR::PST + p;
      int u = 0;
      while (p >= PR::pairs_of((u + 1) >> 1)) p -= PR::pairs_of((u++ + 1) >> 1);
      const int am = (u + 1) >> 1, mp = (u & 1) ? am : -am;
      const int n = JM + 1 - am, k = (n + 1) / 2 + p;
      double w = 0.0;
      if (am <= j)
        w = 1.4142135623730950488 * dj[jmg_jx_off(j) + (m + j) * (2 * j + 1) + mp + j] *
            tl[TB.q + jmg_q_off(JM, am) + (j - am) * n + k];
      W[pw] = static_cast<T>(w);
      if (r == 0) xe[pw] = static_cast<T>(en * tl[TB.x + jmg_x_off(JM, am) + k]);
    }
  }
  if constexpr (LATE) {
#pragma unroll
    for (int p = 0; p < R1; ++p) vv[p] = psi[loff + R2 * p];
  }
  __syncthreads();

  const cx<T> eim = ph[b - jl * jl - jl + JM];   // this line's e^{i m alpha}
  double ab = 0.0;
  const int n_steps = ONE ? 1 : a.n_steps;
  for (int step = 0; step < n_steps; ++step) {
    const cx<T>* kin;
    const cx<T>* tw;
    const T* mask;
    if constexpr (stage_tables<NR, T>()) {
      kin = kin_s;
      tw = tw_s;
      mask = mask_s;
    } else {
      kin = opaque(kin_g);
      tw = opaque(tw_g);
      mask = opaque(mask_g);
    }
    const cx<T>* vph = opaque(vph_g);
    kinetic_half<T, NR, false, SP, TBL::TWC, tw_scaled<NR, T>(), S::W>(vv, slot, q, kin, tw);
    const JmgOps<T, NR, JM> ops(W, xe);
#pragma unroll
    for (int h = 0; h < SP; ++h) {
#pragma unroll
      for (int pp = 0; pp < PH; ++pp) {
        const int p = h * PH + pp;
        vv[p] = phase_mul(vv[p], vph[voff + R2 * p]);
        slot[q + R2 * pp] = cmul(eim, vv[p]);
      }
      // the previous round's coupling ended at a barrier: reset its counter
      if (tid == 0) *ctr = 0;
      __syncthreads();
      jmg_couple<T, NR, JM>(sh, ops, mudt + h * NRH, ctr);
      __syncthreads();
      vph = opaque(vph_g);   // read again rather than kept across the coupling
#pragma unroll
      for (int pp = 0; pp < PH; ++pp) {
        const int p = h * PH + pp;
        vv[p] = phase_mul(vv[p] + cmul_conj(slot[q + R2 * pp], eim), vph[voff + R2 * p]);
      }
    }
    kinetic_half<T, NR, false, SP, TBL::TWC, tw_scaled<NR, T>(), S::W>(vv, slot, q, kin, tw);
    constexpr int P0 = (3 * R1) / 4;
    if (a.kmask >= R2 * P0) {
#pragma unroll
      for (int p = P0; p < R1; ++p) absorb_point_nb(vv[p], mask[q + R2 * p], ab);
    } else {
#pragma unroll
      for (int p = 0; p < R1; ++p) absorb_point(vv[p], mask[q + R2 * p], ab);
    }
  }

  // the norm (finiteness check) and the dipole vector, in the same rounds of radial
  // points
  double nrm = 0.0;
#pragma unroll
  for (int p = 0; p < R1; ++p) nrm += static_cast<double>(norm2(vv[p]));
  double dc[3] = {0.0, 0.0, 0.0};
  if (a.want_d && a.d_mol) {
    const double* dip = tg + TB.dip;
#pragma unroll
    for (int h = 0; h < SP; ++h) {
      __syncthreads();   // the previous users of the slots are done
#pragma unroll
      for (int pp = 0; pp < PH; ++pp) slot[q + R2 * pp] = vv[h * PH + pp];
      __syncthreads();
      // Tasks of one j and 64 radial points, the heaviest first (j = JM has terms with
      // j - 1 only), given out to and fro over the whole wavefronts: fixed, so that the
      // sums are the same in every run.  With two or more wavefronts for each 64 points,
      // an equal number of them, which the execution units share alike (9 wavefronts
      // -> 8 at j_max = 5; 6.04 -> 5.70 ms for 30,000 molecules at n_r = 256).
      constexpr int NC = NRH / 64, NW = nthr / 64, NWD = NW >= 2 * NC ? NW / NC * NC : NW;
      const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      for (int pass = 0; pass * NWD < NC * (JM + 1); ++pass) {
        const int t = pass * NWD + ((pass & 1) ? NWD - 1 - wave : wave);
        if (wave >= NWD || t >= NC * (JM + 1)) continue;
        constexpr int top = (JM + 1) / 2;   // tasks with a larger sum than j = JM's
        const int u = t / NC, rl = (t - u * NC) * 64 + (tid & 63);
        const int j = u == top ? JM : JM - 1 - u + (u > top ? 1 : 0);
        double tx, ty, tz;
        jmg_dipole_point<T, NR, JM>(sh, dip, j, rl, &tx, &ty, &tz);
        const double m = mu[h * NRH + rl];
        dc[0] += m * tx;
        dc[1] += m * ty;
        dc[2] += m * tz;
      }
    }
  }
  // workgroup sums of (ab, nrm, dx, dy, dz) in a fixed order
  double vals[5] = {ab, nrm, dc[0], dc[1], dc[2]};
  const int lane = tid & 63, wid = tid >> 6;
  constexpr int nw = (nthr + 63) >> 6;
#pragma unroll
  for (int k = 0; k < 5; ++k) vals[k] = wave_sum(vals[k]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 5; ++k) red[wid * 5 + k] = vals[k];
  }
  __syncthreads();
  if (tid == 0) {
    double sm[5];
    for (int k = 0; k < 5; ++k) {
      double t = 0.0;
      for (int w = 0; w < nw; ++w) t += red[w * 5 + k];
      sm[k] = t;
    }
    const double dr = a.dr;
    const double absorbed = a.absorbed[mol] + sm[0] * dr;
    a.absorbed[mol] = absorbed;
    if (a.want_d && a.d_mol) {
      for (int k = 0; k < 3; ++k) a.d_mol[3 * mol + k] = 2.0 * dr * sm[2 + k];
    }
    if (!isfinite(sm[1]) || !isfinite(sm[2]) || !isfinite(sm[3]) || !isfinite(sm[4]) || !isfinite(absorbed))
      atomicOr(a.status, 1);
  }
#pragma unroll
  for (int p = 0; p < R1; ++p) psi[loff + R2 * p] = vv[p];
}

template <typename T, int NR, int JM, bool ONE>
int launch_jmg_t1(const MolArgs& a, hipStream_t s) {
  typedef JmgShape<T, NR, JM> S;
  if constexpr (!S::fits) {
    return static_cast<int>(hipErrorInvalidValue);
  } else {
    const size_t shm = S::bytes;
    if (shm > mol_lds_limit()) return static_cast<int>(hipErrorInvalidValue);
    static std::atomic<unsigned long long> lds_set{0};
    if (shm > 64 * 1024) {
      const hipError_t e = allow_large_lds(reinterpret_cast<const void*>(&mol_jmg_kernel<T, NR, JM, ONE>), lds_set);
      if (e != hipSuccess) return static_cast<int>(e);
    }
    hipLaunchKernelGGL((mol_jmg_kernel<T, NR, JM, ONE>), dim3(a.n_mol), dim3(S::threads), shm, s, a);
    return static_cast<int>(hipGetLastError());
  }
}

template <typename T, int NR, int JM>
int launch_jmg_t(const MolArgs& a, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (a.n_steps == 1) return launch_jmg_t1<T, NR, JM, true>(a, s);
  }
  return launch_jmg_t1<T, NR, JM, false>(a, s);
}

template <typename T, int JM>
int launch_jmg_nr(const MolArgs& a, int n_r, hipStream_t s) {
  switch (n_r) {
    case 64: return launch_jmg_t<T, 64, JM>(a, s);
    case 128: return launch_jmg_t<T, 128, JM>(a, s);
    case 256: return launch_jmg_t<T, 256, JM>(a, s);
    case 512: return launch_jmg_t<T, 512, JM>(a, s);
    default: return static_cast<int>(hipErrorInvalidValue);
  }
}

template <typename T>
int launch_jmg_prec(const MolArgs& a, int n_r, int jm, hipStream_t s) {
  switch (jm) {
    case 2: return launch_jmg_nr<T, 2>(a, n_r, s);
    case 3: return launch_jmg_nr<T, 3>(a, n_r, s);
    case 4: return launch_jmg_nr<T, 4>(a, n_r, s);
    case 5: return launch_jmg_nr<T, 5>(a, n_r, s);
    default: return static_cast<int>(hipErrorInvalidValue);
  }
}

template <typename T, int JM>
bool jmg_fits_nr(int n_r, size_t* lds) {
  switch (n_r) {
    case 64: *lds = JmgShape<T, 64, JM>::bytes; return JmgShape<T, 64, JM>::fits;
    case 128: *lds = JmgShape<T, 128, JM>::bytes; return JmgShape<T, 128, JM>::fits;
    case 256: *lds = JmgShape<T, 256, JM>::bytes; return JmgShape<T, 256, JM>::fits;
    case 512: *lds = JmgShape<T, 512, JM>::bytes; return JmgShape<T, 512, JM>::fits;
    default: *lds = 0; return false;
  }
}

template <typename T>
bool jmg_fits(int n_r, int jm, size_t* lds) {
  switch (jm) {
    case 2: return jmg_fits_nr<T, 2>(n_r, lds);
    case 3: return jmg_fits_nr<T, 3>(n_r, lds);
    case 4: return jmg_fits_nr<T, 4>(n_r, lds);
    case 5: return jmg_fits_nr<T, 5>(n_r, lds);
    default: *lds = 0; return false;
  }
}

}  // namespace msqd

// Precision: CT is the arithmetic of the contraction with the row tensor (FP32 on the mixed path);
// every product with a QR or SVD factor (R_{c-1} B_c, Q_c G_{c+1}) and the factorisations stay FP64,
// because those factors carry the Schmidt weights that decide the truncation.
//
// One boundary-MPS row step: apply row y to the boundary D_{y-1}, left-canonicalise with
// Householder QR, truncate right to left with one-sided Jacobi SVDs, normalise (SM S-2 eq. project;
// VMC section, cutoff chi).  The state after the step depends only on the state before it, so the
// factorisation routines here need not be LAPACK's: the QR is unblocked Householder (reflectors as
// in LAPACK's dgeqr2/dorg2r, written from their definition) and the SVD is Hestenes' one-sided
// Jacobi method with round-robin pair ordering, sorted descending afterwards.
//
// Mapping: one workgroup per sample, the whole row in one launch, instantiated for the largest
// matrices it holds (RowCfg: fused bonds up to 16, 32, 48, 72, and 128 with the matrices in global
// memory).  The working matrices live in LDS; the Q factors of the row are parked in a per-sample
// global slot between the two sweeps.  Column work inside a factorisation is spread over lane groups,
// dot products are lane-group reductions (all lanes obtain the same bits, so the result is
// deterministic).
//
// What bounds it is the latency of dependent chains (a Jacobi round, a reflector), so what matters is
// how many samples a compute unit holds: the workgroup is no larger than its column pairs and J rows
// need, its matrices no larger than the bonds, and its registers few enough for the samples that fit
// in LDS.  Z2 16 x 16, chi = 16 (1024 samples, one row): one 512-thread workgroup per CU 5.58 ms, four
// of 256 threads 2.18 ms; Z4 13 x 13, chi = 22 (301 samples): in the 72 x 72 kernel, one per CU, 3.14
// ms, in the 48 x 48 one, two per CU, 2.55 ms (before the later changes below).
#pragma once

#include <type_traits>

#include "dev_common.h"
#include "internal.h"
#include "jacobi_scalar.h"

namespace gipeps {

// Every multiply-add below is written as fma where it is one: the batch and the ragged kernel of a class must
// give the same bits, whatever the compiler would contract in each.  (Classes agree to rounding: the partial
// sums of a reflector's dot products follow the rows per lane.)
#pragma clang fp contract(off)

// Largest matrices (fused bond) of each instantiation, its threads and the waves per SIMD it is compiled
// for: the smallest workgroup that gives every column pair GW lanes and every J row two, so that as many
// samples share a compute unit as the LDS allows.
template <int MAXN>
struct RowCfg {
  static_assert(MAXN == 16 || MAXN == 32 || MAXN == 48 || MAXN == 72 || MAXN == kMaxNBig, "row classes");
  static constexpr int NT = MAXN == 16 ? 128 : MAXN == 32 ? 256 : MAXN == 48 ? 384 : 512;
  static constexpr int MINW = MAXN <= 32 ? 4 : MAXN == 48 ? 3 : 2;
};

// Lanes per column group in the Jacobi (GW, 4 or 8) is a template parameter chosen per handle up to 72 columns
// (the autotuner times both): eight measured fastest at chi*Dk = 72, where four lanes double each lane's
// dependent chains and the step is latency-bound (one or two waves per SIMD).  Eight beyond 72.

// ---------------------------------------------------------------------------------------------
// Householder QR of the m x n column-major matrix X (ld = m, in LDS), k = min(m, n) reflectors
// (H_j = I - tau_j v_j v_j^T, v_j[j] = 1, zero above j; as LAPACK's dgeqr2/dorg2r define them).
// On return R (k x n) is in sR (R[i][j] at sR[j*ldr + i], zeros below the diagonal, rows >= k
// untouched), the explicit m x k factor Q is in qdst (global, ld m), and X holds the reflectors.
//
// Column jj belongs to 8-lane group jj mod 64 for the whole factorisation and stays in its
// registers (RPL rows per lane, row = lane + 8t).  Step j: every group applies H_j (read from a
// double-buffered LDS copy of v_j) to its columns right of j; the group owning column j+1 then
// forms H_{j+1} at once from the updated column and publishes it -- one barrier per reflector, and
// per step one column is written to LDS instead of the whole trailing matrix being read and
// rewritten.  Q = H_0 ... H_{k-1} [I; 0] is then accumulated column by column in registers
// (column jj needs H_jj .. H_0 only), reading the reflectors from X, with no barrier at all.
// vbuf: 2 * MAXM doubles of LDS.  qdst may point to LDS.
// ---------------------------------------------------------------------------------------------
//
// The reflectors are taken in panels of 8, unrolled: in panel b the lanes' rows t < b (row = lane + 8 t)
// lie above every reflector, so they take no part and no row but those of t = b and b + 1 needs a test.
// (With the tests on every row, the chain from one reflector to the next held 476 instructions, 46 of
// them reloads of spilled masks; the panels halve the multiply-adds of a square matrix as well.)
template <int B, int E, class F>
__device__ __forceinline__ void unrolled(F f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    unrolled<B + 1, E>(f);
  }
}

template <int MAXM, int NMAX, int NT>
__device__ __forceinline__ void householder_qr(double* X, int m, int n, double* sR, int ldr, double* sTau,
                                               double* vbuf, double* qdst) {
  constexpr int RPL = MAXM / 8;                           // m <= MAXM
  constexpr int kGroups = NT / 8;                         // groups of 8 lanes
  constexpr int CPG = (NMAX + kGroups - 1) / kGroups;     // columns per group (n <= NMAX)
  constexpr int NPAN = NMAX / 8;                          // panels of 8 reflectors
  static_assert(MAXM % 8 == 0 && NMAX % 8 == 0 && NPAN <= RPL, "rows per lane, whole panels");
  // independent partial sums in the per-lane dot products (shorter dependent chains on the
  // reflector's critical path)
  constexpr int kAcc = RPL >= 12 ? 3 : (RPL >= 6 ? 2 : 1);
  const int g = threadIdx.x >> 3, gl = threadIdx.x & 7;
  const int k = m < n ? m : n;
  double c[CPG][RPL];
#pragma unroll
  for (int q = 0; q < CPG; ++q) {
    const int jj = g + q * kGroups;
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      const int row = gl + 8 * t;
      c[q][t] = (jj < n && row < m) ? X[(size_t)jj * m + row] : 0.0;
    }
  }
  auto add_up = [](const double (&p)[kAcc]) {
    double s = p[0];
#pragma unroll
    for (int a = 1; a < kAcc; ++a) s += p[a];
    return group8_sum(s);
  };
  // H_j (8 T0 <= j <= 8 T0 + 8) from the current column col (rows >= j): scale it into v_j in place,
  // publish v_j (rows from 8 T0) and tau_j
  auto make_reflector = [&](auto T, double (&col)[RPL], int j) {
    constexpr int T0 = T;
    double s2p[kAcc] = {}, alpha = 0.0;
#pragma unroll
    for (int t = T0; t < RPL; ++t) {
      const int row = gl + 8 * t;
      const double below = (t >= T0 + 2 || row > j) ? col[t] : 0.0;
      s2p[t % kAcc] = fma(below, below, s2p[t % kAcc]);
      if (t < T0 + 2) alpha += (row == j) ? col[t] : 0.0;
    }
    const double s2 = add_up(s2p);
    alpha = group8_sum(alpha);
    double tau = 0.0, beta = alpha, scal = 1.0;
    if (s2 != 0.0) {
      beta = -copysign(sqrt(fma(alpha, alpha, s2)), alpha);
      tau = (beta - alpha) / beta;
      scal = 1.0 / (alpha - beta);
    }
    double* v = vbuf + (j & 1) * MAXM;
#pragma unroll
    for (int t = T0; t < RPL; ++t) {
      const int row = gl + 8 * t;
      if (t >= T0 + 2) {
        col[t] *= scal;
        v[row] = col[t];
      } else {
        const double scaled = col[t] * scal;
        col[t] = row > j ? scaled : row == j ? beta : col[t];
        v[row] = row > j ? scaled : row == j ? 1.0 : 0.0;
      }
    }
    if (gl == 0) sTau[j] = tau;
  };
  if (g == 0 && k > 0) make_reflector(std::integral_constant<int, 0>{}, c[0], 0);
  __syncthreads();
  // the reflector's rows are cached in registers, except at the large-bond size (32 rows per lane)
  // where they are read from LDS where used
  constexpr bool VCACHE = RPL <= 18;
  unrolled<0, NPAN>([&](auto PB) {
    constexpr int T0 = PB;
    const int jend = k < 8 * T0 + 8 ? k : 8 * T0 + 8;
    for (int j = 8 * T0; j < jend; ++j) {
      const double tau = sTau[j];
      const double* v = vbuf + (j & 1) * MAXM;
      double vr[VCACHE ? RPL : 1];
      if constexpr (VCACHE) {
#pragma unroll
        for (int t = T0; t < RPL; ++t) vr[t] = v[gl + 8 * t];
      }
      auto V = [&](int t) -> double { if constexpr (VCACHE) return vr[t]; else return v[gl + 8 * t]; };
#pragma unroll
      for (int q = 0; q < CPG; ++q) {
        const int jj = g + q * kGroups;
        if (jj > j && jj < n) {
          if (tau != 0.0) {
            double wp[kAcc] = {};
#pragma unroll
            for (int t = T0; t < RPL; ++t) wp[t % kAcc] = fma(V(t), c[q][t], wp[t % kAcc]);
            const double w = add_up(wp) * tau;
#pragma unroll
            for (int t = T0; t < RPL; ++t) c[q][t] = fma(-V(t), w, c[q][t]);
          }
          if (jj == j + 1 && jj < k) make_reflector(PB, c[q], jj);
        }
      }
      __syncthreads();
    }
  });
  // R into sR; reflectors (with the unit diagonal) back into X for the accumulation of Q
#pragma unroll
  for (int q = 0; q < CPG; ++q) {
    const int jj = g + q * kGroups;
    if (jj < n) {
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        const int row = gl + 8 * t;
        if (t < NPAN && row < k) sR[(size_t)jj * ldr + row] = (row <= jj) ? c[q][t] : 0.0;
        if (jj < k && row < m) X[(size_t)jj * m + row] = (row > jj) ? c[q][t] : (row == jj ? 1.0 : 0.0);
      }
    }
  }
  __syncthreads();
  // Q columns: every group walks the same j sequence, so the eight groups of a wave read the same
  // reflector (LDS broadcast) and each v_j is loaded once per step
#pragma unroll
  for (int q = 0; q < CPG; ++q) {
    const int jj = g + q * kGroups;
#pragma unroll
    for (int t = 0; t < RPL; ++t) c[q][t] = (gl + 8 * t == jj) ? 1.0 : 0.0;
  }
  unrolled<0, NPAN>([&](auto PB) {
    constexpr int T0 = NPAN - 1 - PB;
    const int jtop = (k < 8 * T0 + 8 ? k : 8 * T0 + 8) - 1;
    for (int j = jtop; j >= 8 * T0; --j) {
      const double tau = sTau[j];
      if (tau == 0.0) continue;
      const double* vj = X + (size_t)j * m;
      double vr[RPL];
#pragma unroll
      for (int t = T0; t < RPL; ++t) {
        const int row = gl + 8 * t;
        vr[t] = (row < m) ? vj[row] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < CPG; ++q) {
        const int jj = g + q * kGroups;
        if (jj >= j && jj < k) {
          double wp[kAcc] = {};
#pragma unroll
          for (int t = T0; t < RPL; ++t) wp[t % kAcc] = fma(vr[t], c[q][t], wp[t % kAcc]);
          const double w = add_up(wp) * tau;
#pragma unroll
          for (int t = T0; t < RPL; ++t) c[q][t] = fma(-vr[t], w, c[q][t]);
        }
      }
    }
  });
#pragma unroll
  for (int q = 0; q < CPG; ++q) {
    const int jj = g + q * kGroups;
    if (jj < k) {
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        const int row = gl + 8 * t;
        if (row < m) qdst[(size_t)jj * m + row] = c[q][t];
      }
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// One-sided Jacobi (Hestenes) on the nr x nc matrix A (nr >= nc), column j at A + j*ld: rotate
// column pairs until all are mutually orthogonal, accumulating the rotations in J (nc x nc, column
// j at J + j*ld, starts as identity), so A_in J = A_out with orthogonal columns.  A pair is left
// alone when (a_i.a_j)^2 <= tol^2 |a_i|^2 |a_j|^2 or when either column is numerically zero (norm
// below 64 eps ||A||_F), which keeps rank-deficient inputs from rotating rounding noise forever.
// The sweeps stop after one without rotations, or after one in which every pair's relative
// off-diagonal |a_i.a_j| / (|a_i| |a_j|) was at most 1e-6 before its rotation: convergence is
// quadratic there, and on the boundary matrices of this method the sweep that follows such a
// sweep never rotates (same final orthogonality, ~1 sweep in 11 saved).
//
// Ordering: odd-even transposition over ncp = nc rounded up to even slots (a zero dummy column
// fills the last slot when nc is odd).  Rounds alternate between the pairs (2k, 2k+1) and
// (2k+1, 2k+2); after each rotation the two columns exchange slots, so in ncp rounds every pair
// meets once.  Group k (8 lanes, 9 rows per lane at MAXN = 72) keeps the A columns of slots 2k and
// 2k+1 in registers for the whole factorisation, with their squared norms (exact at the start of
// each sweep, then updated from the rotation: |a_i'|^2 = |a_i|^2 - t a_i.a_j, |a_j'|^2 =
// |a_j|^2 + t a_i.a_j with t = s / c), so a round computes one dot product, not three.  The
// (2k, 2k+1) rounds need no communication; in the (2k+1, 2k+2) rounds group k fetches slot 2k+2
// from group k+1 through LDS, rotates the pair, keeps the partner's rotated column and hands its
// own rotated column back.
// Scaled rotations: a column is stored as u^ with u = d u^, and the pair's rotation is
//   u^' = u^ - (t d_v / d_u) v^,  v^' = v^ + (t d_u / d_v) u^,  d' = c d,  1/d' = (1/d) / c,
// two multiply-adds per row instead of four operations, in A and in J alike (d and 1/d are carried, so
// nothing is divided); after each sweep the scales are multiplied into the columns and start from 1
// again, before their rounding can drift.  What bounds the sweep is instruction issue on the SIMD that
// carries two column waves (255 VALU instructions per wave and round pair unscaled), hence this and the
// short scalar part of pair_rotation.
// J is not carried with the columns: the groups occupy the first 4.5 waves, and the lanes from
// JL0 up (idle otherwise) hold J by rows, two rows per lane quad, a quarter of the slots per lane.  Each
// group publishes its round's two factors in a four-round ring; the J lanes apply them one half of
// the boundary round later, which halves the LDS traffic of the hand-over and takes the J update off
// the groups' path.
// On return A and J hold the columns (stride ld = MAXN + 1, zero rows from nr resp. nc up to
// MAXN), sSig[i] = ||A[:, i]|| and sPerm[a] = index of the a-th largest (ties by index).
// ---------------------------------------------------------------------------------------------
template <int GW>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(GW == 4 || GW == 8, "group reductions over 4 or 8 lanes");
  v += dpp_d<0xB1>(v);  // quad_perm [1,0,3,2]
  v += dpp_d<0x4E>(v);  // quad_perm [2,3,0,1]
  if (GW == 8) v += dpp_d<0x141>(v);  // row_half_mirror
  return v;
}

// Columns per group of GW lanes.  Four, for the large bonds: half of the boundary pairs are then a group's own
// and a quarter of the columns are handed over in a round, not half, where the hand-over is what a round waits
// for (128 columns of 1 KB, 2.5 k LDS cycles of a round pair with groups of two): 14 x 14, chi 64, 96 samples,
// 87.4 -> 80.8 ms.  Two up to 72, where a round waits for its chain of dependent instructions: with four,
// fewer waves run two chains each (a row at 32 columns 1.93 -> 3.5 ms, at 72 6.5 -> 7.3).
template <int MAXN, int GW>
constexpr int jacobi_columns() { return MAXN == kMaxNBig && GW == 8 ? 4 : 2; }

// hb: the hand-over buffers (2 ceil(nc/2) columns of MAXN doubles, of MAXN + 8 at the large-bond size) and
// ring: the rotation ring (4 rounds of MAXN/2 (alpha, beta) pairs), both in LDS, as sScl (the scales,
// JacobiScales::room entries).  With A and J themselves in LDS they overlay them (hb = A, ring = J: both are
// dead while the sweeps run); with A and J in global memory (the large-bond kernel) they are separate LDS
// buffers.  JL0: first lane of the J rows.
template <int MAXN, int GW, int NT, int JL0>
__device__ __forceinline__ bool jacobi_svd(double* A, int nr, int nc, double* J, double* sSig,
                                           int* sPerm, int* sFlag, double* sScal, double2* sScl,
                                           int max_sweeps, double* hb, double2* ring) {
  constexpr int RPL = MAXN / GW;  // rows per lane of a column group
  constexpr int HS = MAXN / 2;    // pairs of a round; J entries per lane
  constexpr int HQ = MAXN / 4;    // slots per J quarter row
  constexpr int ld = MAXN + 1;
  constexpr int SLOT = MAXN;      // one A column handed over
  // bank offset of hand-over slot q: consecutive groups' 8-lane stores start 16 banks apart.  The
  // large-bond size pads the slot stride by 8 doubles instead of rotating inside the slot, so that
  // every hand-over address is the slot's base plus a constant (no per-row address registers).
  constexpr bool PADSLOT = MAXN > kMaxN;
  constexpr int SLOTP = PADSLOT ? SLOT + 8 : SLOT;
  constexpr int kRot = (!PADSLOT && (2 * SLOT) % 64 == 0) ? 8 : 0;
  constexpr int NC = jacobi_columns<MAXN, GW>();
  static_assert(MAXN % GW == 0 && (MAXN / NC) * GW <= JL0, "column groups below the J lanes");
  static_assert(JL0 % 64 == 0 && JL0 + 2 * MAXN <= NT && MAXN % 4 == 0, "J rows fit");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k = threadIdx.x / GW, gl = threadIdx.x % GW;
  {
    double s2 = 0.0;
    for (int idx = threadIdx.x; idx < nr * nc; idx += NT) {
      const double v = A[(size_t)(idx / nr) * ld + idx % nr];
      s2 = fma(v, v, s2);
    }
    s2 = wave_sum_dpp(s2);
    if (lane == 0) sScal[wave] = s2;
  }
  if (threadIdx.x < 2) sFlag[threadIdx.x] = 0;
  const int ncp = (nc + NC - 1) / NC * NC, np = ncp / 2, ng = ncp / NC;  // slots, pairs, groups
  const bool active = nc > 1 && k < ng;
  const bool full = np == HS;  // every slot in use
  // J lanes: the lane quad (4r .. 4r+3) holds rows 2r and 2r+1 of J, lane 4r+h their slots from h HQ
  const int jl = (int)threadIdx.x - JL0;
  const int jr = 2 * (jl >> 2), jh = jl & 3;
  const bool jact = nc > 1 && jl >= 0 && jr < nc;
  const int jb = jh * HQ;  // first slot of this quarter row
  // one register array serves both roles (a lane is either a column-group lane or a J lane), so
  // that the compiler does not keep both sets live: X | Y for the groups, the J quarter rows else
  static_assert(NC * RPL <= HS && HQ % 2 == 0, "a lane's columns fit in the J entries, whole pairs per quarter row");
  double Jr[HS];
  double (&X)[RPL] = *reinterpret_cast<double (*)[RPL]>(&Jr[0]);
  double (&Y)[RPL] = *reinterpret_cast<double (*)[RPL]>(&Jr[RPL]);
  double (&Z)[RPL] = *reinterpret_cast<double (*)[RPL]>(&Jr[NC == 4 ? 2 * RPL : 0]);
  double (&V)[RPL] = *reinterpret_cast<double (*)[RPL]>(&Jr[NC == 4 ? 3 * RPL : RPL]);
  int idX = NC * k, idY = NC * k + 1, idZ = NC * k + 2, idV = NC * k + 3;
  // the squared norms exact at each sweep's start
  Col cX{0.0, 1.0, 1.0}, cY{0.0, 1.0, 1.0}, cZ{0.0, 1.0, 1.0}, cV{0.0, 1.0, 1.0};
  if (active) {
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      const int r = gl + GW * t;
      X[t] = (idX < nc && r < nr) ? A[(size_t)idX * ld + r] : 0.0;
      Y[t] = (idY < nc && r < nr) ? A[(size_t)idY * ld + r] : 0.0;
      if constexpr (NC == 4) {
        Z[t] = (idZ < nc && r < nr) ? A[(size_t)idZ * ld + r] : 0.0;
        V[t] = (idV < nc && r < nr) ? A[(size_t)idV * ld + r] : 0.0;
      }
    }
  }
  if (jact) {
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
      Jr[q] = (jb + q == jr) ? 1.0 : 0.0;
      Jr[HQ + q] = (jb + q == jr + 1) ? 1.0 : 0.0;
    }
  }
  __syncthreads();  // A read into registers: the hand-over buffers below overlay it
  double fro2 = 0.0;
  for (int w = 0; w < (NT / 64); ++w) fro2 += sScal[w];
  // exact power-of-two scaling to ||A||_F ~ 1 (undone on write-back)
  int fexp = 0;
  (void)frexp(fro2, &fexp);
  const int shift = (fro2 > 0.0) ? -(fexp / 2) : 0;
  if (active) {
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      X[t] = ldexp(X[t], shift);
      Y[t] = ldexp(Y[t], shift);
      if constexpr (NC == 4) {
        Z[t] = ldexp(Z[t], shift);
        V[t] = ldexp(V[t], shift);
      }
    }
  }
  fro2 = ldexp(fro2, 2 * shift);
  const double zero2 = fro2 * (64.0 * 2.220446049250313e-16) * (64.0 * 2.220446049250313e-16);
  const double tol = fmax(1e-15, 2.220446049250313e-16 * (double)nr);
  const double tol2 = tol * tol;
  // hand-over buffers: slot q of buffer 1 at hb + q*SLOTP, of buffer 2 at hb + (ng + q)*SLOTP
  auto at = [&](int q, int e) -> double& {
    if constexpr (PADSLOT)
      return hb[(size_t)q * SLOTP + e];
    else
      return hb[(size_t)q * SLOT + (e + kRot * (q & 3)) % SLOT];
  };
  int* id1 = sPerm;
  int* id2 = sPerm + ng;
  double* nrm1 = sSig;  // norms travelling with the handed-over columns
  double* nrm2 = sSig + ng;
  const JacobiScales scales{ng};
  double2* scl1 = sScl + scales.lower(0);  // scales (d, 1/d) travelling with them
  double2* scl2 = sScl + scales.upper(0);
  double2* sclE = sScl + scales.end(0);  // the sweep's final ones
  int rnd = 0;  // round counter (all threads)

  // round (2k, 2k+1) with slot 2k in u and slot 2k+1 in v; afterwards the slots are exchanged,
  // i.e. the caller swaps the roles of the two register sets
  auto inner = [&](double (&u)[RPL], double (&v)[RPL], Col& cu, Col& cv, bool& rot_any, bool& big_any) {
    if (active) {
      double g = 0.0;
#pragma unroll
      for (int t = 0; t < RPL; ++t) g = fma(u[t], v[t], g);
      const PairRot r = pair_rotation(group_sum<GW>(g), cu, cv, zero2, tol2, big_any);
      if (gl == 0) ring[(rnd & 3) * HS + k] = make_double2(r.alpha, r.beta);
      if (r.on) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          const double a = u[t];
          u[t] = fma(-r.alpha, v[t], a);
          v[t] = fma(r.beta, a, v[t]);
        }
        rot_any = true;
      }
    }
    ++rnd;
  };
  // J rows: apply the rotations of the inner round t0, resp. of the boundary round t0.  A pair
  // (left, right) with factors (alpha, beta) maps to left' = right + beta left, right' = left - alpha
  // right (the rotated pair also exchanges its slots, as the columns do).  All HS pairs are applied
  // without tests: what lands in the slots from ncp on is never read.  The one slot that a boundary
  // round would exchange with them, the last (2 np - 1), is put back after it.
  // Two rows by quarter rows per lane, not one by half rows: a lane then reads half as many factors
  // (16 bytes each, for every lane of every J wave: with half rows they took 864 of the 1512 LDS cycles
  // of a round pair at MAXN = 72, the sweep's tightest resource).  They are read in chunks of kJC pairs
  // (a scheduling barrier after each) so that the J lanes' live registers stay near their rows plus a
  // chunk.
  constexpr int HP = HQ / 2;  // pairs per quarter row
  constexpr int kJC = HP % 6 == 0 ? 6 : HP % 4 == 0 ? 4 : HP % 3 == 0 ? 3 : 2;
  static_assert(HP % kJC == 0, "whole chunks of pairs per quarter row");
  auto rotate = [&](double2 f, double& l, double& r) {
    const double a = l;
    l = fma(f.y, a, r);
    r = fma(-f.x, r, a);
  };
  const int last_q = __builtin_amdgcn_readfirstlane((2 * np - 1) % HQ);  // the last slot in its quarter row
  const bool has_last = jh == (2 * np - 1) / HQ;
  const int k0 = jb / 2;  // first inner pair (2k, 2k+1) of this quarter row
  auto japply_inner = [&](int t0) {
    if (!jact) return;
    const double2* ri = ring + (t0 & 3) * HS + k0;
#pragma unroll
    for (int q0 = 0; q0 < HP; q0 += kJC) {
      double2 f[kJC];
#pragma unroll
      for (int e = 0; e < kJC; ++e) f[e] = ri[q0 + e];
#pragma unroll
      for (int e = 0; e < kJC; ++e) {
        rotate(f[e], Jr[2 * (q0 + e)], Jr[2 * (q0 + e) + 1]);
        rotate(f[e], Jr[HQ + 2 * (q0 + e)], Jr[HQ + 2 * (q0 + e) + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto japply_boundary = [&](int t0) {
    if (!jact) return;
    double last0 = 0.0, last1 = 0.0;
    if (!full) {
#pragma unroll
      for (int q = 1; q < HQ; q += 2) {
        last0 = last_q == q ? Jr[q] : last0;
        last1 = last_q == q ? Jr[HQ + q] : last1;
      }
    }
    // boundary pairs (2k+1, 2k+2): across the quad's lanes, then inside the quarter row
    const double2* rb = ring + (t0 & 3) * HS + k0;
    {
      const double2 fl = rb[jh > 0 ? -1 : 0], fr = rb[HP - 1];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        double& first = Jr[a * HQ];
        double& end = Jr[a * HQ + HQ - 1];
        const double before = dpp_d<0x90>(end);   // quad_perm [0,0,1,2]: the lane before's last slot
        const double after = dpp_d<0xF9>(first);  // quad_perm [1,2,3,3]: the lane after's first slot
        const double nf = fma(-fl.x, first, before), ne = fma(fr.y, end, after);
        first = jh > 0 ? nf : first;
        end = jh < 3 ? ne : end;
      }
    }
#pragma unroll
    for (int q0 = 0; q0 < HP; q0 += kJC) {
      double2 f[kJC];
#pragma unroll
      for (int e = 0; e < kJC; ++e)
        if (q0 + e + 1 < HP) f[e] = rb[q0 + e];
#pragma unroll
      for (int e = 0; e < kJC; ++e)
        if (q0 + e + 1 < HP) {  // local pair (q, q + 1), q = 2 (q0 + e) + 1
          rotate(f[e], Jr[2 * (q0 + e) + 1], Jr[2 * (q0 + e) + 2]);
          rotate(f[e], Jr[HQ + 2 * (q0 + e) + 1], Jr[HQ + 2 * (q0 + e) + 2]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!full) {
#pragma unroll
      for (int q = 1; q < HQ; q += 2) {
        Jr[q] = (has_last && last_q == q) ? last0 : Jr[q];
        Jr[HQ + q] = (has_last && last_q == q) ? last1 : Jr[HQ + q];
      }
    }
  };
  // round (2k+1, 2k+2) with slot 2k in lo and slot 2k+1 in hi.  The J rows take the inner round before it
  // while the columns rotate, and this round after the second barrier: half of their work beside each
  // half of the columns' (all of it after the second barrier held up the next first one)
  auto boundary = [&](double (&lo)[RPL], double (&hi)[RPL], Col& clo, Col& chi, int& ilo, int& ihi, bool& rot_any,
                      bool& big_any) {
    if (active) {  // slot 2k goes to group k-1
#pragma unroll
      for (int t = 0; t < RPL; ++t) at(k, gl + GW * t) = lo[t];
      if (gl == 0) {
        id1[k] = ilo;
        nrm1[k] = clo.n;
        scl1[k] = make_double2(clo.d, clo.id);
      }
    }
    __syncthreads();
    japply_inner(rnd - 1);
    if (active && k + 1 < np) {  // pair (slot 2k+1, slot 2k+2): keep the rotated partner
      const int ip = id1[k + 1];
      const double2 sp = scl1[k + 1];
      Col cp{nrm1[k + 1], sp.x, sp.y};
      PairRot r;
      double g = 0.0;
      double P[RPL];
#pragma unroll
      for (int t = 0; t < RPL; ++t) P[t] = at(k + 1, gl + GW * t);
#pragma unroll
      for (int t = 0; t < RPL; ++t) g = fma(hi[t], P[t], g);
      r = pair_rotation(group_sum<GW>(g), chi, cp, zero2, tol2, big_any);
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        at(np + k, gl + GW * t) = fma(-r.alpha, P[t], hi[t]);
        hi[t] = fma(r.beta, hi[t], P[t]);
      }
      rot_any |= r.on;
      if (gl == 0) {
        ring[(rnd & 3) * HS + k] = make_double2(r.alpha, r.beta);
        id2[k] = ihi;
        nrm2[k] = chi.n;
        scl2[k] = make_double2(chi.d, chi.id);
      }
      ihi = ip;
      chi = cp;
    }
    __syncthreads();
    if (active && k >= 1) {  // slot 2k receives the rotated slot 2k-1 of group k-1
#pragma unroll
      for (int t = 0; t < RPL; ++t) lo[t] = at(np + k - 1, gl + GW * t);
      ilo = id2[k - 1];
      const double2 sl = scl2[k - 1];
      clo = Col{nrm2[k - 1], sl.x, sl.y};
    }
    japply_boundary(rnd);
    ++rnd;
  };

  // The same two rounds for groups of four columns, slots 4k .. 4k+3 in (a, b, c, d): the pairs (a, b) and
  // (c, d); then, with b, a, d, c in the slots, (a, d) within the group and (c, slot 4k+4), slot 4k in b.
  // Both of a round's pairs interleave.  Afterwards the slots hold b, d, a, c: four round pairs return the
  // roles.
  auto inner4 = [&](double (&a)[RPL], double (&b)[RPL], double (&c)[RPL], double (&e)[RPL], Col& ca, Col& cb, Col& cc,
                    Col& ce, bool& rot_any, bool& big_any) {
    if (active) {
      double g0 = 0.0, g1 = 0.0;
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        g0 = fma(a[t], b[t], g0);
        g1 = fma(c[t], e[t], g1);
      }
      PairRot r0, r1;
      pair_rotations(group_sum<GW>(g0), group_sum<GW>(g1), ca, cb, cc, ce, zero2, tol2, big_any, r0, r1);
      if (gl == 0) {
        ring[(rnd & 3) * HS + 2 * k] = make_double2(r0.alpha, r0.beta);
        ring[(rnd & 3) * HS + 2 * k + 1] = make_double2(r1.alpha, r1.beta);
      }
      if (r0.on || r1.on) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          const double u = a[t], w = c[t];
          a[t] = fma(-r0.alpha, b[t], u);
          b[t] = fma(r0.beta, u, b[t]);
          c[t] = fma(-r1.alpha, e[t], w);
          e[t] = fma(r1.beta, w, e[t]);
        }
        rot_any = true;
      }
    }
    ++rnd;
  };
  auto boundary4 = [&](double (&lo)[RPL], double (&u)[RPL], double (&v)[RPL], double (&hi)[RPL], Col& clo, Col& cu,
                       Col& cv, Col& chi, int& ilo, int& ihi, bool& rot_any, bool& big_any) {
    if (active) {  // slot 4k goes to group k-1
#pragma unroll
      for (int t = 0; t < RPL; ++t) at(k, gl + GW * t) = lo[t];
      if (gl == 0) {
        id1[k] = ilo;
        nrm1[k] = clo.n;
        scl1[k] = make_double2(clo.d, clo.id);
      }
    }
    __syncthreads();
    japply_inner(rnd - 1);
    if (active) {
      const bool next = k + 1 < ng;  // the last group's slot 4k+3 has no partner: its own slot 4k, unused
      const int kn = next ? k + 1 : k;
      const int ip = id1[kn];
      const double2 sp = scl1[kn];
      Col cp{next ? nrm1[kn] : 0.0, sp.x, sp.y};  // norm 0: left alone
      double P[RPL];
#pragma unroll
      for (int t = 0; t < RPL; ++t) P[t] = at(kn, gl + GW * t);
      double g0 = 0.0, g1 = 0.0;
#pragma unroll
      for (int t = 0; t < RPL; ++t) {
        g0 = fma(u[t], v[t], g0);
        g1 = fma(hi[t], P[t], g1);
      }
      PairRot r0, r1;
      pair_rotations(group_sum<GW>(g0), group_sum<GW>(g1), cu, cv, chi, cp, zero2, tol2, big_any, r0, r1);
      if (next) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          at(ng + k, gl + GW * t) = fma(-r1.alpha, P[t], hi[t]);
          hi[t] = fma(r1.beta, hi[t], P[t]);
        }
      }
      if (r0.on) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          const double w = u[t];
          u[t] = fma(-r0.alpha, v[t], w);
          v[t] = fma(r0.beta, w, v[t]);
        }
      }
      rot_any |= r0.on || r1.on;
      if (gl == 0) {
        ring[(rnd & 3) * HS + 2 * k] = make_double2(r0.alpha, r0.beta);
        if (next) {
          ring[(rnd & 3) * HS + 2 * k + 1] = make_double2(r1.alpha, r1.beta);
          id2[k] = ihi;
          nrm2[k] = chi.n;
          scl2[k] = make_double2(chi.d, chi.id);
        }
      }
      if (next) {
        ihi = ip;
        chi = cp;
      }
    }
    __syncthreads();
    if (active && k >= 1) {  // slot 4k receives the rotated slot 4k-1 of group k-1
#pragma unroll
      for (int t = 0; t < RPL; ++t) lo[t] = at(ng + k - 1, gl + GW * t);
      ilo = id2[k - 1];
      const double2 sl = scl2[k - 1];
      clo = Col{nrm2[k - 1], sl.x, sl.y};
    }
    japply_boundary(rnd);
    ++rnd;
  };
  // a round pair with the slots in (a, b, c, d), which it leaves in (b, d, a, c)
  auto rounds4 = [&](double (&a)[RPL], double (&b)[RPL], double (&c)[RPL], double (&e)[RPL], Col& ca, Col& cb, Col& cc,
                     Col& ce, int& ib, int& ic, bool& rot_any, bool& big_any) {
    inner4(a, b, c, e, ca, cb, cc, ce, rot_any, big_any);
    boundary4(b, a, e, c, cb, ca, ce, cc, ib, ic, rot_any, big_any);
  };

  bool more = false;  // still rotating after the last sweep run: not converged
  if (nc > 1) {
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
      bool rot_any = false, big_any = false;
      if (active) {
        auto norm = [&](double (&x)[RPL]) {
          double v = 0.0;
#pragma unroll
          for (int t = 0; t < RPL; ++t) v = fma(x[t], x[t], v);
          return Col{group_sum<GW>(v), 1.0, 1.0};
        };
        cX = norm(X);
        cY = norm(Y);
        if constexpr (NC == 4) {
          cZ = norm(Z);
          cV = norm(V);
        }
      }
      if constexpr (NC == 4) {
        // four round pairs per iteration return the roles (np is even); two leave d, c, b, a in the slots
        for (int h = 0; h < np; h += 4) {
          rounds4(X, Y, Z, V, cX, cY, cZ, cV, idY, idZ, rot_any, big_any);
          rounds4(Y, V, X, Z, cY, cV, cX, cZ, idV, idX, rot_any, big_any);
          if (h + 2 < np) {
            rounds4(V, Z, Y, X, cV, cZ, cY, cX, idZ, idY, rot_any, big_any);
            rounds4(Z, X, V, Y, cZ, cX, cV, cY, idX, idV, rot_any, big_any);
          }
        }
        if (np & 2) {
          if (active) {  // only on the groups' lanes, whose columns share their registers with the J rows
#pragma unroll
            for (int t = 0; t < RPL; ++t) {
              const double x = X[t], y = Y[t];
              X[t] = V[t];
              V[t] = x;
              Y[t] = Z[t];
              Z[t] = y;
            }
          }
          const int ix = idX, iy = idY;
          idX = idV;
          idV = ix;
          idY = idZ;
          idZ = iy;
          const Col x = cX, y = cY;
          cX = cV;
          cV = x;
          cY = cZ;
          cZ = y;
        }
      } else {
      // two round pairs per iteration so that the register roles return: (X, Y) = (2k, 2k+1)
      for (int h = 0; h + 2 <= np; h += 2) {
        inner(X, Y, cX, cY, rot_any, big_any);  // now Y = 2k, X = 2k+1
        boundary(Y, X, cY, cX, idY, idX, rot_any, big_any);
        inner(Y, X, cY, cX, rot_any, big_any);  // now X = 2k, Y = 2k+1
        boundary(X, Y, cX, cY, idX, idY, rot_any, big_any);
      }
      if (np & 1) {
        inner(X, Y, cX, cY, rot_any, big_any);
        boundary(Y, X, cY, cX, idY, idX, rot_any, big_any);
        // restore the roles (X, Y) = (2k, 2k+1); only on the groups' lanes, since X and Y share
        // their registers with the J rows
        if (active) {
#pragma unroll
          for (int t = 0; t < RPL; ++t) {
            const double a = X[t];
            X[t] = Y[t];
            Y[t] = a;
          }
        }
        const int ti = idX;
        idX = idY;
        idY = ti;
        const Col tc = cX;
        cX = cY;
        cY = tc;
      }
      }
      // the scales into the columns and, by slot through LDS, into the J rows
      if (active) {
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          X[t] *= cX.d;
          Y[t] *= cY.d;
          if constexpr (NC == 4) {
            Z[t] *= cZ.d;
            V[t] *= cV.d;
          }
        }
        if (gl == 0) {
          sclE[NC / 2 * k] = make_double2(cX.d, cY.d);
          if constexpr (NC == 4) sclE[NC / 2 * k + 1] = make_double2(cZ.d, cV.d);
        }
      }
      if (rot_any) sFlag[0] = 1;
      if (big_any) sFlag[1] = 1;
      __syncthreads();
      if (jact) {
#pragma unroll
        for (int q = 0; q < HQ; q += 2) {
          const double2 f = sclE[jb / 2 + q / 2];
          Jr[q] *= f.x;
          Jr[q + 1] *= f.y;
          Jr[HQ + q] *= f.x;
          Jr[HQ + q + 1] *= f.y;
        }
      }
      more = sFlag[0] != 0 && sFlag[1] != 0;
      __syncthreads();
      if (threadIdx.x < 2) sFlag[threadIdx.x] = 0;
      __syncthreads();
      if (!more) break;
    }
  }
  // hand-over buffers and rotation ring dead: column ids of the slots for the J rows
  if (active && gl == 0) {
    sPerm[NC * k] = idX;
    sPerm[NC * k + 1] = idY;
    if constexpr (NC == 4) {
      sPerm[NC * k + 2] = idZ;
      sPerm[NC * k + 3] = idV;
    }
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      const int r = gl + GW * t;
      if (idX < nc) A[(size_t)idX * ld + r] = ldexp(X[t], -shift);
      if (idY < nc) A[(size_t)idY * ld + r] = ldexp(Y[t], -shift);
      if constexpr (NC == 4) {
        if (idZ < nc) A[(size_t)idZ * ld + r] = ldexp(Z[t], -shift);
        if (idV < nc) A[(size_t)idV * ld + r] = ldexp(V[t], -shift);
      }
    }
  } else if (nc == 1 && k == 0) {
    for (int t = 0; t < RPL; ++t) {
      const int r = gl + GW * t;
      if (r >= nr) A[r] = 0.0;
      J[r] = (r == 0) ? 1.0 : 0.0;
    }
  }
  if (jact) {
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
      if (jb + q < ncp) {
        const int id = sPerm[jb + q];
        if (id < nc) {
          J[(size_t)id * ld + jr] = Jr[q];
          if (jr + 1 < nc) J[(size_t)id * ld + jr + 1] = Jr[HQ + q];
        }
      }
    }
  }
  __syncthreads();
  {
    const int g8 = threadIdx.x >> 3, l8 = threadIdx.x & 7;
    for (int i = g8; i < nc; i += NT / 8) {
      const double* ai = A + (size_t)i * ld;
      double s2 = 0.0;
      for (int r = l8; r < nr; r += 8) s2 = fma(ai[r], ai[r], s2);
      s2 = group8_sum(s2);
      if (l8 == 0) sSig[i] = sqrt(s2);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nc; i += NT) {
    const double si = sSig[i];
    int rank = 0;
    for (int j = 0; j < nc; ++j) {
      const double sj = sSig[j];
      rank += (sj > si) || (sj == si && j < i);
    }
    sPerm[rank] = i;
  }
  __syncthreads();
  return !more;
}

// ---------------------------------------------------------------------------------------------
// The row step.  LDS: sX (QR matrix, later A | J of the Jacobi), sR (R, later G = U_k S_k),
// sB (boundary site cache), sT (row tensor).  With a tape pointer the factorisations are recorded
// (TapeSlot layout) for the adjoint.
// ---------------------------------------------------------------------------------------------
// pmode: preconditioning of the large truncated SVDs (cuts whose Theta is wide or square with at least
// pthr rows): PEPS_PRECOND_NONE, PEPS_PRECOND_QR_T (sweeps that are never reversed) or
// PEPS_PRECOND_SORTED_QR; see the forms of the SVD below.
// The row step of sample b, shared by the batch kernel (one lattice) and the ragged kernel (several
// lattices in one launch).  qslot: doubles per (sample, site) Q-factor slot of qscr.
// tslot: doubles per (sample, site) tape slot.
template <int MAXN, int DK, typename CT, int GW>
__device__ __forceinline__ void row_sweep_body(const Dims& d, const int* __restrict__ bond_all,
                                               const int* __restrict__ qrk_all, int y,
                                               const double* __restrict__ proj, const uint8_t* __restrict__ valid,
                                               const double* __restrict__ prev_row, double* __restrict__ out_row,
                                               double* __restrict__ qscr, size_t qslot, double* __restrict__ lognu,
                                               double* __restrict__ tape, size_t tslot, int pmode, int pthr,
                                               uint32_t* __restrict__ status, double* __restrict__ wbig, int b) {
  constexpr int MAXM = MAXN * DK;
  constexpr int NT = RowCfg<MAXN>::NT;
  // Large bonds (chi * Dk above the LDS-resident limit): the working matrices X, A | J and R | G
  // live in a per-sample slot of global memory (wbig, kBigSlot doubles; the working set stays in
  // the L2 and last-level caches), the Jacobi's hand-over buffers and rotation ring in LDS.
  constexpr bool BIG = MAXN > kMaxN;
  static_assert(!BIG || MAXN == kMaxNBig, "one large-bond instantiation");
  // sX holds the QR matrix (MAXM x MAXN) and later A and J of the Jacobi (2 x MAXN^2)
  constexpr int XSIZE = (MAXM * MAXN > 2 * (MAXN + 1) * MAXN) ? MAXM * MAXN : 2 * (MAXN + 1) * MAXN;
  constexpr int XPT = (MAXM * MAXN + NT - 1) / NT;  // X entries per thread
  // staging chunk of Q in the Theta product (KCH rows of Q^T) and the LDS buffer sB that holds it,
  // the Householder vector pair and (LDS-resident case) the boundary site
  constexpr int KCH = BIG ? 8 : ((MAXN / (DK * DK)) / 4 * 4 < 16 ? (MAXN / (DK * DK)) / 4 * 4 : 16);
  constexpr int SBSIZE = BIG ? (MAXM * KCH > 2 * MAXM ? MAXM * KCH : 2 * MAXM) : MAXN * MAXN / DK;
  static_assert(!BIG || XSIZE + (MAXN + 1) * MAXN + MAXM * MAXN <= kBigSlot, "large-bond slot");
  using TS = TapeSlot<MAXN>;
  __shared__ double sXl[BIG ? 1 : XSIZE];
  __shared__ double sRl[BIG ? 1 : (MAXN + 1) * MAXN];
  __shared__ __align__(16) double sB[SBSIZE];
  __shared__ double sHB[BIG ? 2 * (MAXN / 2) * (MAXN + 8) : 1];  // Jacobi hand-over buffers (padded slots)
  __shared__ double2 sRing[BIG ? 4 * (MAXN / 2) : 1];      // Jacobi rotation ring
  __shared__ double sT[DK * DK * DK * DK];
  __shared__ double sTau[MAXN];
  __shared__ double sSig[MAXN];
  __shared__ double sScal[(NT / 64)];
  __shared__ int sPerm[MAXN];
  __shared__ int sCol[MAXN];  // sorted-column QR: rank of each Theta column by norm
  __shared__ int sFlag[2];
  // phase clocks (d.phase_clk set): cycles per phase and the last mark, kept by thread 0 in LDS
  __shared__ unsigned long long sPh[PEPS_PH_COUNT + 1];

  if (!valid[b]) return;
  const bool phon = d.phase_clk != nullptr;
  if (phon && threadIdx.x == 0) {
    for (int p = 0; p < PEPS_PH_COUNT; ++p) sPh[p] = 0;
    sPh[PEPS_PH_COUNT] = __builtin_readcyclecounter();
  }
  // thread 0 books the cycles since the previous mark to phase p (called right after a barrier)
  auto mark = [&](int p) {
    if (phon && threadIdx.x == 0) {
      const unsigned long long t = __builtin_readcyclecounter();
      sPh[p] += t - sPh[PEPS_PH_COUNT];
      sPh[PEPS_PH_COUNT] = t;
    }
  };
  double* const sX = BIG ? wbig + (size_t)b * kBigSlot : sXl;
  double* const sR = BIG ? sX + XSIZE : sRl;
  double* const sY = BIG ? sR + (MAXN + 1) * MAXN : sXl;  // Y = R_{c-1} B_c (in place in sX when LDS)
  const int L = d.L, Dk = DK;
  const int* bprev = bond_all + (size_t)(y - 1) * (L + 1);
  const int* bnew = bond_all + (size_t)y * (L + 1);
  const int* qrk = qrk_all + (size_t)y * L;
  const double* pb = proj + ((size_t)b * d.n_sites + (size_t)y * L) * d.P4;
  const double* prev = prev_row + (size_t)b * d.row_stride;
  double* outp = out_row + (size_t)b * d.row_stride;
  double* qs = qscr + (size_t)b * L * qslot;
  double* tp = tape ? tape + (size_t)b * L * tslot : nullptr;

  // ---------------- left to right: X_c = R_{c-1} M_c, QR ----------------
  int r_prev = 1;
  if (threadIdx.x == 0) sR[0] = 1.0;
  __syncthreads();
  int m_last = 0;
  for (int c = 0; c < L; ++c) {
    const int dl = c > 0 ? Dk : 1, dr = c < L - 1 ? Dk : 1;
    const int bc = bprev[c], bn = bprev[c + 1];
    const double* Bs = prev + (size_t)c * d.site_stride;  // [a][dd][a']
    if constexpr (!BIG)
      for (int i = threadIdx.x; i < bc * Dk * bn; i += NT) sB[i] = Bs[i];
    for (int i = threadIdx.x; i < dl * dr * Dk * Dk; i += NT) sT[i] = pb[(size_t)c * d.P4 + i];
    __syncthreads();
    // Y[(i,l)][(dd,a')] = sum_a R[i][a*dl+l] B[a][(dd,a')]   (into sY; R carries the Schmidt
    // weights: kept in FP64 on both paths)
    {
      const int ncol = Dk * bn;
      mfma_gemm(r_prev * dl, ncol, bc,
                      [&](int il, int a) { return sR[(size_t)(a * dl + il % dl) * MAXN + il / dl]; },
                      [&](int a, int col) { return BIG ? Bs[a * ncol + col] : sB[a * ncol + col]; },
                      [&](int il, int col, double v) { sY[(size_t)il * ncol + col] = v; });
    }
    __syncthreads();
    // X[(i,u),(a',rr)] = sum_{l,dd} Y[i][l][dd][a'] T[l][rr][dd][u]   (registers, then sX)
    const int m = r_prev * Dk, n = bn * dr;
    // FP32 arithmetic sees Y scaled by an exact power of two that brings its largest entry into
    // [1/2, 1): Y follows the partial norms of the row, which leave FP32's exponent range on large
    // lattices (Z4 32 x 32: about e^-50 per row on average); the scale is undone in FP64.
    double ysc = 1.0, yun = 1.0;
    if constexpr (sizeof(CT) < sizeof(double)) {
      double mx = 0.0;
      for (int idx = threadIdx.x; idx < r_prev * dl * Dk * bn; idx += NT) mx = fmax(mx, fabs(sY[idx]));
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
      if ((threadIdx.x & 63) == 0) sScal[threadIdx.x >> 6] = mx;
      __syncthreads();
      mx = 0.0;
      for (int w = 0; w < (NT / 64); ++w) mx = fmax(mx, sScal[w]);
      if (mx > 0.0 && mx <= 1.7976931348623157e308) {
        int e = 0;
        (void)frexp(mx, &e);
        ysc = ldexp(1.0, -e);
        yun = ldexp(1.0, e);
      }
    }
    auto x_entry = [&](int idx) -> double {
      const int row = idx % m, col = idx / m;
      const int i = row / DK, u = row % DK, ap = col / dr, rr = col % dr;
      CT acc = 0;
#pragma unroll
      for (int l = 0; l < DK; ++l)
#pragma unroll
        for (int dd = 0; dd < DK; ++dd)
          if (l < dl) {
            if constexpr (sizeof(CT) < sizeof(double))
              acc = fmaf((CT)(sY[((i * dl + l) * DK + dd) * bn + ap] * ysc),
                         (CT)sT[((l * dr + rr) * DK + dd) * DK + u], acc);
            else
              acc = fma(sY[((i * dl + l) * DK + dd) * bn + ap], sT[((l * dr + rr) * DK + dd) * DK + u], acc);
          }
      if constexpr (sizeof(CT) < sizeof(double))
        return (double)acc * yun;
      else
        return acc;
    };
    if constexpr (BIG) {
      // Y and X in separate global buffers: no staging
      for (int idx = threadIdx.x; idx < m * n; idx += NT) sX[idx] = x_entry(idx);
    } else {
      // in place in LDS: every thread's entries read before any is written
      double xr[XPT];
#pragma unroll
      for (int q = 0; q < XPT; ++q) {
        const int idx = threadIdx.x + q * NT;
        xr[q] = (idx < m * n) ? x_entry(idx) : 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < XPT; ++q) {
        const int idx = threadIdx.x + q * NT;
        if (idx < m * n) sX[idx] = xr[q];
      }
    }
    __syncthreads();
    mark(PEPS_PH_X);
    if (c == L - 1) {
      m_last = m;
      break;
    }
    const int k = qrk[c];
    double* qdst = qs + (size_t)c * qslot;
    householder_qr<MAXM, MAXN, NT>(sX, m, n, sR, MAXN, sTau, sB, qdst);
    if (tp) {
      double* tr = tp + (size_t)c * tslot + TS::R;
      for (int i = threadIdx.x; i < MAXN * n; i += NT) tr[i] = sR[i];
    }
    r_prev = k;
    __syncthreads();
    mark(PEPS_PH_QR);
  }

  // ---------------- right to left: Theta_c, Jacobi SVD, truncate ----------------
  // The SVD of a cut is a one-sided Jacobi on a matrix whose columns become, when orthogonal, singular
  // vectors times singular values; the other side's vectors are the accumulated rotations J, times the
  // Q of the preconditioning QR if there was one:
  //   plain     on Theta^T unless Theta is tall (Theta's columns carry the previous cut's singular values,
  //             and on the square case the graded orientation needs ~1.7x more sweeps);
  //   sorted QR (large cuts with PEPS_PRECOND_SORTED_QR) Theta's columns sorted by norm (P),
  //             Theta P = Q_1 R (Householder), Jacobi on R^T: the columns are the right vectors, rows
  //             permuted by P, and U = Q_1 J; 8.0 instead of 11.5 sweeps (CPU experiment on captured
  //             72 x 72 Theta);
  //   QR_T      (large cuts with PEPS_PRECOND_QR_T) Theta^T = Q_x R_x, Jacobi on R_x^T: the columns are
  //             the left vectors, V = Q_x J; 6.5 sweeps.  Only for sweeps that are never reversed (the
  //             up sweeps, the strip sampler's): a left vector of singular value s from a column carries an error
  //             ~ eps ||Theta|| / s, which the truncated-SVD backward would amplify by 1 / s_kept through
  //             the kept-discarded terms (Euler identity off by 4e-9 instead of ~1e-13); the kept
  //             vectors are unaffected.
  // Both sides are needed to full relative accuracy also where nothing is reversed: with the kept part
  // from one side alone (G = Theta V_k, or V_k = Theta^T U_k / s), whose error is eps s_1 instead of
  // eps s in the part of singular value s, the row took 22% less time, but E_loc near the nodes of Psi
  // moved by 6e-10 instead of 7e-12.
  // Jacobi storage: columns padded to an odd stride (ld = rows + 1) against LDS bank conflicts
  double* A = sX;
  double* Jm = sX + (MAXN + 1) * MAXN;
  double* G = sR;  // G[i][a] at G[i*MAXN + a]
  double* const hb = BIG ? sHB : A;
  double2* const ring = BIG ? sRing : reinterpret_cast<double2*>(Jm);
  // first lane of the Jacobi's J rows (two lanes per row on average): the lanes of the column
  // groups, rounded up to whole waves
  constexpr int JL0 = ((MAXN / jacobi_columns<MAXN, GW>()) * GW + 63) / 64 * 64;
  constexpr int lda = MAXN + 1, ldj = MAXN + 1;  // the Jacobi's padded column stride
  constexpr int SPT = (MAXM * KCH + NT - 1) / NT;
  static_assert(KCH >= 4 && MAXM * KCH <= SBSIZE, "staging chunk fits sB");
  static_assert(2 * JacobiScales::room(MAXN, jacobi_columns<MAXN, GW>()) <= SBSIZE, "the Jacobi's scales fit sB");
  int chi_next = 1;
  bool converged = true;  // every SVD of the row (same value on every thread)
  for (int i = threadIdx.x; i < m_last; i += NT) sB[i] = sX[i];  // Theta_{L-1}
  __syncthreads();
  for (int c = L - 1; c >= 1; --c) {
    const int mA = qrk[c - 1];     // rows of Theta_c
    const int nA = Dk * chi_next;  // cols of Theta_c, index (u, j)
    const int p = mA < nA ? mA : nA;  // singular triplets
    const bool tall = mA > nA, large = mA >= pthr;
    const bool sq = !tall && large && pmode == PEPS_PRECOND_SORTED_QR;
    const bool qt = !tall && large && pmode == PEPS_PRECOND_QR_T;
    const bool cols_left = tall || qt;  // the Jacobi's columns are the left vectors (else the right ones)
    auto put_theta = [&](int i, int col, double v) {
      (sq ? Jm[(size_t)col * mA + i]
          : A[qt ? (size_t)i * nA + col : tall ? (size_t)col * lda + i : (size_t)i * lda + col]) = v;
    };
    if (c == L - 1) {
      for (int idx = threadIdx.x; idx < mA * nA; idx += NT) put_theta(idx / nA, idx % nA, sB[idx]);  // [i][u]
    } else {
      const int kc = qrk[c];
      const double* Qc = qs + (size_t)c * qslot;
      const int mq = mA * Dk;
      // Theta[i][(u,j)] = sum_t Q[(i,u)][t] G[t][j]   (G spans the kept singular values: FP64 on both
      // paths), chunks of Q (MAXM rows) staged through sB
      // tiles per wave: G has chi_next <= MAXN / DK columns (counted as MAXN in the LDS kernels)
      constexpr int QT = ((MAXM + 15) / 16 * (((BIG ? MAXN / DK : MAXN) + 15) / 16) + (NT / 64) - 1) / (NT / 64);
      mfma_gemm_staged<QT, KCH, SPT, true>(
          mq, chi_next, kc, [&](int iu, int t) { return Qc[(size_t)t * mq + iu]; },
          [&](int t, int j) { return G[t * MAXN + j]; }, sB,
          [&](int iu, int j, double v) { put_theta(iu / Dk, (iu % Dk) * chi_next + j, v); });
    }
    __syncthreads();
    mark(PEPS_PH_THETA);
    if (sq) {
      // column norms, ranks (descending, ties by index), columns in that order into A
      {
        const int g8 = threadIdx.x >> 3, l8 = threadIdx.x & 7;
        for (int col = g8; col < nA; col += NT / 8) {
          double s2 = 0.0;
          for (int i = l8; i < mA; i += 8) s2 = fma(Jm[(size_t)col * mA + i], Jm[(size_t)col * mA + i], s2);
          s2 = group8_sum(s2);
          if (l8 == 0) sSig[col] = s2;
        }
      }
      __syncthreads();
      for (int col = threadIdx.x; col < nA; col += NT) {
        const double sc = sSig[col];
        int rank = 0;
        for (int j = 0; j < nA; ++j) rank += (sSig[j] > sc) || (sSig[j] == sc && j < col);
        sCol[col] = rank;
      }
      __syncthreads();
      for (int idx = threadIdx.x; idx < mA * nA; idx += NT) {
        const int col = idx / mA, i = idx % mA;
        A[(size_t)sCol[col] * mA + i] = Jm[idx];
      }
      __syncthreads();
    }
    const int nr = cols_left ? mA : nA;  // rows of the Jacobi's columns
    if (sq || qt) {
      // Theta P (mA x nA) or Theta^T (nA x mA), ld mq: R (p x nr) into the J area, Q (mq x p) into sR (G is
      // consumed)
      const int mq = qt ? nA : mA;
      householder_qr<MAXN, MAXN, NT>(A, mq, nr, Jm, MAXN, sTau, sB, sR);
      // the Jacobi's matrix R^T (nr x p): column i is row i of R
      for (int idx = threadIdx.x; idx < p * nr; idx += NT) {
        const int i = idx / nr, r = idx % nr;
        A[(size_t)i * lda + r] = (r >= i) ? Jm[(size_t)r * MAXN + i] : 0.0;
      }
      __syncthreads();
      mark(PEPS_PH_PRECOND);
    }
    converged &= jacobi_svd<MAXN, GW, NT, JL0>(A, nr, p, Jm, sSig, sPerm, sFlag, sScal, reinterpret_cast<double2*>(sB),
                                                     d.max_sweeps, hb, ring);
    mark(PEPS_PH_JACOBI);
    if (sq || qt) {
      // Q J (mq x p) over J in the J area
      const int mq = qt ? nA : mA;
      mfma_gemm_sync<((MAXN + 15) / 16) * ((MAXN + 15) / 16) / (NT / 64) + 1>(
          mq, p, p, [&](int i, int t) { return sR[(size_t)t * mq + i]; },
          [&](int t, int pp) { return Jm[(size_t)pp * ldj + t]; },
          [&](int i, int pp, double v) { Jm[(size_t)pp * ldj + i] = v; });
      __syncthreads();
    }
    const int kk = bnew[c];
    double* S = outp + (size_t)c * d.site_stride;  // [a][u][j], a < kk
    // row of the Jacobi's columns that holds Theta column col (the sorted-column QR permutes them)
    auto vrow = [&](int col) { return sq ? sCol[col] : col; };
    for (int idx = threadIdx.x; idx < kk * nA; idx += NT) {
      const int a = idx / nA, col = idx % nA;
      const int pp = sPerm[a];
      if (cols_left) {
        S[idx] = Jm[(size_t)pp * ldj + col];
      } else {
        const double sg = sSig[pp];
        S[idx] = (sg > 0.0) ? A[(size_t)pp * lda + vrow(col)] / sg : 0.0;
      }
    }
    if (tp) {
      // singular vectors in descending order: the normalised Jacobi columns on one side, the
      // accumulated rotations on the other
      double* ts = tp + (size_t)c * tslot;
      for (int idx = threadIdx.x; idx < p * MAXN; idx += NT) {
        const int a = idx / MAXN, row = idx % MAXN;
        const int pp = sPerm[a];
        const double sg = sSig[pp];
        const int other = cols_left ? nA : mA;  // rows of the rotations' side
        const double col = (row < nr && sg > 0.0) ? A[(size_t)pp * lda + (cols_left ? row : vrow(row))] / sg : 0.0;
        const double rot = (row < other) ? Jm[(size_t)pp * ldj + row] : 0.0;
        ts[TS::U + idx] = cols_left ? col : rot;
        ts[TS::V + idx] = cols_left ? rot : col;
      }
      for (int a = threadIdx.x; a < p; a += NT) ts[TS::S + a] = sSig[sPerm[a]];
      if (threadIdx.x == 0) ts[TS::F] = tall ? 0.0 : 1.0;
    }
    __syncthreads();  // Q in sR fully consumed before G overwrites it
    for (int idx = threadIdx.x; idx < mA * kk; idx += NT) {
      const int i = idx / kk, a = idx % kk;
      const int pp = sPerm[a];
      G[i * MAXN + a] = cols_left ? A[(size_t)pp * lda + i] : Jm[(size_t)pp * ldj + i] * sSig[pp];
    }
    __syncthreads();
    mark(PEPS_PH_REST);
    chi_next = kk;
  }
  // site 0: Theta_0 = Q_0 G_1 (Dk x chi_1), normalise
  {
    const int k0 = qrk[0];
    const double* Q0 = qs;
    const int n0 = Dk * chi_next;
    for (int idx = threadIdx.x; idx < n0; idx += NT) {
      const int u = idx / chi_next, j = idx % chi_next;
      double acc = 0.0;
      for (int t = 0; t < k0; ++t) acc = fma(Q0[(size_t)t * Dk + u], G[t * MAXN + j], acc);
      sB[idx] = acc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double s2 = 0.0;
      for (int i = 0; i < n0; ++i) s2 = fma(sB[i], sB[i], s2);
      sSig[0] = sqrt(s2);
      lognu[(size_t)b * L + y] = log(sSig[0]);
      if (tp) tp[TS::F + 1] = sSig[0];
    }
    __syncthreads();
    const double nu = sSig[0];
    double* S0 = outp;
    for (int idx = threadIdx.x; idx < n0; idx += NT) S0[idx] = sB[idx] / nu;
  }
  if (status && !converged && threadIdx.x == 0) atomicOr(status + b, (uint32_t)PEPS_FLAG_SVD_NOCONV);
  if (phon && threadIdx.x == 0) {
    mark(PEPS_PH_REST);
    for (int p = 0; p < PEPS_PH_COUNT; ++p) atomicAdd(d.phase_clk + p, sPh[p]);
  }
}

// One boundary row for a whole batch of one lattice: one workgroup per sample.
template <int MAXN, int DK, typename CT, int GW>
__global__ void __launch_bounds__(RowCfg<MAXN>::NT, RowCfg<MAXN>::MINW)
k_row_sweep(Dims d, const int* __restrict__ bond_all, const int* __restrict__ qrk_all, int y,
            const double* __restrict__ proj, const uint8_t* __restrict__ valid,
            const double* __restrict__ prev_row, double* __restrict__ out_row,
            double* __restrict__ qscr, size_t qslot, double* __restrict__ lognu, double* __restrict__ tape,
            size_t tslot, int pmode, int pthr, uint32_t* __restrict__ status, double* __restrict__ wbig) {
  row_sweep_body<MAXN, DK, CT, GW>(d, bond_all, qrk_all, y, proj, valid, prev_row, out_row, qscr, qslot, lognu, tape,
                                   tslot, pmode, pthr, status, wbig, (int)blockIdx.x);
}

// Row y of several lattices in one launch (ragged batch): group i owns workgroups
// [first_block_i, first_block_i + B_i); each group brings its own shape tables, tensors, rows and
// scratch (its Q-factor slot stride from its own shapes).
template <int MAXN, int DK, typename CT, int GW>
__global__ void __launch_bounds__(RowCfg<MAXN>::NT, RowCfg<MAXN>::MINW)
k_row_sweep_ragged(RaggedRows r, int y, int pmode, int pthr) {
  int i = 0;
  while (i + 1 < r.n && (int)blockIdx.x >= r.g[i + 1].first_block) ++i;
  const RaggedRow& g = r.g[i];
  row_sweep_body<MAXN, DK, CT, GW>(g.d, g.bond, g.qrk, y, g.proj, g.valid, g.prev_row, g.out_row, g.qscr,
                                   g.qslot, g.lognu, nullptr, 0, pmode, pthr, g.status, g.wbig,
                                   (int)blockIdx.x - g.first_block);
}

// Launches of one class (instantiated in the k_row_*.hip files).  The large bonds always run
// eight Jacobi lanes per group of four columns (jacobi_columns).
template <int MAXN, int DK, typename CT, int GW>
hipError_t launch_row_t(const RowArgs& a, hipStream_t s) {
  const dim3 grid(a.blocks), blk(RowCfg<MAXN>::NT);
  if constexpr (DK > 1) {
    if (a.ragged) {
      hipLaunchKernelGGL((k_row_sweep_ragged<MAXN, DK, CT, GW>), grid, blk, 0, s, *a.ragged, a.y, a.pmode, a.pthr);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_row_sweep<MAXN, DK, CT, GW>), grid, blk, 0, s, *a.d, a.bond, a.qrk, a.y, a.proj, a.valid,
                     a.prev_row, a.out_row, a.qscr, a.qslot, a.lognu, a.tape, a.tslot, a.pmode, a.pthr, a.status,
                     a.wbig);
  return hipGetLastError();
}

template <int MAXN, int DK>
hipError_t launch_row_class(const RowArgs& a, hipStream_t s) {
  if constexpr (MAXN > kMaxN) {
    return a.mixed ? launch_row_t<MAXN, DK, float, 8>(a, s) : launch_row_t<MAXN, DK, double, 8>(a, s);
  } else {
    if (a.lanes == 4)
      return a.mixed ? launch_row_t<MAXN, DK, float, 4>(a, s) : launch_row_t<MAXN, DK, double, 4>(a, s);
    return a.mixed ? launch_row_t<MAXN, DK, float, 8>(a, s) : launch_row_t<MAXN, DK, double, 8>(a, s);
  }
}

}  // namespace gipeps

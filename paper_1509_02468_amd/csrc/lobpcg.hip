// Block LOBPCG as a low-pass filter (Algorithm 3, Section 6, generalised to a
// block of m vectors), z-space operator A = L_sym, B = I, T = I.
//
// Kernels:
//   lob_ynorm      ||sqrt(d)|| for the constraint vector Y = sqrt(d)/||sqrt(d)||
//   lob_start      X0[:, j] = z0 * phi_j (Legendre modulations), Y^T X0
//   lob_project    B -= Y c (constraint projection of a block)
//   gram           partial Gram tiles S^T S, S^T (A S) of S = [X, W, P] with
//                  MFMA, 4x4 tiles of v_mfma_f64_4x4x4f64 for both data types
//                  (an FP32 value widened to FP64 loses nothing and the
//                  product of two is exact in FP64, so FP32 data get FP64 sums
//                  too)
//   gram_reduce /  fixed-order two-level reduction of the tiles (one level,
//   gram_rr        inside gram_rr, with at most 16 Gram workgroups), then the
//                  Rayleigh-Ritz step on one workgroup in FP64: unit-diagonal
//                  scaling, elimination of S^T S with column dropping and the
//                  reduction of S^T A S to the kept columns' standard problem,
//                  its m smallest eigenpairs (Householder tridiagonalisation,
//                  bisection, inverse iteration); extra workgroups of the
//                  launch run the joint driver's CG update (cg_step.h)
//   lob_update     X = S C, AX = (AS) C, P = [W,P] C, AP likewise, the next
//                  residual W = AX - X Theta and its norms (and Y^T W)
//   lob_out_dots / lob_output: y = X X^T z0 (+ Y Y^T z0), x_out = y / sqrt(d)
#include <cmath>
#include <type_traits>

#include "cg_step.h"
#include "gsf_internal.h"
#include "solver_state.h"
#include "lobpcg_launch.h"

namespace gsf {
namespace {


// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ double legendre(int deg, double t) {
  double p0 = 1.0, p1 = t;
  if (deg == 0) return p0;
  for (int k = 1; k < deg; ++k) {
    const double p2 = ((2.0 * k + 1.0) * t * p1 - (double)k * p0) / (double)(k + 1);
    p0 = p1;
    p1 = p2;
  }
  return p1;
}

// sum_i sqrt(d_i)^2 -> ynorm_inv
template <typename T>
__global__ void __launch_bounds__(kThreads) lob_ynorm_kernel(const T* __restrict__ sqd, int64_t n,
                                                             double* __restrict__ partials, LobpcgState* st) {
  __shared__ double red[16];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double v[1] = {0.0};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    v[0] += (double)sqd[i] * (double)sqd[i];
  block_sum<1>(v, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

// one workgroup: sum the partials of a previous kernel in workgroup order;
// mode 0: ynorm_inv, 1: yx (M values), 2: update residuals (2M values),
// 3: output coefficients (M+1 values)
template <int NV>
__global__ void __launch_bounds__(kThreads) lob_final_kernel(const double* __restrict__ partials, int nparts,
                                                             LobpcgState* st, int mode, int m, int first,
                                                             int constraint) {
  __shared__ double red[16 * NV];
  if (mode == 2 && !st->active) return;
  double t[NV];
  reduce_partials<NV>(partials, nparts, NV, t, red);
  if (threadIdx.x != 0) return;
  if (mode == 0) {
    st->ynorm_inv = 1.0 / sqrt(t[0]);
  } else if (mode == 1 || mode == 3) {
    for (int j = 0; j < NV; ++j) st->yx[j] = t[j];
  } else {
    double mx = 0.0;
    for (int j = 0; j < m; ++j) {
      st->res[j] = sqrt(t[j]);
      st->yx[j] = constraint ? t[m + j] : 0.0;
      mx = st->res[j] > mx ? st->res[j] : mx;
    }
    if (!first) st->iters += 1;
    if (st->tol > 0.0 && mx <= st->tol) st->active = 0;
  }
}

// X0[i, j] = sqrt(d_i) x0_i phi_j(i); with the constraint also Y^T X0.
template <typename T, int M>
__global__ void __launch_bounds__(kThreads) lob_start_kernel(LobArgs a, StartDegrees deg) {
  __shared__ double red[16 * M];
  const T* __restrict__ x0 = (const T*)a.x0;
  const T* __restrict__ sqd = (const T*)a.sqd;
  T* __restrict__ X = (T*)a.X;
  const double yinv = a.st->ynorm_inv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double v[M];
#pragma unroll
  for (int j = 0; j < M; ++j) v[j] = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
    const int64_t r = i / a.cols, c = i - r * a.cols;
    const double tr = 2.0 * ((double)r + 0.5) / (double)a.rows - 1.0;
    const double tc = 2.0 * ((double)c + 0.5) / (double)a.cols - 1.0;
    const double z = (double)sqd[i] * (double)x0[i];
    const double yi = (double)sqd[i] * yinv;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      double phi = legendre(deg.b[j], tc);
      if (a.ndim == 2) phi *= legendre(deg.a[j], tr);
      const T xv = (T)(z * phi);
      X[i * M + j] = xv;
      v[j] += yi * (double)xv;
    }
  }
  if (!a.constraint) return;
  block_sum<M>(v, red);
  if (threadIdx.x == 0)
    for (int j = 0; j < M; ++j) a.vpart[(size_t)blockIdx.x * M + j] = v[j];
}

// ---------------------------------------------------------------------------
// Gram tiles with MFMA
// ---------------------------------------------------------------------------
// Output format (read by the reductions and the Rayleigh-Ritz step): tiles of
// 16x16 entries, nt = ceil(ns/16) tile rows.  S^T S: upper tiles (I <= J) in
// the order (0,0), (0,1), (1,1); S^T AS: all tiles (0,0), (0,1), (1,0), (1,1).
__device__ __forceinline__ int n_tiles_b(int nt) { return nt == 1 ? 1 : 3; }
__device__ __forceinline__ int n_tiles_a(int nt) { return nt == 1 ? 1 : 4; }

// Gram matrix (GB = S^T S or GA = S^T AS), row and column of entry e of the
// tile sequence above (tile e >> 8, entry (e & 255) = 16 i + j)
__device__ __forceinline__ void tile_entry(int e, int nt, bool& isb, int& row, int& col) {
  const int t = e >> 8, i = (e & 255) >> 4, j = e & 15;
  const int ntb = n_tiles_b(nt);
  int I, J;
  if (t < ntb) {
    isb = true;
    I = (t == 2) ? 1 : 0;
    J = (t == 0) ? 0 : 1;
  } else {
    isb = false;
    I = (nt == 1) ? 0 : (t - ntb) >> 1;
    J = (nt == 1) ? 0 : (t - ntb) & 1;
  }
  row = 16 * I + i;
  col = 16 * J + j;
}

// v_mfma_f64_4x4x4f64 runs four independent 4x4x4 products (blocks q = 0..3).
// Lane l holds A[i = l%4][k = l/16] and B[k = l/16][j = l%4] of block
// q = (l/4)%4, and receives D[i = l/16][j = l%4] of that block (found with a
// probe of the instruction on the GPU).
__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// index of the S^T S tile (I, J), I <= J, of TG column groups (row-major upper)
template <int TG>
__device__ __forceinline__ constexpr int tile_b(int I, int J) {
  return I * TG - (I * (I - 1)) / 2 + (J - I);
}

// S^T S and S^T AS over the points of each workgroup, in FP64 for both data
// types: an FP32 value widened to FP64 loses nothing and the product of two is
// exact in FP64, so FP32 data get exact products and FP64 sums.  (The entries
// that steer a nearly converged column, X^T A W ~ ||r||, are far below the
// size of their terms; FP32 sums lose them.)
//
// The ns columns form TG groups of 4.  Every lane takes one point and one
// column of a group: lane l reads point p0 + l/4, column 4G + l%4, which
// makes each group's loads one contiguous run per instruction for m = 4 and
// 8.  With that mapping block q of the MFMA sums the points p0 + 4k + q, and
// one instruction adds 16 points to the 4x4 tile of groups (I, J):
// A = the S values of group I, B = the AS (or S) values of group J.  A stage
// of 16 points is TG loads of S and TG of AS per lane, TG^2 + TG(TG+1)/2
// MFMAs.  The four blocks are summed across lanes at the end, then the four
// waves, in fixed order.
template <typename T, int TG>
__global__ void __launch_bounds__(kThreads) gram_kernel(GramArgs g) {
  typedef const __attribute__((address_space(1))) T* gptr;
  constexpr int NA = TG * TG, NB = TG * (TG + 1) / 2;
  constexpr int NS = 3;        // register stages (loads of the next two in flight)
  constexpr int FL = NS * 16;  // points of one loop trip
  __shared__ double red[4][NA + NB][16];
  if (g.active != nullptr && *g.active == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ns = g.ns, m = g.m;
  const int pl = lane >> 2, cl = lane & 3;

  // the S / AS column this lane feeds for group G; lanes past the last
  // column read column 0 and feed zeros as A operands
  gptr sp[TG], ap[TG];
  float lv[TG];
#pragma unroll
  for (int G = 0; G < TG; ++G) {
    const int c = 4 * G + cl;
    const bool live = c < ns;
    const int cc = live ? c : 0;
    const int b = cc / m, j = cc - (cc / m) * m;
    sp[G] = (gptr)g.S[b] + j;
    ap[G] = (gptr)g.AS[b] + j;
    lv[G] = live ? 1.0f : 0.0f;
  }

  const int64_t nw = (int64_t)gridDim.x * 4;
  const int64_t wid = (int64_t)blockIdx.x * 4 + wave;
  int64_t chunk = (g.n + nw - 1) / nw;
  chunk = (chunk + FL - 1) / FL * FL;
  const int64_t p_begin = wid * chunk;
  const int64_t p_end = (p_begin + chunk < g.n) ? p_begin + chunk : g.n;

  double acca[NA], accb[NB];
#pragma unroll
  for (int t = 0; t < NA; ++t) acca[t] = 0.0;
#pragma unroll
  for (int t = 0; t < NB; ++t) accb[t] = 0.0;

  // loads are unconditional (a point past the end re-reads p_begin); its
  // 0/1 mask multiplies only the A operands, when the stage's MFMAs run
  auto load = [&](int64_t p0, T (&sv)[TG], T (&av)[TG], T& mk) {
    const int64_t p = p0 + pl;
    const bool ok = p < p_end;
    const int64_t off = (ok ? p : p_begin) * m;
#pragma unroll
    for (int G = 0; G < TG; ++G) {
      sv[G] = sp[G][off];
      av[G] = ap[G][off];
    }
    mk = ok ? T(1) : T(0);
  };
  auto mfmas = [&](const T (&sv)[TG], const T (&av)[TG], T mk) {
    double sa[TG], sb[TG], ab[TG];
#pragma unroll
    for (int G = 0; G < TG; ++G) {
      sa[G] = (double)(sv[G] * (mk * (T)lv[G]));
      sb[G] = (double)sv[G];
      ab[G] = (double)av[G];
    }
#pragma unroll
    for (int I = 0; I < TG; ++I)
#pragma unroll
      for (int J = 0; J < TG; ++J) acca[I * TG + J] = mfma4(sa[I], ab[J], acca[I * TG + J]);
#pragma unroll
    for (int I = 0; I < TG; ++I)
#pragma unroll
      for (int J = I; J < TG; ++J) accb[tile_b<TG>(I, J)] = mfma4(sa[I], sb[J], accb[tile_b<TG>(I, J)]);
  };

  if (p_begin < p_end) {
    T sv[NS][TG], av[NS][TG], mk[NS];
#pragma unroll
    for (int q = 0; q < NS - 1; ++q) load(p_begin + (int64_t)q * 16, sv[q], av[q], mk[q]);
    for (int64_t pf = p_begin; pf < p_end; pf += FL) {
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        // refill the slot the previous stage's MFMAs consumed; the scheduling
        // barriers keep each stage's loads ahead of the other stages' MFMAs
        const int lq = (q + NS - 1) % NS;
        load(pf + (int64_t)(q + NS - 1) * 16, sv[lq], av[lq], mk[lq]);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(sv[q], av[q], mk[q]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // blocks q = 0..3 (lanes 4q apart within each row of 16) summed as
  // (q0 + q1) + (q2 + q3); lane 16i + j then holds D[i][j]
#pragma unroll
  for (int t = 0; t < NA + NB; ++t) {
    double v = t < NA ? acca[t] : accb[t - NA];
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    if ((lane & 12) == 0) red[wave][t][4 * (lane >> 4) + cl] = v;
  }
  __syncthreads();

  // the 16x16 output tiles: entry (row, col) of GB or GA from its 4x4 tile,
  // the lower S^T S tiles as mirrors of the upper ones (the same products in
  // the same order); the four waves in order.  Entries past ns are neither
  // written nor read by the reductions.
  const int nt = (ns + 15) >> 4;
  const int ntot = n_tiles_b(nt) + n_tiles_a(nt);
  for (int e = threadIdx.x; e < ntot * 256; e += kThreads) {
    bool isb;
    int row, col;
    tile_entry(e, nt, isb, row, col);
    if (row >= ns || col >= ns) continue;
    const int GI = row >> 2, GJ = col >> 2;
    int t, sub;
    if (!isb) {
      t = GI * TG + GJ;
      sub = 4 * (row & 3) + (col & 3);
    } else if (GI <= GJ) {
      t = NA + tile_b<TG>(GI, GJ);
      sub = 4 * (row & 3) + (col & 3);
    } else {
      t = NA + tile_b<TG>(GJ, GI);
      sub = 4 * (col & 3) + (row & 3);
    }
    const double sm = red[0][t][sub] + red[1][t][sub] + red[2][t][sub] + red[3][t][sub];
    g.partials[(size_t)blockIdx.x * ntot * 256 + e] = sm;
  }
}

// ---------------------------------------------------------------------------
// Rayleigh-Ritz on one workgroup of four waves (FP64)
// ---------------------------------------------------------------------------
// Every phase is a chain of dependent FP64 operations, and the step runs once
// per iteration between kernels that evict its code from the instruction
// cache, so straight-line code costs about twice its issue time (measured in
// place against back-to-back launches: about 50 cycles per 64 bytes).  The
// phases therefore spread each matrix over all 256 threads (thread (tr, tc) of
// a 16 x 16 grid owns entry (tr, tc), and three more above 16 columns) and
// loop over columns instead of being unrolled; rows of 16 lanes are DPP rows,
// so row sums need no LDS; and every padded size is a kernel of its own with
// everything inlined.  In place, per call: m = 4 (12 columns, with CG's update)
// 21.0 us, m = 3 FP64 (9) 17.8, m = 8 (24) 54.6, m = 1 (3) 8.1, against 39.9,
// 28.7, 90.6 and 12.8 for lane-per-row phases unrolled over the columns and
// called as functions (52 KB of code at 12 columns, 2.2 KB of scratch).
//
// Lanes of one wave issue their LDS accesses in program order and the LDS unit
// completes them in that order, so a store by one lane is seen by a later load
// of another lane of the same wave with no barrier, only a compiler-level
// fence that keeps LDS accesses in program order.
__device__ __forceinline__ void wave_fence() { __asm__ volatile("" ::: "memory"); }

// Reciprocal square root and reciprocal: the hardware approximation (a relative
// error e below 2^-20) and one step of third order, r (1 + e/2 + 3 e^2/8) and
// r (1 + e + e^2).  The product x r of the first is rounded: within 1 ulp, 0.27
// in the mean (the correctly rounded root and quotient of 1 / sqrt(x): 1.5 and
// 0.33); the second is correctly rounded but for ties (0.51 ulp).
__device__ __forceinline__ double rsq_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}
__device__ __forceinline__ double rcp_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
constexpr int KMAX = 24;
constexpr int LD = KMAX + 1;

struct RRShared {
  double A[2][KMAX * LD];  // double-buffered exchange copies of the matrices that are spread over the threads
  double B[2][KMAX * LD];
  double G[2][KMAX * LD];
  double pv[KMAX];         // M v of a reflector step
  double td[KMAX];         // the tridiagonal matrix
  double te[KMAX];
  double diag[KMAX];
  double Y[8][KMAX];       // eigenvectors of T
  double ev[8];
  double C[8][KMAX];       // the Ritz coefficients, before their signs
};

__device__ __forceinline__ double readlane_d(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
// Sum (maximum) over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_move<0x141>(v);  // row_half_mirror: the other quad of the half row
  v += dpp_move<0x140>(v);  // row_mirror: the other half of the row
  return v;
}
__device__ __forceinline__ double row_max(double v) {
  v = fmax(v, dpp_move<0xB1>(v));
  v = fmax(v, dpp_move<0x4E>(v));
  v = fmax(v, dpp_move<0x141>(v));
  return fmax(v, dpp_move<0x140>(v));
}
// The maximum over the wave's first KB lanes, in every lane; the lanes past the
// matrix, up to 31, repeat one of its rows.
template <int KB>
__device__ __forceinline__ double max_rows(double v) {
  v = row_max(v);
  if constexpr (KB <= 16) return readlane_d(v, 0);
  return fmax(readlane_d(v, 0), readlane_d(v, 16));
}

constexpr double kPadDiag = 1e4;  // diagonal of the padding rows: far above any eigenvalue of a T of norm below 1

// Number of eigenvalues of T below sigma: sign changes of the leading
// principal minors p_i of T - sigma I (Sturm), by the three-term recurrence
// p_i = (d_i - sigma) p_(i-1) - e_(i-1)^2 p_(i-2), no divisions.  A zero minor
// needs no case of its own: with every e^2 > 0 the minor after it has the sign
// opposite to the one before it, one change in all whichever sign the zero
// carries (e2 holds max(e^2, kMinE2); a coupling of 1e-30 moves no eigenvalue of
// a T whose norm is in [0.5, 1): the caller scales it).  With at most 24 rows the
// minors then stay within about 1e+-100 (the padding rows multiply by ~1e4
// each), so no rescaling is needed between them.
constexpr double kMinE2 = 1e-60;
// A coupling below this is none to the inverse iteration: as a pivot, 1e140 in
// the back substitution, it overflowed the vector's norm.
constexpr double kNoCoupling = 1e-100;
template <int KB>
__device__ __forceinline__ int sturm_count(const double (&d)[KB], const double (&e2)[KB], double sigma) {
  double pm2 = 1.0, pm1 = d[0] - sigma;
  // the minors' sign bits, shifted in one after the other (below p_0 = 1)
  unsigned signs = (unsigned)__double2hiint(pm1) >> 31;
#pragma unroll
  for (int i = 1; i < KB; ++i) {
    const double p = fma(d[i] - sigma, pm1, -e2[i - 1] * pm2);
    signs = __builtin_amdgcn_alignbit(signs, (unsigned)__double2hiint(p), 31);
    pm2 = pm1;
    pm1 = p;
  }
  return __popc(signs ^ (signs >> 1));
}

// Entries of a thread: rows tr + 16 i, columns tc + 16 j
template <int KB>
struct RRGrid {
  static constexpr int E = KB > 16 ? 2 : 1;
  // a thread's entries into an exchange copy (entries past the arrays are dropped)
  static __device__ __forceinline__ void store(double* dst, const double (&v)[E][E], int tr, int tc) {
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
      for (int j = 0; j < E; ++j)
        if (E == 1 || (tr + 16 * i < KMAX && tc + 16 * j < KMAX)) dst[(tr + 16 * i) * LD + tc + 16 * j] = v[i][j];
  }
};

// Elimination of the scaled B with column dropping (B = L D L^T on the kept
// columns, L unit lower triangular), the same elementary steps on both sides
// of the scaled A, which leaves L^-1 A L^-T, and on the right of the identity
// g, which leaves L^-T: step k takes row k of both matrices (symmetric: also
// column k) and m_c = B_kc / B_kk for c > k, and subtracts m_r B_kc from B,
// m_r A_kc + m_c (A_kr - m_r A_kk) from A and m_c g_rk from g.  A column whose
// pivot is at most drop_tol, or not a number, is left out: no entry of another
// column is touched (zero factors would carry a NaN on).
// Every thread stores its entries after a step (double-buffered: one barrier
// per column), which takes fewer instructions than choosing the row's owners.
// Returns the kept columns; their pivots in sh.diag.
template <int KB>
__device__ __forceinline__ unsigned rr_reduce(RRShared& sh, double (&a)[RRGrid<KB>::E][RRGrid<KB>::E],
                                              double (&b)[RRGrid<KB>::E][RRGrid<KB>::E],
                                              double (&g)[RRGrid<KB>::E][RRGrid<KB>::E], int ns, unsigned goodm,
                                              double drop_tol) {
  constexpr int E = RRGrid<KB>::E;
  const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;
  int ri[E], ci[E];  // this thread's rows and columns, clamped to the arrays
#pragma unroll
  for (int i = 0; i < E; ++i) {
    ri[i] = E == 1 || tr + 16 * i < KMAX ? tr + 16 * i : 0;
    ci[i] = E == 1 || tc + 16 * i < KMAX ? tc + 16 * i : 0;
#pragma unroll
    for (int j = 0; j < E; ++j) g[i][j] = tr + 16 * i == tc + 16 * j ? 1.0 : 0.0;
  }
  unsigned keptm = 0;
#pragma unroll 1
  for (int k = 0; k < ns; ++k) {
    RRGrid<KB>::store(sh.A[k & 1], a, tr, tc);
    RRGrid<KB>::store(sh.B[k & 1], b, tr, tc);
    RRGrid<KB>::store(sh.G[k & 1], g, tr, tc);
    __syncthreads();
    const double *ra = sh.A[k & 1] + k * LD, *rb = sh.B[k & 1] + k * LD, *cg = sh.G[k & 1] + k;
    const double piv = rb[k], akk = ra[k];
    double br[E], bc[E], ar[E], ac[E], gr[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      br[i] = rb[ri[i]];
      bc[i] = rb[ci[i]];
      ar[i] = ra[ri[i]];
      ac[i] = ra[ci[i]];
      gr[i] = cg[ri[i] * LD];
    }
    const bool keep = __ballot(((goodm >> k) & 1u) && piv > drop_tol) != 0;  // (every thread alike)
    if (!keep) continue;
    keptm |= 1u << k;
    const double rp = rcp_nr(piv);
    double mr[E], mc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      mr[i] = tr + 16 * i > k ? br[i] * rp : 0.0;
      mc[i] = tc + 16 * i > k ? bc[i] * rp : 0.0;
    }
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
      for (int j = 0; j < E; ++j) {
        b[i][j] = fma(-mr[i], bc[j], b[i][j]);
        a[i][j] = fma(-mr[i], ac[j], fma(-mc[j], fma(-mr[i], akk, ar[i]), a[i][j]));
        g[i][j] = fma(-mc[j], gr[i], g[i][j]);
      }
  }
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (tr == tc && ri[i] == tr + 16 * i) sh.diag[ri[i]] = b[i][i];
  return keptm;
}

// Householder tridiagonalisation T = Q^T M Q of the K x K matrix spread over
// the threads (a; zero past K): T into sh.td, sh.te; the reflectors are applied
// to g from the right as they come (g Q, row sums only).  Two barriers per
// column: for the matrix, of which the rows j and j + 1 are read, and for M v.
// With v = x - alpha e_(j+1), M v = M x - alpha M e_(j+1), so that M x is
// summed beside |x|^2.
template <int KB>
__device__ __forceinline__ void rr_tridiagonalize(RRShared& sh, double (&a)[RRGrid<KB>::E][RRGrid<KB>::E],
                                                  double (&g)[RRGrid<KB>::E][RRGrid<KB>::E], int K) {
  constexpr int E = RRGrid<KB>::E;
  const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;
  int ri[E], ci[E];
  bool rin[E], cin[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    rin[i] = E == 1 || tr + 16 * i < KMAX;
    cin[i] = E == 1 || tc + 16 * i < KMAX;
    ri[i] = rin[i] ? tr + 16 * i : 0;
    ci[i] = cin[i] ? tc + 16 * i : 0;
  }
#pragma unroll 1
  for (int j = 0; j + 2 < K; ++j) {
    RRGrid<KB>::store(sh.A[0], a, tr, tc);
    __syncthreads();
    const double* row = sh.A[0] + j * LD;
    double vr[E], vc[E], nr[E], pr[E], pc[E], mx[E];
    double s2 = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      vr[i] = row[ri[i]];
      vc[i] = row[ci[i]];
      nr[i] = row[LD + ri[i]];
    }
    const double x0 = row[j + 1];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      vr[i] = rin[i] && tr + 16 * i > j ? vr[i] : 0.0;
      vc[i] = cin[i] && tc + 16 * i > j ? vc[i] : 0.0;
      s2 = fma(vc[i], vc[i], s2);
    }
    s2 = row_sum(s2);
#pragma unroll
    for (int i = 0; i < E; ++i) {
      double p = 0.0;
#pragma unroll
      for (int q = 0; q < E; ++q) p = fma(a[i][q], vc[q], p);
      mx[i] = row_sum(p);
    }
    // |x| = s2 / sqrt(s2)
    const double nrm = s2 > 0.0 ? s2 * rsq_nr(s2) : 0.0;
    const double alpha = x0 >= 0.0 ? -nrm : nrm;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      // (M v)_r; zero in the rows that are already tridiagonal
      pr[i] = rin[i] && tr + 16 * i > j ? fma(-alpha, nr[i], mx[i]) : 0.0;
      if (rin[i]) sh.pv[ri[i]] = pr[i];  // (the row's 16 lanes alike)
      if (tr + 16 * i == j + 1) vr[i] = x0 - alpha;
      if (tc + 16 * i == j + 1) vc[i] = x0 - alpha;
    }
    sh.te[j] = alpha;  // (every thread alike)
    // beta = 2 / v^T v = 1 / (s2 - alpha x0)
    const double hv = fma(-alpha, x0, s2);
    const double beta = hv > 0.0 ? rcp_nr(hv) : 0.0;
    // g (I - beta v v^T)
#pragma unroll
    for (int i = 0; i < E; ++i) {
      double p = 0.0;
#pragma unroll
      for (int q = 0; q < E; ++q) p = fma(g[i][q], vc[q], p);
      p = -beta * row_sum(p);
#pragma unroll
      for (int q = 0; q < E; ++q) g[i][q] = fma(p, vc[q], g[i][q]);
    }
    __syncthreads();
    double kc = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      pc[i] = cin[i] ? sh.pv[ci[i]] : 0.0;
      kc = fma(vc[i], pc[i], kc);
    }
    // M - v w^T - w v^T with w = beta M v - (beta^2 / 2) (v^T M v) v, one beta
    // after the other (their square overflows for a coupling below 1e-77)
    kc = 0.5 * beta * (beta * row_sum(kc));
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const double wr = fma(-kc, vr[i], beta * pr[i]), wc = fma(-kc, vc[q], beta * pc[q]);
        a[i][q] = fma(-vr[i], wc, fma(-wr, vc[q], a[i][q]));
      }
  }
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int r = tr + 16 * i, c = tc + 16 * q;
      if (r == c && r < K) sh.td[r] = a[i][q];
      if (r == K - 1 && c == K - 2) sh.te[c] = a[i][q];
    }
  __syncthreads();
}

// Eigenvalues t = wave (and wave + 4 for m > 4) of T into sh.ev[t], their
// eigenvectors into sh.Y[t], every wave its own: multisection bisection of the
// Sturm count (the wave's 64 lanes, 32 for m > 4, evaluate it at evenly spaced
// shifts of the bracket, which shrinks by 65 (33) per round, down to 2^-60 of
// the Gershgorin interval), then two steps of inverse iteration from a fixed
// start vector (Gaussian elimination with partial pivoting of T - lambda I in
// registers).  T is taken at a norm in [0.5, 1), by an exact power of two: the
// counts and the padding hold at any scale of the pencil (a graph of weights of
// 1e-30, say).  Rows past K are padded with a diagonal far above the spectrum.
template <int KB>
__device__ __forceinline__ void rr_eig_pairs(RRShared& sh, int K, int m) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double d[KB], e2[KB], eo[KB];
  double lo, hi, tnorm, unit;
  {
    // Gershgorin, lane = row (lanes past K repeat row 0)
    const int i = lane < K ? lane : 0;
    const double r = (i + 1 < K ? fabs(sh.te[i]) : 0.0) + (i > 0 ? fabs(sh.te[i > 0 ? i - 1 : 0]) : 0.0);
    const double di = sh.td[i];
    lo = -max_rows<KB>(r - di);
    hi = max_rows<KB>(di + r);
    tnorm = fmax(fabs(lo), fabs(hi));
    const int ex = __builtin_amdgcn_frexp_exp(tnorm);  // 0 for a zero or non-finite norm
    const int e = ex < -1000 ? -1000 : (ex > 1000 ? 1000 : ex);
    unit = ldexp(1.0, e);
    const double inv = ldexp(1.0, -e);
    lo *= inv;
    hi *= inv;
    tnorm *= inv;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      d[k] = k < K ? sh.td[k] * inv : kPadDiag;
      const double o = k + 1 < K ? sh.te[k] * inv : 0.0;  // T[k+1][k] = T[k][k+1]
      eo[k] = fabs(o) < kNoCoupling ? 0.0 : o;
      e2[k] = fmax(eo[k] * eo[k], kMinE2);
    }
  }
  const int half = m > 4 ? 1 : 0;            // two eigenvalues per wave
  const int G = half ? 32 : 64;              // lanes per eigenvalue
  const int rounds = half ? 12 : 10;         // 33^12, 65^10 > 2^60
  const int sub = half ? (lane >> 5) : 0;
  const int t = wave + 4 * sub;              // this lane's eigenvalue (t >= m: idle copy)
  const int tc = t < m ? t : m - 1;
  const int s = lane & (G - 1);
  const double pad = 1e-14 * tnorm + 1e-300;
  lo -= pad;
  hi += pad;
#pragma unroll 1
  for (int rnd = 0; rnd < rounds; ++rnd) {
    const double step = (hi - lo) * (half ? 1.0 / 33.0 : 1.0 / 65.0);
    const double sig = fma((double)(s + 1), step, lo);
    const int c = sturm_count<KB>(d, e2, sig);
    const unsigned long long bal = __ballot(c <= tc);
    const unsigned long long grp = half ? ((bal >> (32 * sub)) & 0xFFFFFFFFull) : bal;
    const int top = grp ? 63 - __clzll(grp) : -1;  // highest shift whose count is <= t
    const double nlo = top >= 0 ? fma((double)(top + 1), step, lo) : lo;
    const double nhi = top + 1 < G ? fma((double)(top + 2), step, lo) : hi;
    lo = nlo;
    hi = nhi;
  }
  const double lam = 0.5 * (lo + hi);
  const double ptiny = 1e-16 * (tnorm > 0.0 ? tnorm : 1.0);
  // elimination: one reciprocal per row, of the pivot (kept away from zero),
  // which the multiplier divides by and the back substitution as well (u0)
  double u0[KB], u1[KB], u2[KB], f[KB], y[KB];
  bool sw[KB];
  auto off_zero = [&](double v) {
    const double w = fmax(fabs(v), ptiny);
    return __hiloint2double(__double2hiint(w) | (__double2hiint(v) & 0x80000000), __double2loint(w));
  };
  {
    double c0 = d[0] - lam, c1 = eo[0];
#pragma unroll
    for (int i = 0; i + 1 < KB; ++i) {
      const double sb = eo[i], dn = d[i + 1] - lam, sp = i + 1 < KB - 1 ? eo[i + 1] : 0.0;
      sw[i] = fabs(sb) > fabs(c0);
      const double r = rcp_nr(sw[i] ? sb : off_zero(c0));
      const double fi = (sw[i] ? c0 : sb) * r;
      u0[i] = r;
      u1[i] = sw[i] ? dn : c1;
      u2[i] = sw[i] ? sp : 0.0;
      f[i] = fi;
      c0 = fma(-fi, u1[i], sw[i] ? c1 : dn);
      c1 = sw[i] ? -fi * sp : sp;
    }
    u0[KB - 1] = rcp_nr(off_zero(c0));
    u1[KB - 1] = 0.0;
    u2[KB - 1] = 0.0;
    f[KB - 1] = 0.0;
    sw[KB - 1] = false;
  }
  // start vectors that differ between the eigenvalues (of a cluster)
#pragma unroll
  for (int i = 0; i < KB; ++i) y[i] = fma(0.0625, (double)((3 * i + 5 * tc) & 7), 0.75);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    // (the running element in a variable of its own: a choice between two
    // elements of y became an indexed read, a chain of selects over all of y)
    double cur = y[0];
#pragma unroll
    for (int i = 0; i + 1 < KB; ++i) {
      const double nx = y[i + 1];
      const double ri = sw[i] ? nx : cur, rn = sw[i] ? cur : nx;
      y[i] = ri;
      cur = fma(-f[i], ri, rn);
    }
    y[KB - 1] = cur;
#pragma unroll
    for (int i = KB - 1; i >= 0; --i) {
      double v = y[i];
      if (i + 2 < KB) v = fma(-u2[i], y[i + 2], v);
      if (i + 1 < KB) v = fma(-u1[i], y[i + 1], v);
      y[i] = v * u0[i];
    }
    double n0 = 0.0, n1 = 0.0;
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      if (i & 1) n1 = fma(y[i], y[i], n1);
      else n0 = fma(y[i], y[i], n0);
    }
    const double sc = rsq_nr(n0 + n1);
#pragma unroll
    for (int i = 0; i < KB; ++i) y[i] *= sc;
  }
  if (s == 0 && t < m) {
    sh.ev[t] = lam * unit;
#pragma unroll
    for (int i = 0; i < KB; ++i) sh.Y[t][i] = i < K ? y[i] : 0.0;
    if constexpr (KB < KMAX)
      for (int i = KB; i < KMAX; ++i) sh.Y[t][i] = 0.0;
  }
}

// Orthonormal sh.Y[0..m) on wave 0: lane group g (16 lanes, one DPP row) holds
// the vectors g and g + 4, lane l of it the rows l and l + 16.  The unit
// vectors of separated eigenvalues come out of the inverse iteration
// orthogonal to about 1e-16 / gap: with every dot product d below 1e-9 one
// correction y_q - sum_(p < q) d_pq y_p, all pairs at once, leaves d^2.
// Otherwise (a cluster) modified Gram-Schmidt, a second pass of it if a vector
// had a component of more than 1e-2 along an earlier one.
template <int KB>
__device__ __forceinline__ void rr_orthonormalize(RRShared& sh, int m) {
  constexpr int E = RRGrid<KB>::E;
  const int lane = threadIdx.x & 63, g = lane >> 4, l = lane & 15;
  double z[2][E];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int q = g + 4 * u, r = l + 16 * i;
      z[u][i] = (q < m && r < KMAX) ? sh.Y[q < m ? q : 0][r < KMAX ? r : 0] : 0.0;
    }
  {
    double worst = 0.0, cz[2][E];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < E; ++i) cz[u][i] = z[u][i];
#pragma unroll
    for (int p = 0; p < 7; ++p) {
      if (p + 1 >= m) break;
      double zp[E];
#pragma unroll
      for (int i = 0; i < E; ++i) zp[i] = l + 16 * i < KMAX ? sh.Y[p][l + 16 * i < KMAX ? l + 16 * i : 0] : 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u == 0 ? p >= 3 : m <= 4) continue;
        double dq = 0.0;
#pragma unroll
        for (int i = 0; i < E; ++i) dq = fma(z[u][i], zp[i], dq);
        dq = g + 4 * u > p ? row_sum(dq) : 0.0;
        worst = fmax(worst, fabs(dq));
#pragma unroll
        for (int i = 0; i < E; ++i) cz[u][i] = fma(-dq, zp[i], cz[u][i]);
      }
    }
    if (__ballot(!(worst <= 1e-9)) == 0) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < E; ++i)
          if (g + 4 * u < m && l + 16 * i < KMAX) sh.Y[g + 4 * u][l + 16 * i] = cz[u][i];
      return;
    }
  }
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    double worst = 0.0;
#pragma unroll 1
    for (int p = 0; p < m; ++p) {
      double zs[E], nq = 0.0;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        zs[i] = p >= 4 ? z[1][i] : z[0][i];
        nq = fma(zs[i], zs[i], nq);
      }
      const double sc = rsq_nr(row_sum(nq));
      if (g == (p & 3)) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
          zs[i] *= sc;
          if (p >= 4) z[1][i] = zs[i];
          else z[0][i] = zs[i];
          if (l + 16 * i < KMAX) sh.Y[p][l + 16 * i] = zs[i];
        }
      }
      wave_fence();
      double zp[E];
#pragma unroll
      for (int i = 0; i < E; ++i) zp[i] = l + 16 * i < KMAX ? sh.Y[p][l + 16 * i < KMAX ? l + 16 * i : 0] : 0.0;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = g + 4 * u;
        double dq = 0.0;
#pragma unroll
        for (int i = 0; i < E; ++i) dq = fma(z[u][i], zp[i], dq);
        dq = row_sum(dq);
        if (q > p && q < m) {
          worst = fmax(worst, fabs(dq));
#pragma unroll
          for (int i = 0; i < E; ++i) z[u][i] = fma(-dq, zp[i], z[u][i]);
        }
        if (m <= 4) break;
      }
    }
    if (__ballot(worst > 1e-2) == 0) break;
  }
}

// C = delta (L^-T Q) Y with g = L^-T Q spread over the threads (row sums), then
// per column the largest-magnitude coefficient (the first on ties) made
// positive, so that Ritz vectors (and residuals) have a fixed sign for a
// non-odd T.  Rows of dropped columns hold zeros in g.
template <int KB>
__device__ __forceinline__ void rr_output(RRShared& sh, const double (&g)[RRGrid<KB>::E][RRGrid<KB>::E],
                                          const double (&dr)[RRGrid<KB>::E], int ns, int m, double* Cout,
                                          double* theta) {
  constexpr int E = RRGrid<KB>::E;
  const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;
#pragma unroll
  for (int t = 0; t < (KB < 8 ? KB : 8); ++t) {
    if (t >= m) break;
    double y[E];
#pragma unroll
    for (int q = 0; q < E; ++q) y[q] = sh.Y[t][tc + 16 * q < KMAX ? tc + 16 * q : KMAX - 1];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < E; ++q) v = fma(g[i][q], y[q], v);
      v = dr[i] * row_sum(v);
      if (tc == 0 && tr + 16 * i < KMAX) sh.C[t][tr + 16 * i] = v;
    }
  }
  __syncthreads();
  // thread (t, l) of the first 128: rows l and l + 16 of column t
  const int t = threadIdx.x >> 4, l = threadIdx.x & 15;
  if (t < 8) {
    double v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = t < m && l + 16 * i < ns ? sh.C[t][l + 16 * i < KMAX ? l + 16 * i : 0] : 0.0;
    const double big = row_max(fmax(fabs(v[0]), fabs(v[1])));
    const unsigned at = (unsigned)(__ballot(fabs(v[0]) == big) >> (threadIdx.x & 48)) & 0xFFFFu;
    const unsigned at2 = (unsigned)(__ballot(fabs(v[1]) == big) >> (threadIdx.x & 48)) & 0xFFFFu;
    const int first = at ? __ffs(at) - 1 : 15 + __ffs(at2);
    const double lead = t < m && first < ns ? sh.C[t][first] : 0.0;
    const int flip = __double2hiint(lead) & 0x80000000;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (t < m && l + 16 * i < ns)
        Cout[(l + 16 * i) * m + t] = __hiloint2double(__double2hiint(v[i]) ^ flip, __double2loint(v[i]));
    if (t < m && l == 0) theta[t] = sh.ev[t];
  }
}

// Solves the Rayleigh-Ritz problem for the Gram pair GA, GB (ns x ns), spread
// over the 256 threads of the workgroup (ga, gb; every thread must call it):
// C (ns x m, row-major with leading dimension m) and theta (ascending) of the
// m smallest Ritz pairs.  Steps: symmetrise; scale to unit diag(GB) (columns
// with a negligible diagonal are dropped); elimination GB = L D L^T that drops
// columns with a pivot at most drop_tol, and M = D^-1/2 L^-1 GA L^-T D^-1/2 on the
// kept columns; the m smallest eigenpairs Z of M (tridiagonalisation, bisection,
// inverse iteration); C = L^-T D^-1/2 Z.  Returns the kept columns; with fewer than m
// of them nothing is written.
template <int KB>
__device__ __forceinline__ unsigned rayleigh_ritz(RRShared& sh, const double (&ga)[RRGrid<KB>::E][RRGrid<KB>::E],
                                                  const double (&gb)[RRGrid<KB>::E][RRGrid<KB>::E], int ns, int m,
                                                  double drop_tol, double zero_tol, double* Cout, double* theta) {
  constexpr int E = RRGrid<KB>::E;
  const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int r = tr + 16 * i, c = tc + 16 * j;
      if (r < ns && c < ns) {
        sh.A[1][r * LD + c] = ga[i][j];
        sh.B[1][r * LD + c] = gb[i][j];
        if (r == c) sh.diag[r] = gb[i][j];
      }
    }
  __syncthreads();
  // unit-diagonal scaling: delta_j = diag(GB)_j^-1/2, 0 for a negligible column
  double dc[E], dr[E], mx = 0.0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int r = tr + 16 * i, c = tc + 16 * i;
    dr[i] = r < ns ? sh.diag[r < ns ? r : 0] : 0.0;
    dc[i] = c < ns ? sh.diag[c < ns ? c : 0] : 0.0;
    mx = fmax(mx, dc[i] > 0.0 ? dc[i] : 0.0);
  }
  const double least = zero_tol * zero_tol * row_max(mx);
  unsigned goodm = 0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    goodm |= (unsigned)(__ballot(dc[i] > least) & 0xFFFFull) << (16 * i);
    dc[i] = dc[i] > least ? rsq_nr(dc[i]) : 0.0;
    dr[i] = dr[i] > least ? rsq_nr(dr[i]) : 0.0;
  }
  double a[E][E], b[E][E];
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int r = tr + 16 * i, c = tc + 16 * j;
      // (a negligible or non-finite column is zeros)
      const bool in = ((goodm >> r) & 1u) && ((goodm >> c) & 1u);
      const double at = sh.A[1][in ? c * LD + r : 0], bt = sh.B[1][in ? c * LD + r : 0];
      const double sc = dr[i] * dc[j];
      a[i][j] = in ? (r == c ? ga[i][j] : 0.5 * (ga[i][j] + at)) * sc : 0.0;
      b[i][j] = in ? (r == c ? gb[i][j] : 0.5 * (gb[i][j] + bt)) * sc : 0.0;
    }
  double gm[E][E];
  const unsigned keptm = rr_reduce<KB>(sh, a, b, gm, ns, goodm, drop_tol);
  const int K = __popc(keptm);
  if (K < m) return keptm;
  // the kept columns moved together and scaled by D^-1/2: M symmetrised, L^-T
  // with zero rows at the dropped columns
  auto rank = [&](int r) { return __popc(keptm & ((1u << r) - 1u)); };
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int r = tr + 16 * i, c = tc + 16 * j;
      const bool kr = (keptm >> r) & 1u, kc = (keptm >> c) & 1u;
      const double sr = kr ? rsq_nr(sh.diag[r]) : 0.0, scl = kc ? rsq_nr(sh.diag[c]) : 0.0;
      if (kr && kc) sh.A[0][rank(r) * LD + rank(c)] = a[i][j] * (sr * scl);
      if (r < ns && kc) sh.G[0][r * LD + rank(c)] = kr ? gm[i][j] * scl : 0.0;
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int r = tr + 16 * i, c = tc + 16 * j;
      a[i][j] = r < K && c < K ? 0.5 * (sh.A[0][r * LD + c] + sh.A[0][c * LD + r]) : 0.0;
      gm[i][j] = r < ns && c < K ? sh.G[0][r * LD + c] : 0.0;
    }
  __syncthreads();
  rr_tridiagonalize<KB>(sh, a, gm, K);
  rr_eig_pairs<KB>(sh, K, m);
  __syncthreads();
  if (threadIdx.x < 64) rr_orthonormalize<KB>(sh, m);
  __syncthreads();
  rr_output<KB>(sh, gm, dr, ns, m, Cout, theta);
  return keptm;
}

// The previous update's residual sums (|R_j|^2 for j < m, summed over its
// workgroup partials in workgroup order) into fin[0..7], for the
// Rayleigh-Ritz step that finalizes them; one workgroup.
__device__ void fin_reduce(const RRArgs& r, int m, double* fin) {
  __shared__ double fred[8 * 16];
  double t[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) t[k] = 0.0;
  for (int b0 = 0; b0 < r.fin_nparts; b0 += 4 * (int)blockDim.x) {
    double fv[4][8];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int b = b0 + it * (int)blockDim.x + (int)threadIdx.x;
      const int bb = b < r.fin_nparts ? b : 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) fv[it][k] = r.fin_partials[(size_t)bb * r.fin_stride + (k < m ? k : 0)];
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const bool ok = b0 + it * (int)blockDim.x + (int)threadIdx.x < r.fin_nparts;
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] += (ok && k < m) ? fv[it][k] : 0.0;
    }
  }
  block_sum<8>(t, fred);
  if (threadIdx.x == 0)
    for (int k = 0; k < 8; ++k) fin[k] = t[k];
}

// First stage of the Gram reduction: workgroup (tile, chunk) sums the partials
// of its chunk of Gram workgroups for the 256 entries of one tile; the
// workgroup column after the tiles reduces the previous update's residual
// partials for the Rayleigh-Ritz step, off its critical path.
__global__ void __launch_bounds__(kThreads) gram_reduce_kernel(GramArgs g, RRArgs r) {
  const int ntiles = n_tiles_b((g.ns + 15) >> 4) + n_tiles_a((g.ns + 15) >> 4);
  if (g.active != nullptr && *g.active == 0) return;
  if ((int)blockIdx.x == ntiles) {
    if (blockIdx.y == 0 && r.fin_partials != nullptr) fin_reduce(r, g.m, g.level2 + kGramFinSlot);
    return;
  }
  const int nt = (g.ns + 15) >> 4;
  const int ntot = n_tiles_b(nt) + n_tiles_a(nt);
  const int tile = blockIdx.x, chunk = blockIdx.y, nchunks = gridDim.y;
  const int per = (g.nparts + nchunks - 1) / nchunks;
  const int b0 = chunk * per, b1 = (b0 + per < g.nparts) ? b0 + per : g.nparts;
  const int e = tile * 256 + threadIdx.x;
  const size_t st = (size_t)ntot * 256;
  {
    bool isb;
    int row, col;
    tile_entry(e, nt, isb, row, col);
    if (row >= g.ns || col >= g.ns) return;  // not written by the Gram kernel, not read
  }
  // up to kGramPerChunk partials, loaded together, summed in order
  double v[kGramPerChunk];
#pragma unroll
  for (int k = 0; k < kGramPerChunk; ++k) v[k] = (b0 + k < b1) ? g.partials[(size_t)(b0 + k) * st + e] : 0.0;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kGramPerChunk; ++k) s += v[k];
  g.level2[(size_t)chunk * st + e] = s;
}

// Workgroup 0: sums the chunks of its threads' Gram entries (the 16 x 16 tile
// format is the thread grid of the Rayleigh-Ritz step) and runs the step.
// Workgroups 1.. (cg.nblk of them) run a CG update phase of the joint driver
// on the CUs the step leaves idle.
//
// direct != 0 (at most kGramDirect Gram workgroups): no
// reduction launch ran; the partials take the place of the chunk sums (the
// reduction would have copied them one to one, so the sums are bitwise the
// same) and this workgroup sums the previous update's residual partials.
template <int KB>
__global__ void __launch_bounds__(kThreads) gram_rr_kernel(GramArgs g, RRArgs r, CgStepArgs cg, int direct) {
  if (blockIdx.x > 0) {
    cg_aupdate_step(cg, (int)blockIdx.x - 1);
    return;
  }
  constexpr int E = RRGrid<KB>::E;
  constexpr int NT = KB <= 16 ? 2 : 7;  // tiles of the Gram pair
  __shared__ RRShared sh;
  __shared__ int live;
  // Everything this kernel reads from global memory was written by earlier
  // kernels (other XCDs), so each load is a long trip: the chunk values, the
  // solver state and the residual sums are all issued before any of them is
  // used (also before the state says whether the step runs at all).
  const double* chunks = direct ? g.partials : g.level2;
  const int nchunks = direct ? g.nparts : kGramChunks;
  const int tr = threadIdx.x >> 4, tc = threadIdx.x & 15;
  // tile and entry of this thread's entries: GB's lower off-diagonal tile is
  // the mirror of the upper one
  auto sum = [&](int tile, int e) {
    double v[kGramDirect], t = 0.0;
#pragma unroll
    for (int c = 0; c < kGramDirect; ++c) v[c] = c < nchunks ? chunks[(size_t)c * (NT * 256) + tile * 256 + e] : 0.0;
#pragma unroll
    for (int c = 0; c < kGramDirect; ++c) t += v[c];
    return t;
  };
  double ga[E][E], gb[E][E];
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const bool mirror = i > j;
      gb[i][j] = sum(E == 1 ? 0 : (mirror ? 1 : i + j), mirror ? tc * 16 + tr : (int)threadIdx.x);
      ga[i][j] = sum(E == 1 ? 1 : 3 + 2 * i + j, threadIdx.x);
    }
  LobpcgState* st = r.st;
  const int active = st != nullptr ? st->active : 1;
  const double tol = st != nullptr ? st->tol : 0.0;
  const int iters0 = st != nullptr ? st->iters : 0;
  const int dropped0 = st != nullptr ? st->dropped : 0;
  if (!active) return;
  if (r.fin_partials != nullptr) {
    // the previous update's residual norms, iteration count and convergence
    // test (what lob_final_kernel does after an update without the
    // constraint, in the same summation order); the sums come reduced from
    // gram_reduce_kernel's extra workgroup, or from this workgroup (direct)
    __shared__ double fin_here[8];
    if (direct) fin_reduce(r, g.m, fin_here);
    const double* fin = direct ? fin_here : g.level2 + kGramFinSlot;
    double t[8];
    if (threadIdx.x == 0)
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] = fin[k];
    if (threadIdx.x == 0) {
      double mx = 0.0;
      for (int j = 0; j < g.m; ++j) {
        const double rj = sqrt(t[j]);
        st->res[j] = rj;
        st->yx[j] = 0.0;
        mx = rj > mx ? rj : mx;
      }
      st->iters = iters0 + 1;
      live = !(tol > 0.0 && mx <= tol);
      if (!live) st->active = 0;
    }
    // (a run without a tolerance is always live: its other waves go on)
    if (tol > 0.0) {
      __syncthreads();
      if (!live) return;
    }
  }
  // soft locking (tol > 0): a column whose residual is already at the
  // tolerance adds no search direction, i.e. its W column counts as zero:
  // the W rows and columns of both Gram matrices are cleared, and the
  // Rayleigh-Ritz step drops the column
  if (!r.init && st != nullptr && tol > 0.0 && g.ns > g.m) {
    __shared__ int lockm;
    if (threadIdx.x == 0) {
      int mask = 0;
      for (int j = 0; j < g.m; ++j)
        if (st->res[j] <= tol) mask |= 1 << j;
      lockm = mask << g.m;
    }
    __syncthreads();
    const int lk = lockm;
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
      for (int j = 0; j < E; ++j)
        if (((lk >> (tr + 16 * i)) & 1) || ((lk >> (tc + 16 * j)) & 1)) ga[i][j] = gb[i][j] = 0.0;
  }
  if (r.gram_out != nullptr) {
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int row = tr + 16 * i, col = tc + 16 * j;
        if (row < g.ns && col < g.ns) {
          r.gram_out[row * g.ns + col] = ga[i][j];
          r.gram_out[g.ns * g.ns + row * g.ns + col] = gb[i][j];
        }
      }
  }
  const unsigned kept = rayleigh_ritz<KB>(sh, ga, gb, g.ns, g.m, r.drop_tol, r.zero_tol, r.C, r.theta);
  const int nkept = __popc(kept);
  if (st != nullptr) {
    if ((int)threadIdx.x < g.ns) st->kept[threadIdx.x] = (kept >> threadIdx.x) & 1u;
    if (nkept >= g.m && (int)threadIdx.x < g.m) st->theta[threadIdx.x] = sh.ev[threadIdx.x];
    if (threadIdx.x == 0) {
      st->nkept = nkept;
      st->dropped = dropped0 + g.ns - nkept;
      if (nkept < g.m) {
        st->status = GSF_EBREAKDOWN;
        st->active = 0;
        if (r.init) st->start_failed = 1;
      }
    }
  }
  if (r.kept_out != nullptr && (int)threadIdx.x < g.ns) r.kept_out[threadIdx.x] = (kept >> threadIdx.x) & 1u;
  if (r.nkept_out != nullptr && threadIdx.x == 0) *r.nkept_out = nkept;
}

// Runs f<KB> for the smallest padded size KB >= ns (the eigenvalue part of the
// step is unrolled over KB rows)
template <class F>
void rr_dispatch(int ns, F&& f) {
  if (ns <= 4) f(std::integral_constant<int, 4>{});
  else if (ns <= 8) f(std::integral_constant<int, 8>{});
  else if (ns <= 10) f(std::integral_constant<int, 10>{});
  else if (ns <= 12) f(std::integral_constant<int, 12>{});
  else if (ns <= 16) f(std::integral_constant<int, 16>{});
  else f(std::integral_constant<int, KMAX>{});
}

// ---------------------------------------------------------------------------
// update + next residual
// ---------------------------------------------------------------------------
// Row helpers: the M values of one point, as vector memory operations when
// the row is a whole number of 16-byte words.
template <typename T, int M>
__device__ __forceinline__ void load_row(const T* __restrict__ src, T (&v)[M]) {
  if constexpr (sizeof(T) * M % 16 == 0) {
    constexpr int W = (int)(sizeof(T) * M / 16);
    const float4* s4 = reinterpret_cast<const float4*>(src);
#pragma unroll
    for (int w = 0; w < W; ++w) reinterpret_cast<float4*>(v)[w] = s4[w];
  } else {
#pragma unroll
    for (int j = 0; j < M; ++j) v[j] = src[j];
  }
}

template <typename T, int M>
__device__ __forceinline__ void store_row(T* __restrict__ dst, const T (&v)[M]) {
  if constexpr (sizeof(T) * M % 16 == 0) {
    constexpr int W = (int)(sizeof(T) * M / 16);
    float4* d4 = reinterpret_cast<float4*>(dst);
#pragma unroll
    for (int w = 0; w < W; ++w) d4[w] = reinterpret_cast<const float4*>(v)[w];
  } else {
#pragma unroll
    for (int j = 0; j < M; ++j) dst[j] = v[j];
  }
}

// store_row as streaming (non-temporal) stores: for the blocks that are read
// again only after the next stencil pass (X, AX, P, AP), so that they displace
// fewer of its weight planes from the caches (1024^2, 11x11, m = 4: the joint
// apply inside the steps 71.5 us against 72.3, the update 37.0 against 37.3;
// the joint CG50 + LOBPCG50 call 9.593-9.615 ms against 9.629-9.635 in
// alternating runs on one GPU; streaming loads of the update's inputs as well
// sped the apply up further but slowed the Gram and the update more).
template <typename T, int M>
__device__ __forceinline__ void store_row_nt(T* __restrict__ dst, const T (&v)[M]) {
  if constexpr (sizeof(T) * M % 16 == 0) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int W = (int)(sizeof(T) * M / 16);
    f4* d4 = reinterpret_cast<f4*>(dst);
#pragma unroll
    for (int w = 0; w < W; ++w) __builtin_nontemporal_store(reinterpret_cast<const f4*>(v)[w], d4 + w);
  } else {
#pragma unroll
    for (int j = 0; j < M; ++j) __builtin_nontemporal_store(v[j], dst + j);
  }
}

// B[i, j] -= Y_i c_j with c = st->yx.  Bound by HBM (B in and out): 16-byte
// pieces by consecutive threads where a point's row is a multiple of them
// (1531 x 2047, FP64, m = 8: 77 us, 148 with a thread per point and its
// columns one by one).
template <typename T, int M>
__global__ void __launch_bounds__(kThreads) lob_project_kernel(T* __restrict__ B, const T* __restrict__ sqd,
                                                               int64_t n, const LobpcgState* st) {
  if (!st->active) return;
  const double yinv = st->ynorm_inv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if constexpr (sizeof(T) * M % 16 == 0) {
    constexpr int V = 16 / (int)sizeof(T), Q = M / V;  // pieces of a row
    typedef T piece_t __attribute__((ext_vector_type(V)));
    __shared__ double c[M];
    if (threadIdx.x < M) c[threadIdx.x] = st->yx[threadIdx.x];
    __syncthreads();
    piece_t* __restrict__ P = (piece_t*)B;
#pragma unroll 4
    for (int64_t e = t0; e < n * Q; e += stride) {
      const int64_t i = e / Q;
      const int j = (int)(e - i * Q) * V;
      const double yi = (double)sqd[i] * yinv;
      piece_t v = P[e];
#pragma unroll
      for (int k = 0; k < V; ++k) v[k] = (T)((double)v[k] - yi * c[j + k]);
      P[e] = v;
    }
  } else {
    double c[M];
#pragma unroll
    for (int j = 0; j < M; ++j) c[j] = st->yx[j];
    for (int64_t i = t0; i < n; i += stride) {
      const double yi = (double)sqd[i] * yinv;
      T v[M];
      load_row<T, M>(B + i * M, v);
#pragma unroll
      for (int j = 0; j < M; ++j) v[j] = (T)((double)v[j] - yi * c[j]);
      store_row<T, M>(B + i * M, v);
    }
  }
}

// NB = number of blocks in the trial basis: 1 (start block), 2 ([X, W]),
// 3 ([X, W, P]).  Coefficients C (NB*M x M, FP64) are read from LDS; every
// output column is accumulated in FP64 and rounded once.  The last cg.nblk
// workgroups run a CG direction phase of the joint driver (same element
// type): the update streams the LOBPCG block, and the direction's three
// vector passes share the launch instead of adding one to the step.
template <typename T, int M, int NB>
__global__ void __launch_bounds__(kThreads) lob_update_kernel(LobArgs a, int first, CgStepArgs cg) {
  __shared__ double Cs[3 * M * M];
  __shared__ double th[M];
  __shared__ double red[16 * 2 * M];
  const int nupd = (int)gridDim.x - cg.nblk;
  if ((int)blockIdx.x >= nupd) {
    cg_pbeta_body<T>((const T*)cg.r, (T*)cg.p, cg.n, cg.upd, cg.nblk, cg.st, cg.k, (int)blockIdx.x - nupd, cg.nblk);
    return;
  }
  LobpcgState* st = a.st;
  if (!st->active) return;
  for (int e = threadIdx.x; e < NB * M * M; e += blockDim.x) Cs[e] = a.C[e];
  if (threadIdx.x < M) th[threadIdx.x] = st->theta[threadIdx.x];
  __syncthreads();
  T* __restrict__ X = (T*)a.X;
  T* __restrict__ W = (T*)a.W;
  T* __restrict__ P = (T*)a.P;
  T* __restrict__ AX = (T*)a.AX;
  T* __restrict__ AW = (T*)a.AW;
  T* __restrict__ AP = (T*)a.AP;
  const T* __restrict__ sqd = (const T*)a.sqd;
  const double yinv = st->ynorm_inv;
  const int64_t stride = (int64_t)nupd * blockDim.x;
  double v[2 * M];
#pragma unroll
  for (int j = 0; j < 2 * M; ++j) v[j] = 0.0;
  // one point: s, as -> the new X, AX, P, AP and W rows
  auto point = [&](const T (&s)[NB][M], const T (&as)[NB][M], double yi, T (&xo)[M], T (&axo)[M], T (&po)[M],
                   T (&apo)[M], T (&ro)[M]) {
#pragma unroll
    for (int t = 0; t < M; ++t) {
      double px = 0.0, pax = 0.0, pp = 0.0, pap = 0.0;
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const double c = Cs[j * M + t];
        px += (double)s[0][j] * c;
        pax += (double)as[0][j] * c;
      }
#pragma unroll
      for (int b = 1; b < NB; ++b) {
#pragma unroll
        for (int j = 0; j < M; ++j) {
          const double c = Cs[(b * M + j) * M + t];
          pp += (double)s[b][j] * c;
          pap += (double)as[b][j] * c;
        }
      }
      const double xn = px + pp, axn = pax + pap;
      const double rt = axn - xn * th[t];
      xo[t] = (T)xn;
      axo[t] = (T)axn;
      po[t] = (T)pp;
      apo[t] = (T)pap;
      ro[t] = (T)rt;
      v[t] += rt * rt;
      v[M + t] += yi * rt;
    }
  };
  // rows of less than 16 bytes go GP points at a time, 16 bytes per block where
  // the blocks are aligned to that (m = 1, FP32, 1024^2: 11.6 us per launch, 13.8
  // a point at a time, as in a workspace off the 16-byte grid)
  constexpr int GP = sizeof(T) * M < 16 && 16 % (sizeof(T) * M) == 0 ? (int)(16 / (sizeof(T) * M)) : 1;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t done = 0;
  if constexpr (GP > 1) {
    const int64_t ng = chunk_aligned(X, W, P, AX, AW, AP) ? a.n / GP : 0;
    done = ng * GP;
    for (int64_t g = t0; g < ng; g += stride) {
      constexpr int E = GP * M;
      const T* __restrict__ sp[3] = {X, W, P};
      const T* __restrict__ asp[3] = {AX, AW, AP};
      T s[NB][E], as[NB][E], y[GP];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        load_row<T, E>(sp[b] + g * E, s[b]);
        load_row<T, E>(asp[b] + g * E, as[b]);
      }
#pragma unroll
      for (int q = 0; q < GP; ++q) y[q] = sqd[g * GP + q];
      T xo[E], axo[E], po[E], apo[E], ro[E];
#pragma unroll
      for (int q = 0; q < GP; ++q) {
        T s1[NB][M], as1[NB][M], x1[M], ax1[M], p1[M], ap1[M], r1[M];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int j = 0; j < M; ++j) {
            s1[b][j] = s[b][q * M + j];
            as1[b][j] = as[b][q * M + j];
          }
        point(s1, as1, (double)y[q] * yinv, x1, ax1, p1, ap1, r1);
#pragma unroll
        for (int j = 0; j < M; ++j) {
          xo[q * M + j] = x1[j];
          axo[q * M + j] = ax1[j];
          po[q * M + j] = p1[j];
          apo[q * M + j] = ap1[j];
          ro[q * M + j] = r1[j];
        }
      }
      store_row_nt<T, E>(X + g * E, xo);
      store_row_nt<T, E>(AX + g * E, axo);
      if (!first) {
        store_row_nt<T, E>(P + g * E, po);
        store_row_nt<T, E>(AP + g * E, apo);
      }
      store_row<T, E>(W + g * E, ro);
    }
  }
  for (int64_t i = done + t0; i < a.n; i += stride) {
    // keep the coefficients in LDS: without this the loop-invariant reads are
    // hoisted into (NB*M*M doubles of) registers and occupancy collapses
    __asm__ volatile("" ::: "memory");
    T s[NB][M], as[NB][M];
    load_row<T, M>(X + i * M, s[0]);
    load_row<T, M>(AX + i * M, as[0]);
    if constexpr (NB > 1) {
      load_row<T, M>(W + i * M, s[1]);
      load_row<T, M>(AW + i * M, as[1]);
    }
    if constexpr (NB > 2) {
      load_row<T, M>(P + i * M, s[2]);
      load_row<T, M>(AP + i * M, as[2]);
    }
    const double yi = (double)sqd[i] * yinv;
    T xo[M], axo[M], po[M], apo[M], ro[M];
    point(s, as, yi, xo, axo, po, apo, ro);
    store_row_nt<T, M>(X + i * M, xo);
    store_row_nt<T, M>(AX + i * M, axo);
    if (!first) {
      store_row_nt<T, M>(P + i * M, po);
      store_row_nt<T, M>(AP + i * M, apo);
    }
    store_row<T, M>(W + i * M, ro);
  }
  block_sum<2 * M>(v, red);
  if (threadIdx.x == 0)
    for (int j = 0; j < 2 * M; ++j) a.vpart[(size_t)blockIdx.x * (2 * M) + j] = v[j];
}

// ---------------------------------------------------------------------------
// output: y = X X^T z0 (+ Y Y^T z0), x_out = y / sqrt(d)
// ---------------------------------------------------------------------------
template <typename T, int M>
__global__ void __launch_bounds__(kThreads) lob_out_dots_kernel(LobArgs a) {
  __shared__ double red[16 * (M + 1)];
  LobpcgState* st = a.st;
  if (st->start_failed) return;
  const T* __restrict__ X = (const T*)a.X;
  const T* __restrict__ x0 = (const T*)a.x0;
  const T* __restrict__ sqd = (const T*)a.sqd;
  const double yinv = st->ynorm_inv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double v[M + 1];
#pragma unroll
  for (int j = 0; j <= M; ++j) v[j] = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
    const double z = (double)sqd[i] * (double)x0[i];
#pragma unroll
    for (int j = 0; j < M; ++j) v[j] += (double)X[i * M + j] * z;
    v[M] += (double)sqd[i] * yinv * z;
  }
  block_sum<M + 1>(v, red);
  if (threadIdx.x == 0)
    for (int j = 0; j <= M; ++j) a.vpart[(size_t)blockIdx.x * (M + 1) + j] = v[j];
}

template <typename T, int M>
__global__ void __launch_bounds__(kThreads) lob_output_kernel(LobArgs a) {
  const LobpcgState* st = a.st;
  const bool broke = st->start_failed != 0;
  const T* __restrict__ X = (const T*)a.X;
  const T* __restrict__ x0 = (const T*)a.x0;
  const T* __restrict__ sqd = (const T*)a.sqd;
  T* __restrict__ out = (T*)a.xout;
  T* __restrict__ rv = (T*)a.ritz;
  double c[M], sg[M];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    c[j] = st->yx[j];
    sg[j] = c[j] >= 0.0 ? 1.0 : -1.0;
  }
  const double cy = a.constraint ? st->yx[M] : 0.0;
  const double yinv = st->ynorm_inv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
    if (broke) {
      out[i] = x0[i];
      continue;
    }
    const double sq = (double)sqd[i];
    double y = sq * yinv * cy;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const double xv = (double)X[i * M + j];
      y += xv * c[j];
      if (rv != nullptr) rv[i * M + j] = (T)(sg[j] * xv);
    }
    out[i] = (T)(y / sq);
  }
}

template <typename T, int M>
void launch_m_kernels(int which, const LobArgs& a, int nb, int ns, int first, StartDegrees deg,
                      const CgStepArgs& cg, hipStream_t s) {
  const CgStepArgs none{};
  const int nbc = nb + cg.nblk;  // the update launches, with the CG phase's workgroups
  switch (which) {
    case 0:
      lob_start_kernel<T, M><<<nb, kThreads, 0, s>>>(a, deg);
      if (a.constraint) lob_final_kernel<M><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 1, M, 0, 1);
      break;
    case 1:
      if (ns == M)
        lob_update_kernel<T, M, 1><<<nbc, kThreads, 0, s>>>(a, first, cg);
      else if (ns == 2 * M)
        lob_update_kernel<T, M, 2><<<nbc, kThreads, 0, s>>>(a, first, cg);
      else
        lob_update_kernel<T, M, 3><<<nbc, kThreads, 0, s>>>(a, first, cg);
      lob_final_kernel<2 * M><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 2, M, first, a.constraint);
      break;
    case 4:
      if (ns == M)
        lob_update_kernel<T, M, 1><<<nbc, kThreads, 0, s>>>(a, first, cg);
      else if (ns == 2 * M)
        lob_update_kernel<T, M, 2><<<nbc, kThreads, 0, s>>>(a, first, cg);
      else
        lob_update_kernel<T, M, 3><<<nbc, kThreads, 0, s>>>(a, first, cg);
      break;
    case 5:
      lob_final_kernel<2 * M><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 2, M, first, a.constraint);
      break;
    case 6:  // W = AX - X Theta of a recomputed AX (a.C = I: X, AX copied, P, AP kept), finalized as an update
      lob_update_kernel<T, M, 1><<<nb, kThreads, 0, s>>>(a, 1, none);
      lob_final_kernel<2 * M><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 2, M, 0, a.constraint);
      break;
    case 7:  // the same, its finalize folded into the next Rayleigh-Ritz step
      lob_update_kernel<T, M, 1><<<nb, kThreads, 0, s>>>(a, 1, none);
      break;
    case 2:
      lob_out_dots_kernel<T, M><<<nb, kThreads, 0, s>>>(a);
      lob_final_kernel<M + 1><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 3, M, 0, a.constraint);
      break;
    default: lob_output_kernel<T, M><<<nb, kThreads, 0, s>>>(a); break;
  }
}

template <typename T>
void launch_m_dispatch(int which, const LobArgs& a, int nb, int ns, int first, StartDegrees deg, const CgStepArgs& cg,
                       hipStream_t s) {
  switch (a.m) {
    case 1: launch_m_kernels<T, 1>(which, a, nb, ns, first, deg, cg, s); break;
    case 2: launch_m_kernels<T, 2>(which, a, nb, ns, first, deg, cg, s); break;
    case 3: launch_m_kernels<T, 3>(which, a, nb, ns, first, deg, cg, s); break;
    case 4: launch_m_kernels<T, 4>(which, a, nb, ns, first, deg, cg, s); break;
    case 5: launch_m_kernels<T, 5>(which, a, nb, ns, first, deg, cg, s); break;
    case 6: launch_m_kernels<T, 6>(which, a, nb, ns, first, deg, cg, s); break;
    case 7: launch_m_kernels<T, 7>(which, a, nb, ns, first, deg, cg, s); break;
    default: launch_m_kernels<T, 8>(which, a, nb, ns, first, deg, cg, s); break;
  }
}

}  // namespace

gsf_status lob_launch_ynorm(const LobArgs& a, int nb, hipStream_t s) {
  if (a.prec == GSF_F32)
    lob_ynorm_kernel<float><<<nb, kThreads, 0, s>>>((const float*)a.sqd, a.n, a.vpart, a.st);
  else
    lob_ynorm_kernel<double><<<nb, kThreads, 0, s>>>((const double*)a.sqd, a.n, a.vpart, a.st);
  lob_final_kernel<1><<<1, kThreads, 0, s>>>(a.vpart, nb, a.st, 0, a.m, 0, 0);
  return launch_status();
}

gsf_status lob_launch_mkernel(int which, const LobArgs& a, int nb, int ns, int first, StartDegrees deg,
                              hipStream_t s, const CgStepArgs* cg_direction) {
  const CgStepArgs none{};
  const CgStepArgs& cp = (cg_direction != nullptr && (which == 1 || which == 4)) ? *cg_direction : none;
  if (cp.nblk > 0 && cp.prec != a.prec) return GSF_EINVAL;
  if (a.prec == GSF_F32)
    launch_m_dispatch<float>(which, a, nb, ns, first, deg, cp, s);
  else
    launch_m_dispatch<double>(which, a, nb, ns, first, deg, cp, s);
  return launch_status();
}

gsf_status lob_launch_project(const LobArgs& a, void* B, int nb, hipStream_t s) {
  auto go = [&](auto zero, auto m) {
    typedef decltype(zero) T;
    lob_project_kernel<T, decltype(m)::value><<<nb, kThreads, 0, s>>>((T*)B, (const T*)a.sqd, a.n, a.st);
  };
  auto of = [&](auto zero) {
    switch (a.m) {
      case 1: go(zero, std::integral_constant<int, 1>{}); break;
      case 2: go(zero, std::integral_constant<int, 2>{}); break;
      case 3: go(zero, std::integral_constant<int, 3>{}); break;
      case 4: go(zero, std::integral_constant<int, 4>{}); break;
      case 5: go(zero, std::integral_constant<int, 5>{}); break;
      case 6: go(zero, std::integral_constant<int, 6>{}); break;
      case 7: go(zero, std::integral_constant<int, 7>{}); break;
      default: go(zero, std::integral_constant<int, 8>{}); break;
    }
  };
  if (a.prec == GSF_F32) of(0.0f);
  else of(0.0);
  return launch_status();
}

int gram_tiles_total(int ns) {
  const int nt = (ns + 15) >> 4;
  return nt == 1 ? 2 : 7;
}

template <typename T>
void launch_gram_kernel(const GramArgs& g, hipStream_t s) {
  switch ((g.ns + 3) >> 2) {
    case 1: gram_kernel<T, 1><<<g.nparts, kThreads, 0, s>>>(g); break;
    case 2: gram_kernel<T, 2><<<g.nparts, kThreads, 0, s>>>(g); break;
    case 3: gram_kernel<T, 3><<<g.nparts, kThreads, 0, s>>>(g); break;
    case 4: gram_kernel<T, 4><<<g.nparts, kThreads, 0, s>>>(g); break;
    case 5: gram_kernel<T, 5><<<g.nparts, kThreads, 0, s>>>(g); break;
    default: gram_kernel<T, 6><<<g.nparts, kThreads, 0, s>>>(g); break;
  }
}

gsf_status lob_launch_gram(const GramArgs& g, const RRArgs& r, int prec, hipStream_t s,
                           const CgStepArgs* cg_update) {
  if (g.ns < 1 || g.ns > KMAX) return GSF_EINVAL;
  if (prec == GSF_F32)
    launch_gram_kernel<float>(g, s);
  else
    launch_gram_kernel<double>(g, s);
  const CgStepArgs none{};
  const CgStepArgs& ca = cg_update != nullptr ? *cg_update : none;
  // with at most kGramDirect Gram workgroups the reduction launch would only
  // copy the partials: the Rayleigh-Ritz workgroup reads them itself
  const int direct = g.nparts <= kGramDirect ? 1 : 0;
  if (!direct) {
    dim3 grid(gram_tiles_total(g.ns) + 1, kGramChunks);
    gram_reduce_kernel<<<grid, kThreads, 0, s>>>(g, r);
  }
  // with a CG phase, unused LDS brings each workgroup above half of a CU's
  // 160 KB, which keeps a second workgroup off the Rayleigh-Ritz workgroup's
  // CU: 41.5 us per call at 1024^2, m = 4 against 42.3 us when a CG workgroup
  // shares it (the CG phase itself ends long before the step)
  constexpr size_t kHalfCu = 80 * 1024 + 1024;
  constexpr size_t kReserve = sizeof(RRShared) < kHalfCu ? kHalfCu - sizeof(RRShared) : 0;
  rr_dispatch(g.ns, [&](auto kb) {
    gram_rr_kernel<decltype(kb)::value><<<1 + ca.nblk, kThreads, ca.nblk > 0 ? kReserve : 0, s>>>(g, r, ca, direct);
  });
  return launch_status();
}

namespace {
// Rayleigh-Ritz alone on a Gram pair already in device memory (GA then GB,
// ns x ns each, row-major), one workgroup.
template <int KB>
__global__ void __launch_bounds__(kThreads) rr_only_kernel(const double* __restrict__ G, int ns, int m, RRArgs r) {
  constexpr int E = RRGrid<KB>::E;
  __shared__ RRShared sh;
  double ga[E][E], gb[E][E];
#pragma unroll
  for (int i = 0; i < E; ++i)
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int row = (threadIdx.x >> 4) + 16 * i, col = (threadIdx.x & 15) + 16 * j;
      const bool in = row < ns && col < ns;
      ga[i][j] = in ? G[row * ns + col] : 0.0;
      gb[i][j] = in ? G[ns * ns + row * ns + col] : 0.0;
    }
  const unsigned kept = rayleigh_ritz<KB>(sh, ga, gb, ns, m, r.drop_tol, r.zero_tol, r.C, r.theta);
  if ((int)threadIdx.x < ns) r.kept_out[threadIdx.x] = (kept >> threadIdx.x) & 1u;
  if (threadIdx.x == 0) *r.nkept_out = __popc(kept);
}
}  // namespace

gsf_status lob_launch_rr_only(const double* G, int ns, int m, const RRArgs& r, hipStream_t s) {
  rr_dispatch(ns, [&](auto kb) { rr_only_kernel<decltype(kb)::value><<<1, kThreads, 0, s>>>(G, ns, m, r); });
  return launch_status();
}

}  // namespace gsf

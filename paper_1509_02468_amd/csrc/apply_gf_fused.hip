// Guided-filter operator apply in one pass (Section 3, Algorithm 1 with the
// fixed guidance g, eqs. (5)-(6)), one FP32 column: the two box-filter stages
// of Algorithm 1 chained through on-chip memory, so the window coefficients
// (a_k, b_k) never reach HBM.  (Blocks of columns and FP64 data take the
// two-pass kernels of apply_gf.hip: with the columns of a block interleaved
// per point, a pass over column pairs reads x at a stride and re-reads the
// guidance data per pair, 3.9 ms against 1.5 ms at m = 8, 4096^2, r = 8.)
//
// A workgroup is one wave: it owns a strip of 256 columns, four adjacent ones
// per lane, and a chunk of rows, and walks the window-centre rows k_y top to
// bottom.  Horizontal window sums are differences of prefix sums along pieces of
// 64 columns of the strip row (three adds in the lane, then one scan of the
// lanes' totals by DPP shifts within rows of 16 lanes), plus the left piece's
// total where a window's ends lie in two, so no lane loops over a window and a
// huge or non-finite value reaches no further right than the end of the piece
// after its own (and the window).  Per centre row:
//   A  running FP64 vertical window sums of u = D^-1/2 x and g u over input
//      rows k_y - r .. k_y + r (add the entering row, subtract the leaving
//      one), their prefix sums;
//   C  the centres' horizontal sums from two prefix values each and their
//      coefficients
//        a_k = (mean(g u)_k - mu_k mean(u)_k) / (sigma_k^2 + eps),
//        b_k = mean(u)_k - a_k mu_k
//      (mu_k and 1/(sigma_k^2 + eps) from the operator build), rounded to
//      FP32 as the two-pass path stores them, added to running FP64 vertical
//      sums of (a, b), their prefix sums;
//   E  the output points of row k_y - r: horizontal sums of (a, b) from two
//      prefix values and the output form
//        GF(u)_i = (g_i sum a + sum b) / N_i,  N x = D^1/2 GF(D^-1/2 x), ...;
//      then row k_y - 2r leaves the (a, b) sums and row k_y takes its place in
//      the LDS ring of 2r rows.
// One wave needs no barriers: LDS operations of a wave complete in order, and
// the prefix rows of both stages share one buffer.  Step A of the next row
// runs between the requests for the (a, b) prefix values and their use.
//
// One column per thread (256 threads, four scans and sets of addresses per
// row, two barriers) took four times the vector instructions; now about 330
// per 256 points and row, 40% of the cycles of the one wave per SIMD that the
// ring's LDS allows at r = 8.  4096^2, r = 8: 167 us (2.0 TB/s of the 20 B per
// point), 282 before; a CG filter of 10 steps on 128^2 1.8 (r = 8) to 2.9
// (r = 1) times as fast, on 1024^2 1.6 to 2.2 times.
// The strip's 256 - 4r (to a multiple of 8) output columns carry a halo on
// each side (r for each box); a chunk of rb output rows walks rb + 2r centre
// rows.  Loads run two centre rows ahead in registers (the entering input row,
// the centre row's statistics, the output row's g and x, which is also the
// next centre row's leaving input row).  HBM
// traffic per point is Algorithm 1's own: x, g, mu, 1/(var + eps) in and y out
// (the rows read again for the epilogue hit L2).  Counts and
// 1/sqrt(d) come from the border-truncated window sizes with the same
// expressions as the operator build (interior values computed once), so u
// equals the stored-diagonal product bit for bit.  A 1D signal is one row with
// no vertical window.
#include <cmath>
#include <type_traits>

#include "gsf_internal.h"

namespace gsf {
namespace {

constexpr int kFW = 256;  // columns per strip, four per lane

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

struct FusedArgs {
  const float* x;
  int64_t ldx;
  const float* g;
  const float* mu;
  const float* inv;
  float* y;
  int64_t ldy;
  int rows, cols;
  int rb;       // output rows per workgroup
  int form;
  double omega;  // |w| = (2r+1)^ndim
  double* dots;  // nullable: x^T y partials, one per workgroup
};

__device__ __forceinline__ int fcount(int v, int len, int r) {
  const int lo = v - r < 0 ? 0 : v - r;
  const int hi = v + r >= len ? len - 1 : v + r;
  return hi - lo + 1;
}

// inclusive prefix sums over each row of 16 lanes: shifts by 1, 2, 4, 8; two at
// a time, each filling the other's latency
template <int CTRL>
__device__ __forceinline__ void scan_step(double& v, double& w) {
  const double a = dpp_move<CTRL>(v), b = dpp_move<CTRL>(w);
  v += a;
  w += b;
}
__device__ __forceinline__ void row_scan2(double& v, double& w) {
  scan_step<0x111>(v, w);
  scan_step<0x112>(v, w);
  scan_step<0x114>(v, w);
  scan_step<0x118>(v, w);
}

// Keeps the order of the wave's LDS accesses (other lanes read what a lane
// wrote); the unit itself completes them in order.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <int R, int RV>
struct FusedShape {
  static constexpr int HL = (2 * R + 3) & ~3;        // strip columns left (and right) of the outputs
  static constexpr int NOUT = kFW - 2 * HL;
  static constexpr int PL = (R + 4) / 4, PR = (R + 3) / 4;  // lanes of zeros beside the prefix rows
  static constexpr int PW = 64 + PL + PR;
  static constexpr int NR = RV > 0 ? 2 * RV : 1;
};

template <int R, int RV>
struct FusedShared {
  typedef FusedShape<R, RV> S;
  double P[2][4][S::PW];   // prefix rows of two channels, by column modulo 4
  f4 ring[S::NR][2][64];   // (a, b) of the last 2 RV centre rows
};

enum FusedMode {
  kInner,    // every column of the strip is on the grid
  kEdge,     // some are not; a multiple of four columns
  kRagged,   // the same, any count of at least four columns
  kNarrow,   // fewer than four columns, element by element
};

// R: window radius; RV: vertical radius (R for images, 0 for a 1D signal);
// STRIDED: x and y have strides of their own and go element by element.
template <int R, int RV, FusedMode MODE, bool STRIDED>
__device__ __forceinline__ void gf_fused_strip(const FusedArgs& a, FusedShared<R, RV>& sh) {
  typedef FusedShape<R, RV> Shape;
  constexpr int HL = Shape::HL, NOUT = Shape::NOUT, PL = Shape::PL, PW = Shape::PW, NR = Shape::NR;
  auto& P = sh.P;
  auto& ring = sh.ring;

  const int lane = threadIdx.x;
  const int rows = a.rows, cols = a.cols;
  const int col = (int)blockIdx.x * NOUT - HL + 4 * lane;  // the lane's first column (a multiple of 4)
  const int y0 = (int)blockIdx.y * a.rb;
  const int y1 = y0 + a.rb < rows ? y0 + a.rb : rows;
  const bool scale = a.form == GSF_FORM_N || a.form == GSF_FORM_LSYM;
  const bool lap = a.form == GSF_FORM_LSYM || a.form == GSF_FORM_L;
  // contiguous rows: four columns from cb, in the row, moved left by skip to
  // stand at col (4 or more: all off the grid)
  const int cb = MODE == kInner ? col : (col < 0 ? 0 : (col + 4 > cols ? cols - 4 : col));
  const int skip = col < 0 ? 4 : col - cb;
  const bool whole = MODE == kInner || (col >= 0 && col + 4 <= cols);
  const double sro = 1.0 / sqrt(a.omega);
  // vertical window sizes: 2RV + 1 away from the top and bottom RV rows
  const double rv_in = 1.0 / (double)(2 * RV + 1 < rows ? 2 * RV + 1 : rows);
  auto interior = [&](int v) { return v >= RV && v < rows - RV; };
  auto rv_of = [&](int v) { return interior(v) ? rv_in : 1.0 / (double)fcount(v, rows, RV); };
  // per column 1 / (horizontal window size), 0 off the grid (its u, a and b are zeros)
  auto rh_of = [&](int e) {
    const int c = col + e;
    return MODE == kInner || (c >= 0 && c < cols) ? 1.0 / (double)fcount(c, cols, R) : 0.0;
  };
  // 1/sqrt(d) with d = N / |w|, as the operator build computes and stores it
  auto dinv_of_rv = [&](double rv, int e) {
    const double d = 1.0 / ((rv * rh_of(e)) * a.omega);
    return (double)(float)(1.0 / sqrt(d));
  };
  // away from the top and bottom rows: 1/sqrt(d), 1 / N, and the output's
  // factor c in N x = c GF(u), c = sqrt(1 / N) / sqrt(|w|) (c = 1 / N for the
  // unscaled forms)
  double dinv_in[4], rc_in[4], c_in[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const double rh = rh_of(e);
    rc_in[e] = rv_in * rh;
    dinv_in[e] = scale ? dinv_of_rv(rv_in, e) : 1.0;
    c_in[e] = scale ? (sqrt(rv_in) * sqrt(rh)) * sro : rc_in[e];
  }
  auto clamp_row = [&](int v) { return v < 0 ? 0 : (v >= rows ? rows - 1 : v); };

  // the lane's four values of a row of x (or a plane), zeros off the grid
  auto row_ld = [&](const float* plane, int v) {
    f4 o = *(const f4u*)(plane + (size_t)clamp_row(v) * cols + cb);
    if constexpr (MODE == kRagged) {
      o = skip & 1 ? f4{o[1], o[2], o[3], 0.0f} : o;
      o = skip & 2 ? f4{o[2], o[3], 0.0f, 0.0f} : o;
    }
    if constexpr (MODE != kInner) o = skip >= 4 ? f4{0.0f, 0.0f, 0.0f, 0.0f} : o;
    return o;
  };
  // one by one, unconditionally (loads under a branch each wait for the one before)
  auto row_ld1 = [&](const float* plane, int v, int64_t ld) {
    const float* p = plane + (size_t)clamp_row(v) * cols * ld;
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = MODE == kInner || (col + e >= 0 && col + e < cols);
      const float w = p[(in ? col + e : 0) * ld];
      o[e] = in ? w : 0.0f;
    }
    return o;
  };
  auto row_x = [&](int v) {
    if constexpr (STRIDED) return row_ld1(a.x, v, a.ldx);
    else return row_ld(a.x, v);
  };
  auto row_of = [&](const float* plane, int v) {
    if constexpr (MODE == kNarrow) return row_ld1(plane, v, 1);
    else return row_ld(plane, v);
  };

  // A: the vertical sums of u and g u
  double su[4], sg[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) su[e] = sg[e] = 0.0;
  auto take_row = [&](const f4& xv, const f4& gv, int v, bool add, bool inside) {
    double di[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) di[e] = dinv_in[e];
    if (!inside && scale && !interior(v)) {
      const double rv = rv_of(v);
#pragma unroll
      for (int e = 0; e < 4; ++e) di[e] = dinv_of_rv(rv, e);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double u = (double)xv[e] * di[e];
      if (add) {
        su[e] += u;
        sg[e] += (double)gv[e] * u;
      } else {
        su[e] -= u;
        sg[e] -= (double)gv[e] * u;
      }
    }
  };
  // the four prefix values of a lane's columns, of two channels
  auto prefix = [&](const double (&v)[4], const double (&w)[4], double (&p)[4], double (&q)[4]) {
    p[0] = v[0];
    q[0] = w[0];
#pragma unroll
    for (int e = 1; e < 4; ++e) {
      p[e] = p[e - 1] + v[e];
      q[e] = q[e - 1] + w[e];
    }
    double tp = p[3], tq = q[3];
    row_scan2(tp, tq);
    const double lp = dpp_move<0x111>(tp), lq = dpp_move<0x111>(tq);  // of the lanes to the left
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      p[e] += lp;
      q[e] += lq;
    }
    p[3] = tp;
    q[3] = tq;
  };
  auto put = [&](const double (&p0)[4], const double (&p1)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      P[0][e][PL + lane] = p0[e];
      P[1][e][PL + lane] = p1[e];
    }
  };
  // the prefix values at the ends of the windows c - R .. c + R of the lane's
  // columns c, and the total of the piece that a window leaves for the next one
  struct Ends {
    double hi[2][4], lo[2][4], total[2];
  };
  const int l16 = lane & 15, last = l16 < 8 ? (lane & ~15) - 1 : lane | 15;  // the lane that holds it
  auto get = [&](Ends& w) {
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) w.total[ch] = P[ch][3][PL + last];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        w.hi[ch][e] = P[ch][(e + R) & 3][PL + lane + ((e + R) >> 2)];
        w.lo[ch][e] = P[ch][(e - R - 1) & 3][PL + lane + ((e - R - 1) >> 2)];
      }
    }
  };

  auto box = [&](const Ends& w, int ch, int e) {
    const bool two = l16 + ((e - R - 1) >> 2) < 0 || l16 + ((e + R) >> 2) > 15;  // the window's ends lie in two pieces
    return (w.hi[ch][e] - w.lo[ch][e]) + (two ? w.total[ch] : 0.0);
  };

  for (int e = lane; e < 8 * PW; e += 64) (&P[0][0][0])[e] = 0.0;
  if constexpr (RV > 0) {
    const f4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int q = 0; q < NR; ++q) ring[q][0][lane] = ring[q][1][lane] = z;
  }
  double Sa[4], Sb[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) Sa[e] = Sb[e] = 0.0;
  double dot = 0.0;

  // centre rows of this chunk (those above the image hold no coefficients)
  const int ks = y0 < RV ? 0 : y0 - RV, ke = y1 + RV;
  const int wlo = y0 - 2 * RV < 0 ? 0 : y0 - 2 * RV;
  struct In {
    f4 x, g;
  };
  struct Out {
    f4 mu, inv, eg, ex;
  };
  auto fill_in = [&](int k) { return In{row_x(k + RV), row_of(a.g, k + RV)}; };
  auto fill_out = [&](int k) {
    return Out{row_of(a.mu, k), row_of(a.inv, k), row_of(a.g, k - RV), row_x(k - RV)};
  };
  // row k: the entering row, and the leaving one, which is row k - 1's output
  // row.  steady: both are in range and away from the image's borders.
  Ends wa;
  auto stage_a = [&](const In& in, const f4& xl, const f4& gl, int k, bool steady) {
    const int yin = k + RV, yl = k - RV - 1;
    if (steady || (yin >= 0 && yin < rows)) take_row(in.x, in.g, yin, true, steady);
    if (steady || (yl >= wlo && yl < rows)) take_row(xl, gl, yl, false, steady);
    double p0[4], p1[4];
    prefix(su, sg, p0, p1);
    wave_lds_order();
    put(p0, p1);
    wave_lds_order();
    get(wa);
  };

  In in[2];
  Out ou[2];
  in[0] = fill_in(ks);
  ou[0] = fill_out(ks);
  if constexpr (RV > 0) {
    in[1] = fill_in(ks + 1);
    ou[1] = fill_out(ks + 1);
  }
  __asm__ volatile("" ::: "memory");  // these are the oldest loads of the first pass too
  // input rows of the first centre row's window, without its last
  if constexpr (RV > 0) {
    const int wend = ks + RV < rows ? ks + RV : rows;
    int yy = wlo;
    for (; yy + 4 <= wend; yy += 4) {
      f4 xv[4], gv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        xv[q] = row_x(yy + q);
        gv[q] = row_of(a.g, yy + q);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) take_row(xv[q], gv[q], yy + q, true, false);
    }
    for (; yy < wend; ++yy) take_row(row_x(yy), row_of(a.g, yy), yy, true, false);
  }
  stage_a(in[0], ou[0].ex, ou[0].eg, ks, false);  // no row leaves yet
  if constexpr (RV > 0) in[0] = fill_in(ks + 2);
  __asm__ volatile("" ::: "memory");

  int slot = 0;
  auto step = [&](int k, Out& cur, In& in_next, auto steady_t) {
    constexpr bool steady = decltype(steady_t)::value;
    // C: the centres' (a, b)
    f4 av = {0.0f, 0.0f, 0.0f, 0.0f}, bv = av;
    if (steady || (k >= 0 && k < rows)) {
      double rc[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) rc[e] = rc_in[e];
      if (!steady && !interior(k)) {
        const double rv = rv_of(k);
#pragma unroll
        for (int e = 0; e < 4; ++e) rc[e] = rv * rh_of(e);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double mean_u = box(wa, 0, e) * rc[e], mean_gu = box(wa, 1, e) * rc[e];
        const double mk = (double)cur.mu[e], ik = (double)cur.inv[e];
        const double ak = (mean_gu - mk * mean_u) * ik;
        av[e] = (float)ak;
        bv[e] = (float)(mean_u - ak * mk);
      }
    }
    double p0[4], p1[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Sa[e] += (double)av[e];
      Sb[e] += (double)bv[e];
    }
    prefix(Sa, Sb, p0, p1);
    wave_lds_order();
    put(p0, p1);
    wave_lds_order();
    Ends w;
    get(w);
    f4 oa = av, ob = bv;  // the oldest centre row, k - 2RV
    if constexpr (RV > 0) {
      oa = ring[slot][0][lane];
      ob = ring[slot][1][lane];
      wave_lds_order();
      ring[slot][0][lane] = av;
      ring[slot][1][lane] = bv;
      slot = slot + 1 == NR ? 0 : slot + 1;
    }
    // A of the next row, while the prefix values arrive
    if constexpr (RV > 0) {
      stage_a(in_next, cur.ex, cur.eg, k + 1, steady);
      in_next = fill_in(k + 3);
    }
    // E: the output points of row k - RV
    const int yo = k - RV;
    if (steady || (yo >= y0 && yo < y1)) {
      double c[4], nx[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = c_in[e];
      if (!steady && !interior(yo)) {
        const double rvo = rv_of(yo), srv = sqrt(rvo);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double rh = rh_of(e);
          c[e] = scale ? (srv * sqrt(rh)) * sro : rvo * rh;
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double sa = box(w, 0, e), sb = box(w, 1, e);
        nx[e] = ((double)cur.eg[e] * sa + sb) * c[e];
      }
      if (lap) {
#pragma unroll
        for (int e = 0; e < 4; ++e) nx[e] = (double)cur.ex[e] - nx[e];
      }
      if (a.form == GSF_FORM_L) {
#pragma unroll
        for (int e = 0; e < 4; ++e) nx[e] *= sro * sro / c[e];
      }
      f4 out;
#pragma unroll
      for (int e = 0; e < 4; ++e) out[e] = (float)nx[e];
      if (lane >= HL / 4 && lane < 64 - HL / 4) {
        float* yp = a.y + ((int64_t)yo * cols + col) * a.ldy;
        if (!STRIDED && whole) {
          *(f4u*)yp = out;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (whole || col + e < cols) yp[e * a.ldy] = out[e];
        }
        if (a.dots != nullptr) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (whole || col + e < cols) dot += (double)cur.ex[e] * (double)out[e];
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      Sa[e] -= (double)oa[e];
      Sb[e] -= (double)ob[e];
    }
    // after the last use of the old values: the loads land in their registers
    // (asked for earlier they need copies, which wait for them, every row)
    if constexpr (RV > 0) cur = fill_out(k + 2);
  };
  // Two rows per pass, each with its own registers.  The pass has one way
  // through (an odd count's last row is past the outputs, and writes nothing):
  // with an exit between the rows every wait allowed for a pass that had
  // skipped the younger loads, and drained them all.  Rows whose windows and
  // outputs are all away from the borders take straight-line code.  A signal's
  // one row takes one step.
  const int sk0 = (y0 > RV ? y0 : RV) + RV, sk1 = y1 + RV < rows - 2 * RV - 1 ? y1 + RV : rows - 2 * RV - 1;
  if constexpr (RV == 0) {
    step(ks, ou[0], in[1], std::false_type{});
  } else {
    for (int k = ks; k < ke; k += 2) {
      if (k >= sk0 && k + 1 < sk1) {
        step(k, ou[0], in[1], std::true_type{});
        step(k + 1, ou[1], in[0], std::true_type{});
      } else {
        step(k, ou[0], in[1], std::false_type{});
        step(k + 1, ou[1], in[0], std::false_type{});
      }
    }
  }
  if (a.dots != nullptr) {
    dot = wave_sum(dot);
    if (lane == 0) a.dots[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = dot;
  }
}

template <int R, int RV, FusedMode FORM, bool STRIDED>
__global__ void __launch_bounds__(64) gf_fused_kernel(FusedArgs a) {
  __shared__ FusedShared<R, RV> sh;
  typedef FusedShape<R, RV> Shape;
  const int first = (int)blockIdx.x * Shape::NOUT - Shape::HL;
  if (FORM != kNarrow && first >= 0 && first + kFW <= a.cols)
    gf_fused_strip<R, RV, kInner, STRIDED>(a, sh);
  else
    gf_fused_strip<R, RV, FORM, STRIDED>(a, sh);
}

// Workgroups of one call: as many as the chip holds at once at r = 8 (37 KB of
// LDS: four per CU), so that no second round is left nearly empty; where chunks
// of at most 256 rows are more than that, the fewest rounds, all of them full.
// Short chunks walk 2r rows beside their own but leave no CU idle.
struct FusedGrid {
  int strips, chunks, rb;
};

FusedGrid fused_grid(int rows, int cols, int r, bool two_d) {
  constexpr int kGroups = 1024, kMinRows = 4, kMaxRows = 256;
  FusedGrid g;
  const int nout = kFW - 2 * ((2 * r + 3) & ~3);
  g.strips = (cols + nout - 1) / nout;
  const int64_t rounds = ((int64_t)rows * g.strips + kGroups * kMaxRows - 1) / (kGroups * kMaxRows);
  const int64_t chunks = g.strips < rounds * kGroups ? rounds * kGroups / g.strips : 1;
  g.rb = (int)((rows + chunks - 1) / chunks);
  g.rb = g.rb < kMinRows ? kMinRows : (g.rb > kMaxRows ? kMaxRows : g.rb);
  if (!two_d) g.rb = 1;
  g.chunks = (rows + g.rb - 1) / g.rb;
  return g;
}

template <int R, int RV>
void launch_fused_r(FusedArgs a, const FusedGrid& g, hipStream_t s) {
  a.rb = g.rb;
  const dim3 grid((unsigned)g.strips, (unsigned)g.chunks);
  if (a.cols < 4)
    gf_fused_kernel<R, RV, kNarrow, true><<<grid, 64, 0, s>>>(a);
  else if (a.ldx != 1 || a.ldy != 1)
    gf_fused_kernel<R, RV, kRagged, true><<<grid, 64, 0, s>>>(a);
  else if (a.cols % 4 != 0)
    gf_fused_kernel<R, RV, kRagged, false><<<grid, 64, 0, s>>>(a);
  else
    gf_fused_kernel<R, RV, kEdge, false><<<grid, 64, 0, s>>>(a);
}

void launch_fused(const FusedArgs& a, int r, bool two_d, hipStream_t s) {
  const FusedGrid g = fused_grid(a.rows, a.cols, r, two_d);
#define GSF_FUSED_CASE(RR)                              \
  case RR:                                              \
    if (two_d) launch_fused_r<RR, RR>(a, g, s);          \
    else launch_fused_r<RR, 0>(a, g, s);                 \
    break;
  switch (r) {
    GSF_FUSED_CASE(1)
    GSF_FUSED_CASE(2)
    GSF_FUSED_CASE(3)
    GSF_FUSED_CASE(4)
    GSF_FUSED_CASE(5)
    GSF_FUSED_CASE(6)
    GSF_FUSED_CASE(7)
    default: GSF_FUSED_CASE(8)
  }
#undef GSF_FUSED_CASE
}

}  // namespace

int gf_fused_groups(const Operator& op) {
  const FusedGrid g = fused_grid((int)op.rows, (int)op.cols, op.desc.radius, op.desc.ndim == 2);
  return g.strips * g.chunks;
}

// One-pass GF apply of one FP32 column; dots (nullable): x^T y partials, one
// per workgroup (gf_fused_groups).
gsf_status launch_gf_apply_fused(const Operator& op, int form, const float* x, int64_t ldx, float* y, int64_t ldy,
                                 double* dots, hipStream_t s) {
  FusedArgs a{};
  a.x = x;
  a.y = y;
  a.g = (const float*)op.g;
  a.mu = (const float*)op.mu;
  a.inv = (const float*)op.inv;
  a.ldx = ldx;
  a.ldy = ldy;
  a.rows = (int)op.rows;
  a.cols = (int)op.cols;
  a.form = form;
  a.dots = dots;
  const double w = 2.0 * op.desc.radius + 1.0;
  a.omega = op.desc.ndim == 1 ? w : w * w;
  launch_fused(a, op.desc.radius, op.desc.ndim == 2, s);
  return launch_status();
}

}  // namespace gsf

// Guided-filter operator (Section 3, Algorithm 1, eqs. (5)-(6)): the operator
// build (window statistics of the guidance) and the normalized apply
//   N x = D^1/2 GF(D^-1/2 x),  D = diag(N_i / |w|),
// where GF is Algorithm 1 with the fixed guidance g (a linear filter), mean
// filters over border-truncated windows (N_k points) and the window
// statistics mu_k, inv_k = 1/(sigma_k^2 + eps):
//   u      = D^-1/2 x            (RW form: u = x)
//   a_k    = (box(g u)_k / N_k - mu_k box(u)_k / N_k) inv_k
//   b_k    = box(u)_k / N_k - a_k mu_k
//   GF(u)_i = (g_i box(a)_i + box(b)_i) / N_i
//
// Every window sum runs in one streaming kernel of one wave per workgroup (see
// gf_box_kernel): running FP64 vertical sums in registers, sliding horizontal
// sums over the wave's own LDS row, no barriers.  Cost per point is O(1) in
// the radius.  The apply is two such kernels (u, g u) -> (a, b) and
// (a, b) -> output for up to 8 columns at once; the build is one kernel on
// (g, g^2).  A 1D signal is one row.
#include <cmath>
#include <type_traits>

#include "gsf_internal.h"

namespace gsf {
namespace {

constexpr int kGfLanes = 64;   // one wave per workgroup; lane = halo column
// output rows per workgroup (fewer on small grids); 16 / 24 / 32 / 64 / 128
// compared in alternating runs on one GPU at 4096^2, r = 8, FP32: m = 8 apply
// 1485 / 1462 / 1438-1447 / 1474 / (step +1%) us, m = 4 820 / 798 / 787-791 /
// 807-810 us: more, shorter workgroups hide the row loads better than the
// fewer warm-up rows of long ones save
constexpr int kGfRowsMax = 32;

// 32-bit indices: the operator build rejects GF grids of 2^27 points or more,
// so point * 16 fits.
struct GfGeom {
  int rows, cols;
  int r;
  int rb;  // output rows per workgroup
};

__device__ __forceinline__ int win_count(int v, int len, int r) {
  const int lo = v - r < 0 ? 0 : v - r;
  const int hi = v + r >= len ? len - 1 : v + r;
  return hi - lo + 1;
}

// Keeps the compiler from moving LDS accesses across this point; a wave's
// own LDS operations complete in order, so no hardware barrier is needed.
__device__ __forceinline__ void wave_lds_fence() { __asm__ volatile("" ::: "memory"); }

// One wave owns a strip of 64 CPL - 2r output columns (64 CPL halo columns,
// CPL per lane: lane + 64 k) and g.rb rows (8..64).  Lane l keeps the FP64
// running vertical window sums of its columns c0 - r + l + 64 k for the 2M
// channels (P::M groups of two); per row it
// adds the entering row, writes its sums to the wave's LDS row, and then
// takes the horizontal window sums as lane (group, run of consecutive output
// columns) with a sliding sum over that LDS row, before subtracting the
// leaving row.  Loads are unconditional (clamped addresses, results selected)
// and issued D rows ahead (a register ring, the row loop unrolled by D), so
// a memory latency is spread over D rows.
//   P::Row       raw loads of one point (all groups)
//   P::fetch(i)  -> Row;    P::value(row, j) -> double2 (group j)
//   P::Epi / P::pre(k, j) / P::store(k, j, s0, s1, rc, src, e): epilogue at
//   point k with rc = 1 / (points in the window), src = sqrt(rc).
template <class P, int CPL>
__global__ void __launch_bounds__(kGfLanes) gf_box_kernel(P p, GfGeom g) {
  constexpr int M = P::M;
  constexpr int R = kGfLanes / M;  // runs per group
  constexpr int W = kGfLanes * CPL;  // halo columns of the strip
  constexpr int NO = M * CPL;        // most outputs of one lane's run
  typedef typename P::Row Row;
  typedef typename P::Epi Epi;
  __shared__ double vs[2 * M][W + 1];
  const int r = g.r, ow = W - 2 * r;
  const int lane = threadIdx.x;
  const int c0 = (int)blockIdx.x * ow;
  const int y0 = (int)blockIdx.y * g.rb;
  const int y1 = y0 + g.rb < g.rows ? y0 + g.rb : g.rows;
  // column role: halo columns lane + 64 k of the strip, k < CPL
  bool cok[CPL];
  int gcs[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    const int gc = c0 - r + lane + kGfLanes * k;
    cok[k] = gc >= 0 && gc < g.cols;
    gcs[k] = cok[k] ? gc : 0;
  }
  // run role: group j, output columns [run * L, run * L + L) of the strip
  const int L = (ow + R - 1) / R;
  const int j = lane / R, run = lane - (lane / R) * R;
  const int cb = run * L;
  int nout = ow - cb < L ? ow - cb : L;
  if (c0 + cb + nout > g.cols) nout = (int)(g.cols - c0 - cb);
  if (nout < 0) nout = 0;
  double rh[NO], srh[NO];  // L <= ceil((64 CPL - 2) M / 64) <= M CPL outputs per lane
#pragma unroll
  for (int t = 0; t < NO; ++t) {
    rh[t] = 1.0 / (double)win_count(c0 + cb + t, g.cols, r);
    srh[t] = sqrt(rh[t]);
  }

  double s[CPL][2 * M];
#pragma unroll
  for (int k = 0; k < CPL; ++k)
#pragma unroll
    for (int c = 0; c < 2 * M; ++c) s[k][c] = 0.0;
  auto clamp_row = [&](int y) { return y < 0 ? 0 : (y >= g.rows ? g.rows - 1 : y); };
  const int w0 = y0 - r < 0 ? 0 : y0 - r;
  const int w1 = y0 + r - 1 < g.rows - 1 ? y0 + r - 1 : g.rows - 1;
#pragma unroll
  for (int k = 0; k < CPL; ++k) {
    Row cur = p.fetch(clamp_row(w0) * g.cols + gcs[k]);
    for (int yy = w0; yy <= w1; ++yy) {
      const Row nxt = p.fetch(clamp_row(yy + 1) * g.cols + gcs[k]);
      if (cok[k]) {
#pragma unroll
        for (int q = 0; q < M; ++q) {
          const double2 v = p.value(cur, q);
          s[k][2 * q] += v.x;
          s[k][2 * q + 1] += v.y;
        }
      }
      cur = nxt;
    }
  }
  // ring of the entering / leaving points of the next D output rows
  constexpr int D = M <= 2 ? 4 : (M == 4 ? 2 : 1);
  // and of the epilogue's loads at the output points, the same D rows ahead
  Row fa[D][CPL], fd[D][CPL];
  Epi ep[D][NO];
  auto out_col = [&](int t) { return t < nout ? c0 + cb + t : c0; };
#pragma unroll
  for (int u = 0; u < D; ++u) {
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      fa[u][k] = p.fetch(clamp_row(y0 + u + r) * g.cols + gcs[k]);
      fd[u][k] = p.fetch(clamp_row(y0 + u - r) * g.cols + gcs[k]);
    }
#pragma unroll
    for (int t = 0; t < NO; ++t) ep[u][t] = p.pre(clamp_row(y0 + u) * g.cols + out_col(t), j);
  }
  // The body runs for every u, also past the workgroup's last row in the final
  // group (only the stores are skipped there): a ring slot refilled on some
  // paths only would need a register copy, and so a wait, every row.
  for (int yb = y0; yb < y1; yb += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int yo = yb + u;
      const bool live = yo < y1;
      const int ya = yo + r, yd = yo - r;
      Epi e[NO];
#pragma unroll
      for (int t = 0; t < NO; ++t) {
        e[t] = ep[u][t];
        ep[u][t] = p.pre(clamp_row(yo + D) * g.cols + out_col(t), j);
      }
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const bool add = cok[k] && ya < g.rows;
#pragma unroll
        for (int q = 0; q < M; ++q) {
          const double2 v = p.value(fa[u][k], q);
          s[k][2 * q] += add ? v.x : 0.0;
          s[k][2 * q + 1] += add ? v.y : 0.0;
        }
      }
      wave_lds_fence();
#pragma unroll
      for (int k = 0; k < CPL; ++k)
#pragma unroll
        for (int c = 0; c < 2 * M; ++c) vs[c][lane + kGfLanes * k] = cok[k] ? s[k][c] : 0.0;
      wave_lds_fence();
      const int vc = (ya < g.rows ? ya : g.rows - 1) - (yd < 0 ? 0 : yd) + 1;
      const double rv = 1.0 / (double)vc, srv = sqrt(rv);
      if (nout > 0 && live) {
        const double* v0 = &vs[2 * j][cb];
        const double* v1 = &vs[2 * j + 1][cb];
        double a0 = 0.0, a1 = 0.0;
        for (int h = 0; h < 2 * r; ++h) {
          a0 += v0[h];
          a1 += v1[h];
        }
#pragma unroll
        for (int t = 0; t < NO; ++t) {
          if (t < nout) {
            a0 += v0[t + 2 * r];
            a1 += v1[t + 2 * r];
            p.store(yo * g.cols + c0 + cb + t, j, a0, a1, rv * rh[t], srv * srh[t], e[t]);
            a0 -= v0[t];
            a1 -= v1[t];
          }
        }
      }
      wave_lds_fence();
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const bool sub = cok[k] && yd >= 0;
#pragma unroll
        for (int q = 0; q < M; ++q) {
          const double2 v = p.value(fd[u][k], q);
          s[k][2 * q] -= sub ? v.x : 0.0;
          s[k][2 * q + 1] -= sub ? v.y : 0.0;
        }
        fa[u][k] = p.fetch(clamp_row(ya + D) * g.cols + gcs[k]);
        fd[u][k] = p.fetch(clamp_row(yd + D) * g.cols + gcs[k]);
      }
    }
  }
}

// (u, g u) -> (a, b) at every window centre; AB point-major, pairs per group
template <typename T, int MM, bool SCALE>
struct GfStage1 {
  static constexpr int M = MM;
  const T* x;
  int ldx;
  const T* g;
  const T* dinv;  // 1/sqrt(d) (SCALE), else u = x (RW form)
  const T* mu;
  const T* inv;
  T* ab;
  struct Row {
    T x[M];
    T g, d;
  };
  __device__ __forceinline__ Row fetch(int i) const {
    Row w;
#pragma unroll
    for (int q = 0; q < M; ++q) w.x[q] = x[i * ldx + q];
    w.g = g[i];
    w.d = SCALE ? dinv[i] : T(1);
    return w;
  }
  __device__ __forceinline__ double2 value(const Row& w, int q) const {
    const double u = (double)w.x[q] * (double)w.d;
    return make_double2(u, (double)w.g * u);
  }
  struct Epi {
    T mu, inv;
  };
  __device__ __forceinline__ Epi pre(int k, int) const { return Epi{mu[k], inv[k]}; }
  __device__ __forceinline__ void store(int k, int j, double su, double sgu, double rc, double, const Epi& e) const {
    const double mk = (double)e.mu;
    const double mean_u = su * rc, mean_gu = sgu * rc;
    const double av = (mean_gu - mk * mean_u) * (double)e.inv;
    ab[(k * M + j) * 2] = (T)av;
    ab[(k * M + j) * 2 + 1] = (T)(mean_u - av * mk);
  }
};

// (a, b) -> y = D^1/2 GF(u) (N), x - D^1/2 GF(u) (L_sym), GF(x) (RW) or
// D (x - GF(x)) = L x (L, with d = N/|w|)
template <typename T, int MM>
struct GfStage2 {
  static constexpr int M = MM;
  const T* ab;
  const T* g;
  const T* x;
  int ldx;
  T* y;
  int ldy;
  int form;
  double sromega;  // 1 / sqrt(|w|)
  struct Row {
    T v[2 * M];
  };
  __device__ __forceinline__ Row fetch(int i) const {
    Row w;
#pragma unroll
    for (int q = 0; q < 2 * M; ++q) w.v[q] = ab[i * 2 * M + q];
    return w;
  }
  __device__ __forceinline__ double2 value(const Row& w, int q) const {
    return make_double2((double)w.v[2 * q], (double)w.v[2 * q + 1]);
  }
  struct Epi {
    T g, x;
  };
  __device__ __forceinline__ Epi pre(int i, int j) const {
    return Epi{g[i], (form == GSF_FORM_LSYM || form == GSF_FORM_L) ? x[i * ldx + j] : T(0)};
  }
  __device__ __forceinline__ void store(int i, int j, double sa, double sb, double rc, double src,
                                        const Epi& e) const {
    const double gfu = (double)e.g * sa + sb;
    double out;
    if (form == GSF_FORM_RW) {
      out = gfu * rc;
    } else if (form == GSF_FORM_L) {
      out = ((double)e.x - gfu * rc) * (sromega * sromega / rc);  // d (x - GF(x)), d = N/|w|
    } else {
      const double nx = gfu * (src * sromega);  // (g sum a + sum b) / sqrt(N_i |w|)
      out = form == GSF_FORM_LSYM ? (double)e.x - nx : nx;
    }
    y[i * ldy + j] = (T)out;
  }
};

// build: (g, g^2) -> mu, 1/(var + eps), d = N/|w|, sqrt(d), 1/sqrt(d), copy of g
template <typename T>
struct GfStats {
  static constexpr int M = 1;
  const T* gin;
  T* gcopy;
  T* mu;
  T* inv;
  T* sqd;
  T* dinv;
  double* deg;
  double eps, omega;
  struct Row {
    T v;
  };
  __device__ __forceinline__ Row fetch(int i) const { return Row{gin[i]}; }
  __device__ __forceinline__ double2 value(const Row& w, int) const {
    const double v = (double)w.v;
    return make_double2(v, v * v);
  }
  struct Epi {
    T gk;
  };
  __device__ __forceinline__ Epi pre(int k, int) const { return Epi{gin[k]}; }
  __device__ __forceinline__ void store(int k, int, double s1, double s2, double rc, double, const Epi& e) const {
    const double m = s1 * rc;
    const double var = s2 * rc - m * m;
    mu[k] = (T)m;
    inv[k] = (T)(1.0 / (var + eps));
    const double d = 1.0 / (rc * omega);
    deg[k] = d;
    sqd[k] = (T)sqrt(d);
    dinv[k] = (T)(1.0 / sqrt(d));
    gcopy[k] = e.gk;
  }
};

// Rows per workgroup: as many as possible up to kGfRowsMax (the 2r warm-up
// rows are amortised) while the grid still has about 2048 waves to hide
// memory latency.
template <int CPL>
GfGeom gf_geom(const Operator& op) {
  const int ow = kGfLanes * CPL - 2 * op.desc.radius;
  const int64_t strips = (op.cols + ow - 1) / ow;
  int64_t rb = (op.rows * strips + 2047) / 2048;
  rb = rb < 8 ? 8 : (rb > kGfRowsMax ? kGfRowsMax : rb);
  return GfGeom{(int)op.rows, (int)op.cols, op.desc.radius, (int)rb};
}

template <int CPL>
dim3 gf_grid(const Operator& op, const GfGeom& g) {
  const int ow = kGfLanes * CPL - 2 * op.desc.radius;
  return dim3((unsigned)((op.cols + ow - 1) / ow), (unsigned)((op.rows + g.rb - 1) / g.rb));
}

// Columns per lane: two for the one-column passes (half the LDS reads and
// horizontal adds per output, and a 1/(64 - r) instead of 2r/(64 - 2r) halo
// share), one for blocks, whose lanes already produce M outputs each.
template <int M>
struct GfCpl {
  static constexpr int v = M == 1 ? 2 : 1;
};

// ---------------------------------------------------------------------------
// contiguous blocks of 4 or 8 columns
// ---------------------------------------------------------------------------
// The two passes of the apply for a point-major block whose M columns are all
// of it: a row is one run of memory, read in 16-byte pieces by consecutive
// threads, each of which keeps the FP64 vertical window sums of its pieces
// whatever column they belong to.  (One grid column per lane, the kernel above,
// spreads every load over 64 lines and, in groups of 4 FP64 columns of 8, uses
// half of each.)  Four waves own a strip of 256 columns, 2r of them halo, and
// rb rows; per row they add the entering row, put their sums into an LDS row,
// and after one barrier (the rows alternate between two buffers) take the
// horizontal window sums as (run of consecutive columns, block column).  Per
// apply, r = 8: 1531 x 2047, FP64, m = 8 514 us (2.9 TB/s of the two passes'
// least traffic), 794 as two groups of 4 columns of the kernel above; FP32,
// m = 8 236 us, 335; 256 x 256, FP32, m = 4 23 us, 32.
//
// Rounding.  A horizontal sum takes additions only (a sliding one over runs of
// 8 columns was less exact than the kernel above, whose runs are shorter).  A
// vertical sum gathers a rounding with every row that enters or leaves, and
// keeps a huge or non-finite value after its row has left; chunks of more than
// kGfRowsMax rows, the kernel above's most, therefore renew their sums every
// 2r + 1 rows (RENEW) from a second set that only adds the rows that enter.
// L_sym x of uniform data, FP64, m = 8, r = 8, relative to long double:
// 3.5e-16 at 1531 x 2047 and 3.3e-16 at 4096^2 (147 rows a chunk), 4.2e-16 and
// 4.1e-16 by the kernel above; with sliding sums never renewed 4.7e-16 and
// 6.2e-16.  Renewing costs 1% at 4096^2 (2426 us, 2401 without; 4140 above).
constexpr int kGfBlkThreads = 256;
constexpr int kGfBlkCols = 256;  // halo columns of a strip

template <typename T, int M>
struct GfBlkShared {
  static constexpr int kPitch = 2 * M + 2;  // doubles per column: runs of columns spread over the banks
  // most outputs of a run; a strip's last run may read that many columns past its row
  static constexpr int kRun = (kGfBlkCols * M + kGfBlkThreads - 1) / kGfBlkThreads;
  double vs[(2 * kGfBlkCols + kRun) * kPitch];  // two rows
  double2 rh[kGfBlkCols];                   // 1 / (points of the horizontal window) and its root
};

struct GfBlkArgs {
  const void* in;    // stage 1: x; stage 2: (a, b)
  const void* x;     // stage 2: x (L_sym and L forms)
  int64_t ldx, ldy;  // elements between consecutive points of x and y
  const void* g;
  const void* dinv;  // stage 1: 1/sqrt(d), or nullptr (u = x)
  const void* mu;
  const void* inv;
  void* out;         // stage 1: (a, b); stage 2: y
  int rows, cols, r, rb;
  int form;
  double sromega;    // 1 / sqrt(|w|)
};

// DENSE: the pieces of `in` are aligned runs (else x has a row stride or
// address of its own and is read by elements; the same sums).  RENEW: see above.
template <typename T, int M, int STAGE, bool SCALE, bool DENSE, bool RENEW>
__global__ void __launch_bounds__(kGfBlkThreads, 2) gf_block_kernel(GfBlkArgs a) {
  constexpr int V = 16 / (int)sizeof(T);      // elements of a piece
  constexpr int K = STAGE == 1 ? M : 2 * M;   // elements of a point's row
  constexpr int NP = K / V;                   // pieces per thread
  constexpr int NC = STAGE == 1 ? 2 : 1;      // sums per element
  constexpr int R = kGfBlkThreads / M;        // runs
  constexpr int NO = GfBlkShared<T, M>::kRun;
  constexpr int PITCH = GfBlkShared<T, M>::kPitch;
  typedef T piece_t __attribute__((ext_vector_type(V)));
  __shared__ GfBlkShared<T, M> sh;
  const int t = threadIdx.x, r = a.r, ow = kGfBlkCols - 2 * r;
  const int c0 = (int)blockIdx.x * ow, y0 = (int)blockIdx.y * a.rb;
  const int y1 = y0 + a.rb < a.rows ? y0 + a.rb : a.rows;
  const T* __restrict__ in = (const T*)a.in;
  const T* __restrict__ g = (const T*)a.g;
  const T* __restrict__ dinv = (const T*)a.dinv;

  // piece role: strip column, element of its row, offset in an image row
  int pcol[NP], pel[NP], goff[NP];
  bool ok[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int e = (p * kGfBlkThreads + t) * V;
    pcol[p] = e / K;
    pel[p] = e % K;
    const int gc = c0 - r + pcol[p];
    ok[p] = gc >= 0 && gc < a.cols;
    goff[p] = ok[p] ? gc : 0;
  }
  struct Row {
    piece_t v[NP];
    T g[NP], d[NP];
  };
  auto clamp_row = [&](int y) { return y < 0 ? 0 : (y >= a.rows ? a.rows - 1 : y); };
  auto fetch = [&](int y) {
    Row w;
    const size_t base = (size_t)clamp_row(y) * a.cols;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if constexpr (DENSE) {
        w.v[p] = *(const piece_t*)(in + base * K + ((size_t)goff[p] * K + pel[p]));
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i) w.v[p][i] = in[(base + goff[p]) * a.ldx + pel[p] + i];
      }
      if constexpr (STAGE == 1) {
        w.g[p] = g[base + goff[p]];
        if constexpr (SCALE) w.d[p] = dinv[base + goff[p]];
      }
    }
    return w;
  };
  // the running sums, and their successors: from zero, the entering rows alone
  double s[NP][V][NC], f[NP][V][NC];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int i = 0; i < V; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) s[p][i][c] = f[p][i][c] = 0.0;
  enum { kWarm, kEnter, kLeave };
  auto add_row = [&](const Row& w, int what, bool live = true) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        double u[NC];
        u[0] = (double)w.v[p][i];
        if constexpr (STAGE == 1 && SCALE) u[0] *= (double)w.d[p];
        u[0] = ok[p] && live ? u[0] : 0.0;
        if constexpr (STAGE == 1) u[NC - 1] = ok[p] && live ? (double)w.g[p] * u[0] : 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          s[p][i][c] += what == kLeave ? -u[c] : u[c];
          if (RENEW && what == kEnter) f[p][i][c] += u[c];
        }
      }
    }
  };

  // run role: block column j, output columns [cb, cb + nout) of the strip
  const int L = (ow + R - 1) / R, j = t % M, cb = (t / M) * L;
  int nout = ow - cb < L ? ow - cb : L;
  if (c0 + cb + nout > a.cols) nout = a.cols - c0 - cb;
  struct Epi {
    T p[NO], q[NO];  // stage 1: mu, inv; stage 2: g, x
  };
  const bool need_x = a.form == GSF_FORM_LSYM || a.form == GSF_FORM_L;
  auto pre = [&](int y) {
    Epi e;
    const size_t base = (size_t)clamp_row(y) * a.cols + c0 + cb;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      e.p[o] = e.q[o] = T(0);
      if (o < nout) {
        if constexpr (STAGE == 1) {
          e.p[o] = ((const T*)a.mu)[base + o];
          e.q[o] = ((const T*)a.inv)[base + o];
        } else {
          e.p[o] = g[base + o];
          if (need_x) e.q[o] = ((const T*)a.x)[(base + o) * a.ldx + j];
        }
      }
    }
    return e;
  };

  {
    const int c = c0 + t;  // output column t of the strip
    const double rh = c < a.cols ? 1.0 / (double)win_count(c, a.cols, r) : 0.0;
    sh.rh[t] = make_double2(rh, sqrt(rh));
  }
  // the window rows of the first output row, without its last
  const int w0 = y0 - r < 0 ? 0 : y0 - r;
  const int w1 = y0 + r - 1 < a.rows - 1 ? y0 + r - 1 : a.rows - 1;
  Row enter = fetch(y0 + r), leave = fetch(y0 - r);
  Epi epi = pre(y0);
  for (int yy = w0; yy <= w1; yy += 2) {
    const Row p = fetch(yy), q = fetch(yy + 1);
    add_row(p, kWarm);
    add_row(q, kWarm, yy + 1 <= w1);  // (not under a branch: the compiler then moves the loads there too)
  }
  int age = 0;
  for (int yo = y0; yo < y1; ++yo) {
    const int ya = yo + r, yd = yo - r;
    if (ya < a.rows) add_row(enter, kEnter);
    enter = fetch(ya + 1);
    if (RENEW && ++age == 2 * r + 1) {  // the successors hold the whole window
      age = 0;
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < V; ++i)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            s[p][i][c] = f[p][i][c];
            f[p][i][c] = 0.0;
          }
    }
    double* vs = sh.vs + ((yo - y0) & 1) * (kGfBlkCols * PITCH);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if constexpr (STAGE == 1) {
        double2* w = (double2*)(vs + pcol[p] * PITCH + 2 * pel[p]);
#pragma unroll
        for (int i = 0; i < V; ++i) w[i] = make_double2(s[p][i][0], s[p][i][NC - 1]);
      } else {
        double2* w = (double2*)(vs + pcol[p] * PITCH + pel[p]);
#pragma unroll
        for (int i = 0; i < V; i += 2) w[i / 2] = make_double2(s[p][i][0], s[p][i + 1][0]);
      }
    }
    lds_barrier();
    if (nout > 0) {
      const int vc = (ya < a.rows ? ya : a.rows - 1) - (yd < 0 ? 0 : yd) + 1;
      const double rv = 1.0 / (double)vc, srv = sqrt(rv);
      const double* v = vs + cb * PITCH + 2 * j;
      // window sums of the run, by additions only: of G outputs at a time
      // (2r >= G), what their windows share plus the columns left and right of
      // it that each has; left and right one after the other (both at once
      // spilled at eight FP64 columns)
      double2 sum[NO];
      auto window_sums = [&](auto group) {
        constexpr int G = decltype(group)::value < NO ? decltype(group)::value : NO;
#pragma unroll
        for (int b = 0; b < NO; b += G) {
          const double* vb = v + b * PITCH;
          double2 side[G], core = *(const double2*)(vb + G * PITCH);
#pragma unroll
          for (int o = 0; o < G; ++o) side[o] = *(const double2*)(vb + o * PITCH);
#pragma unroll 4
          for (int h = G + 1; h <= 2 * r; ++h) {
            const double2 w = *(const double2*)(vb + h * PITCH);
            core.x += w.x;
            core.y += w.y;
          }
          core.x += side[G - 1].x;
          core.y += side[G - 1].y;
          sum[b + G - 1] = core;
          double2 t = {0.0, 0.0};
#pragma unroll
          for (int o = G - 2; o >= 0; --o) {
            t.x += side[o].x;
            t.y += side[o].y;
            sum[b + o] = make_double2(core.x + t.x, core.y + t.y);
          }
          if constexpr (RENEW && M * sizeof(T) == 64) __builtin_amdgcn_sched_barrier(0);
          vb += 2 * r * PITCH;
#pragma unroll
          for (int o = 1; o < G; ++o) side[o] = *(const double2*)(vb + o * PITCH);
          t = {0.0, 0.0};
#pragma unroll
          for (int o = 1; o < G; ++o) {
            t.x += side[o].x;
            t.y += side[o].y;
            sum[b + o].x += t.x;
            sum[b + o].y += t.y;
          }
        }
      };
      if (r >= 4) window_sums(std::integral_constant<int, 8>{});
      else if (r >= 2) window_sums(std::integral_constant<int, 4>{});
      else window_sums(std::integral_constant<int, 2>{});
      const size_t base = (size_t)yo * a.cols + c0 + cb;
#pragma unroll
      for (int o = 0; o < NO; ++o) {
        if (o < nout) {
          const double a0 = sum[o].x, a1 = sum[o].y;
          const double2 h = sh.rh[cb + o];
          const double rc = rv * h.x;
          if constexpr (STAGE == 1) {
            const double mk = (double)epi.p[o];
            const double mean_u = a0 * rc, mean_gu = a1 * rc;
            const double av = (mean_gu - mk * mean_u) * (double)epi.q[o];
            typedef T pair_t __attribute__((ext_vector_type(2)));
            ((pair_t*)a.out)[(base + o) * M + j] = pair_t{(T)av, (T)(mean_u - av * mk)};
          } else {
            const double gfu = (double)epi.p[o] * a0 + a1, xi = (double)epi.q[o];
            double out;
            if (a.form == GSF_FORM_RW) {
              out = gfu * rc;
            } else if (a.form == GSF_FORM_L) {
              out = (xi - gfu * rc) * (a.sromega * a.sromega / rc);  // d (x - GF(x)), d = N/|w|
            } else {
              const double nx = gfu * ((srv * h.y) * a.sromega);  // (g sum a + sum b) / sqrt(N_i |w|)
              out = a.form == GSF_FORM_LSYM ? xi - nx : nx;
            }
            ((T*)a.out)[(base + o) * a.ldy + j] = (T)out;
          }
        }
      }
    }
    epi = pre(yo + 1);
    if (yd >= 0) add_row(leave, kLeave);
    leave = fetch(yd + 1);
  }
}

// Strips of a row, and rows per workgroup: the strips and chunks fill the
// chip's workgroup slots (two per CU by registers and LDS) once, down to 4 rows.
struct GfBlkGrid {
  int ow, strips, rb;
};
GfBlkGrid gf_block_grid(const Operator& op) {
  constexpr int kGroups = 512, kMinRows = 4;
  GfBlkGrid g;
  g.ow = kGfBlkCols - 2 * op.desc.radius;
  g.strips = ((int)op.cols + g.ow - 1) / g.ow;
  const int chunks = g.strips < kGroups ? kGroups / g.strips : 1;
  g.rb = ((int)op.rows + chunks - 1) / chunks;
  if (g.rb < kMinRows) g.rb = kMinRows;
  return g;
}

template <typename T, int M>
void gf_apply_block(const Operator& op, T* ab, int form, const T* x, int64_t ldx, T* y, int64_t ldy,
                    hipStream_t s) {
  GfBlkArgs a{};
  a.rows = (int)op.rows;
  a.cols = (int)op.cols;
  a.r = op.desc.radius;
  a.form = form;
  const double w = 2.0 * op.desc.radius + 1.0;
  a.sromega = 1.0 / sqrt(op.desc.ndim == 1 ? w : w * w);
  const GfBlkGrid geo = gf_block_grid(op);
  a.rb = geo.rb;
  const dim3 grid((unsigned)geo.strips, (unsigned)((a.rows + a.rb - 1) / a.rb));
  a.g = op.g;
  a.mu = op.mu;
  a.inv = op.inv;
  a.x = x;
  a.in = x;
  a.out = ab;
  a.ldx = ldx;
  a.ldy = ldy;
  const bool dense = ldx == M && (uintptr_t)x % 16 == 0;
  const bool scale = form != GSF_FORM_RW && form != GSF_FORM_L;
  if (scale) a.dinv = op.diag;
  auto passes = [&](auto renew) {
    constexpr bool N = decltype(renew)::value;
    if (!scale) {
      if (dense) gf_block_kernel<T, M, 1, false, true, N><<<grid, kGfBlkThreads, 0, s>>>(a);
      else gf_block_kernel<T, M, 1, false, false, N><<<grid, kGfBlkThreads, 0, s>>>(a);
    } else {
      if (dense) gf_block_kernel<T, M, 1, true, true, N><<<grid, kGfBlkThreads, 0, s>>>(a);
      else gf_block_kernel<T, M, 1, true, false, N><<<grid, kGfBlkThreads, 0, s>>>(a);
    }
    a.in = ab;
    a.out = y;
    gf_block_kernel<T, M, 2, false, true, N><<<grid, kGfBlkThreads, 0, s>>>(a);
  };
  if (a.rb > kGfRowsMax) passes(std::true_type{});
  else passes(std::false_type{});
}

// Blocks of 4 and 8 columns take gf_block_kernel where it is the faster one,
// else, as other sizes do, gf_box_kernel (in groups of up to 4 columns, FP32 8).
// The strips' idle columns cost gf_block_kernel as much as those in use, so the
// lines lie at parts of the strips in use.  Its time over the other's, r = 2 and
// 8, 4 to 770 columns, 60 to 120000 rows:
// - up to 5 rows per workgroup, where latency bounds both: 0.45 to 1.03 at any
//   width, but for FP64, m = 4, r = 8 where its workgroups (20 rows walked for 4)
//   are more than the CUs and the other's waves no more than the SIMDs: 1.01 to
//   1.145 (fewer workgroups 0.70 to 0.89, more waves 0.92 to 1.10, r = 7 0.75 to
//   0.94); 7 rows: 0.68 to 1.0 at a quarter or more in use, 0.9 to 1.2 below;
//   10 rows: 0.53 to 1.0 from 0.55 on, up to 1.1 at 0.5, 1.4 at 0.03;
// - more rows, FP32, m = 4: one strip 0.76 to 1.01 from 0.7 on and up to 1.36 at
//   0.5, several 0.71 to 1.05 from 0.78 on and up to 1.5 at 0.5;
// - FP32, m = 8: one strip 0.7 to 1.04 from 0.5 on and up to 1.3 at 0.45, several
//   0.63 to 1.0 from 0.66 on and up to 1.2 at 0.5;
// - FP64, m = 4: one strip 0.73 to 0.99 from 0.45 on and up to 1.25 at 0.25,
//   several 0.8 to 1.08 from 0.7 on and up to 1.33 at 0.5;
// - FP64, m = 8 (two calls of the other kernel): 0.5 to 0.95 from 0.25 on, 1.1
//   to 2.6 below 0.2;
// - signals: 0.4 to 0.94 from 65536 samples on, about 1.0 below (FP64, m = 8:
//   0.5 to 0.75 at any length).
template <typename T>
bool gf_block_pays(const Operator& op, int m) {
  if (m != 4 && m != 8) return false;
  const bool f64 = sizeof(T) == 8;
  if (op.desc.ndim == 1) return op.n >= 65536 || (f64 && m == 8);
  const GfBlkGrid g = gf_block_grid(op);
  if (g.rb <= 5) {
    if (!f64 || m != 4 || op.desc.radius != 8) return true;
    const dim3 box = gf_grid<GfCpl<4>::v>(op, gf_geom<GfCpl<4>::v>(op));
    const int64_t groups = (int64_t)g.strips * ((op.rows + g.rb - 1) / g.rb), waves = (int64_t)box.x * box.y;
    return groups <= 256 || waves > 1024;
  }
  const bool one = g.strips == 1;
  double least;
  if (m == 8) least = f64 ? 0.25 : (one ? 0.5 : 0.66);
  else least = f64 ? (one ? 0.45 : 0.7) : (one ? 0.7 : 0.78);
  if (g.rb <= 10 && least > 0.55) least = 0.55;
  if (g.rb <= 7) least = 0.25;
  return (double)op.cols >= least * ((double)g.strips * g.ow);
}

double gf_omega(const Operator& op) {
  const double w = 2.0 * op.desc.radius + 1.0;
  return op.desc.ndim == 1 ? w : w * w;
}

template <typename T, int M>
void gf_apply_group(const Operator& op, T* ab, int form, const T* x, int64_t ldx, T* y, int64_t ldy,
                    hipStream_t s) {
  constexpr int C = GfCpl<M>::v;
  const GfGeom geo = gf_geom<C>(op);
  const dim3 grid = gf_grid<C>(op, geo);
  if (form == GSF_FORM_RW || form == GSF_FORM_L) {
    GfStage1<T, M, false> p1{x, (int)ldx, (const T*)op.g, nullptr, (const T*)op.mu, (const T*)op.inv, ab};
    gf_box_kernel<GfStage1<T, M, false>, C><<<grid, kGfLanes, 0, s>>>(p1, geo);
  } else {
    GfStage1<T, M, true> p1{x, (int)ldx, (const T*)op.g, (const T*)op.diag, (const T*)op.mu, (const T*)op.inv, ab};
    gf_box_kernel<GfStage1<T, M, true>, C><<<grid, kGfLanes, 0, s>>>(p1, geo);
  }
  GfStage2<T, M> p2{ab, (const T*)op.g, x, (int)ldx, y, (int)ldy, form, 1.0 / sqrt(gf_omega(op))};
  gf_box_kernel<GfStage2<T, M>, C><<<grid, kGfLanes, 0, s>>>(p2, geo);
}

template <typename T>
void gf_apply_typed(const Operator& op, void* scratch, int form, int m, const T* x, int64_t ldx, T* y, int64_t ldy,
                    hipStream_t s) {
  T* ab = (T*)scratch;
  // (gf_block_kernel takes the coefficients in 16-byte pieces: not in an
  // operator workspace off the 16-byte grid)
  if ((uintptr_t)ab % 16 == 0 && gf_block_pays<T>(op, m)) {
    if (m == 8) gf_apply_block<T, 8>(op, ab, form, x, ldx, y, ldy, s);
    else gf_apply_block<T, 4>(op, ab, form, x, ldx, y, ldy, s);
    return;
  }
  int c = 0;
  while (c < m) {
    const int left = m - c;
    if (left >= 8 && sizeof(T) == 4) {
      gf_apply_group<T, 8>(op, ab, form, x + c, ldx, y + c, ldy, s);
      c += 8;
    } else if (left >= 4) {
      gf_apply_group<T, 4>(op, ab, form, x + c, ldx, y + c, ldy, s);
      c += 4;
    } else if (left >= 2) {
      gf_apply_group<T, 2>(op, ab, form, x + c, ldx, y + c, ldy, s);
      c += 2;
    } else {
      gf_apply_group<T, 1>(op, ab, form, x + c, ldx, y + c, ldy, s);
      c += 1;
    }
  }
}

}  // namespace

gsf_status launch_gf_apply_fused(const Operator& op, int form, const float* x, int64_t ldx, float* y, int64_t ldy,
                                 double* dots, hipStream_t s);
int gf_fused_groups(const Operator& op);

// One FP32 column: the one-pass kernel (apply_gf_fused.hip).  Blocks and FP64
// data: the two passes above; scratch: 2 * kMaxBlock planes of n elements
// (a, b of up to 8 columns).  dots (nullable, one FP32 column only): x^T y
// partials, *nparts of them (gf_dot_parts).
gsf_status launch_gf_apply(const Operator& op, void* scratch, int form, int m, const void* x, int64_t ldx,
                           void* y, int64_t ldy, double* dots, int* nparts, hipStream_t s) {
  if (op.desc.prec == GSF_F32 && m == 1) {
    if (nparts != nullptr) *nparts = gf_fused_groups(op);
    return launch_gf_apply_fused(op, form, (const float*)x, ldx, (float*)y, ldy, dots, s);
  }
  if (op.desc.prec == GSF_F32)
    gf_apply_typed<float>(op, scratch, form, m, (const float*)x, ldx, (float*)y, ldy, s);
  else
    gf_apply_typed<double>(op, scratch, form, m, (const double*)x, ldx, (double*)y, ldy, s);
  return launch_status();
}

// Partials that the one-column apply can write beside its output, 0 where it
// writes none (FP64 data).
int gf_dot_parts(const Operator& op) { return op.desc.prec == GSF_F32 ? gf_fused_groups(op) : 0; }

gsf_status launch_gf_build(const Operator& op, const void* guidance, hipStream_t s) {
  const GfGeom geo = gf_geom<2>(op);
  const dim3 grid = gf_grid<2>(op, geo);
  if (op.desc.prec == GSF_F32) {
    GfStats<float> p{(const float*)guidance, (float*)op.g, (float*)op.mu, (float*)op.inv,
                     (float*)op.sqd, (float*)op.diag, op.deg, op.desc.gf_eps, gf_omega(op)};
    gf_box_kernel<GfStats<float>, 2><<<grid, kGfLanes, 0, s>>>(p, geo);
  } else {
    GfStats<double> p{(const double*)guidance, (double*)op.g, (double*)op.mu, (double*)op.inv,
                      (double*)op.sqd, (double*)op.diag, op.deg, op.desc.gf_eps, gf_omega(op)};
    gf_box_kernel<GfStats<double>, 2><<<grid, kGfLanes, 0, s>>>(p, geo);
  }
  return launch_status();
}

}  // namespace gsf

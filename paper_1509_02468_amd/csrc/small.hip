// Small 1D signals in one workgroup: when a signal fits in LDS, the whole
// filter runs in one launch (the multi-kernel path pays a few launches and a
// grid-wide reduction per step, which dominate at a few thousand samples).
//
// Re-guided BF power filter (Sections 2-3, eq. (3) with the previous result
// as the guidance): each pass evaluates the weights of eq. (2) from the
// current iterate and takes x_i <- x_i - (1/d_i) sum_j w_ij (x_i - x_j), the
// random-walk form D^-1 W x of the chosen normalisation (d_i = 1 + sum_j w_ij
// with the self-loop, or diag L_i = sum_{j != i} w_ij, taken as 1 where it is
// 0).  Weights and sums are FP64; the iterate is stored in the data type after
// every pass (the guidance of the next pass is the stored iterate).
#include <cmath>

#include "gsf_internal.h"
#include "solver_state.h"

namespace gsf {
namespace {

constexpr int kSmallThreads = 1024;

template <typename T>
struct SmallMax {
  static constexpr int n = 65536 / (int)sizeof(T);  // two buffers in 128 KB of LDS
};

template <typename T>
__global__ void __launch_bounds__(kSmallThreads) rg_power1d_small_kernel(const T* __restrict__ x0,
                                                                         T* __restrict__ xout, int n, int kmax,
                                                                         int r, double cs, double cr, int diagl) {
  __shared__ T buf[2 * SmallMax<T>::n];
  T* a = buf;
  T* b = buf + SmallMax<T>::n;
  for (int i = threadIdx.x; i < n; i += blockDim.x) a[i] = x0[i];
  __syncthreads();
  for (int k = 0; k < kmax; ++k) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const double gi = (double)a[i];
      double acc = 0.0, ws = 0.0;
      for (int o = 1; o <= r; ++o) {
        const double sp = (double)(o * o) * cs;
        if (i + o < n) {
          const double dg = gi - (double)a[i + o];
          const double w = exp(-(sp + dg * dg * cr));
          ws += w;
          acc = fma(w, dg, acc);
        }
        if (i - o >= 0) {
          const double dg = gi - (double)a[i - o];
          const double w = exp(-(sp + dg * dg * cr));
          ws += w;
          acc = fma(w, dg, acc);
        }
      }
      double d = diagl ? ws : 1.0 + ws;
      if (d == 0.0) d = 1.0;
      b[i] = (T)(gi - acc / d);
    }
    __syncthreads();
    T* t = a;
    a = b;
    b = t;
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) xout[i] = a[i];
}

inline double inv_two_sigma2(double s) { return std::isinf(s) ? 0.0 : 1.0 / (2.0 * s * s); }

// CG filter (Algorithm 2 in z-space, as gsf_cg_filter) of a built 1D BF
// operator in one workgroup of up to 16 waves: every thread keeps its PTS
// points' z, r, p, q in registers (point i = thread + j threads), u = D^-1/2 v
// is staged in LDS for the neighbour reads, the weights come from the
// operator's planes (own entry at i, mirrored at i - o; the pads are zeros) and
// stay in registers for radii up to RW, and the scalars are FP64 sums.  The
// same recurrences, tests and state as the multi-kernel filter; the state is
// written once at the end.
//
// Bound by the latency of one step's chain: stage u, barrier, stencil, sum of
// p^T q, barrier, alpha, update, two sums, barrier, beta.  As few waves as hold
// the points; a wave hands over the sums of its four rows of 16 lanes, and
// every lane finishes the total itself (rows of 16 lanes, one per wave), so
// that a sum costs one barrier and no broadcast.  500 samples, FP64, 20 steps:
// 21.5 us per call, 61.8 with 16 waves of 8 points whatever the length, weights
// read again in every step and three barriers per sum (94 with those sums'
// exchanges through LDS); 4096 samples, r = 1 / 5: 41 / 150 us, 109 / 185
// before; 8192: 97 / 256, 128 / 282.
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kCgSmallMax = 8192;  // samples: 8 per thread
constexpr int kCgPad = 8;          // zeros beside u: the largest radius whose weights stay in registers or less

// The wave's NV values to its row of part: row sums of 16 lanes each (the
// wave's four), unused waves' entries are zeros.
template <int NV>
__device__ __forceinline__ void post_rows(double (&v)[NV], double (*part)[kSmallWaves][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<8>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<4>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<2>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<1>(v[k]);
  if ((lane & 15) == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) part[k][wave][lane >> 4] = v[k];
  }
}

// After a barrier: the workgroup's totals, bitwise the same in every lane.
template <int NV>
__device__ __forceinline__ void take_totals(double (&v)[NV], double (*part)[kSmallWaves][4]) {
  const int w = threadIdx.x & 15;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double* p = part[k][w];
    v[k] = (p[0] + p[1]) + (p[2] + p[3]);
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<8>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<4>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<2>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] += row_rotate<1>(v[k]);
}

// PTS: points per thread; RW: the weights of radii up to RW stay in registers
// (0: read in every apply, any radius).
template <typename T, int PTS, int RW>
__global__ void __launch_bounds__(kSmallThreads) cg1d_small_kernel(const T* __restrict__ planes, int64_t pstride,
                                                                   int64_t ppad, int r, const T* __restrict__ isqd,
                                                                   const T* __restrict__ sqd,
                                                                   const T* __restrict__ x0, T* __restrict__ xout,
                                                                   int n, int kmax, CgState init, CgState* st) {
  __shared__ T ubuf[kSmallThreads * PTS + 2 * kCgPad];
  __shared__ T zb[PTS < 8 ? 1 : kSmallThreads * PTS];  // z where the registers have no room for it
  __shared__ __align__(16) double part_q[1][kSmallWaves][4], part_r[2][kSmallWaves][4];
  T* u = ubuf + kCgPad;
  int tid = threadIdx.x;
  const int nt = blockDim.x;
  T z[PTS < 8 ? PTS : 1], rv[PTS], p[PTS], q[PTS], is[PTS];
  T wo[RW > 0 ? RW : 1][PTS], wm[RW > 0 ? RW : 1][PTS];
  auto zr = [&](int j) -> T& {
    if constexpr (PTS < 8) return z[j];
    else return zb[tid + j * nt];
  };
  // q = L_sym v: stage u = D^-1/2 v, then q_i = is_i sum_o w (u_i - u_j)
  auto apply = [&](const T (&v)[PTS]) {
    // eight points' indexes and addresses, kept over the steps, would spill
    if constexpr (PTS >= 8) __asm__ volatile("" : "+v"(tid));
#pragma unroll
    for (int j = 0; j < PTS; ++j) {
      const int i = tid + j * nt;
      if (i < n) u[i] = v[j] * is[j];
    }
    __syncthreads();
    if constexpr (RW > 0) {
      // radii up to RW <= kCgPad: the neighbours off the signal are the pads'
      // zeros, under zero weights
#pragma unroll
      for (int j = 0; j < PTS; ++j) {
        const int i = tid + j * nt;
        T acc = T(0);
        if (i < n) {
          // the rounded u_i that the neighbours read: contracted into the
          // differences the product would keep its low bits, and u_i - u_j no
          // longer be the negative of u_j - u_i (FP32 errors twice as large)
          T ui = v[j] * is[j];
          __asm__ volatile("" : "+v"(ui));
#pragma unroll
          for (int o = 1; o <= RW; ++o) {
            if (o > r) break;
            acc = fma(wo[o - 1][j], ui - u[i + o], acc);
            acc = fma(wm[o - 1][j], ui - u[i - o], acc);
          }
        }
        q[j] = is[j] * acc;
      }
    } else {
      // an offset's weights of G points are requested together
      constexpr int G = PTS < 8 ? PTS : (sizeof(T) == 4 ? 4 : 2);
#pragma unroll
      for (int j0 = 0; j0 < PTS; j0 += G) {
        T acc[G];
#pragma unroll
        for (int j = 0; j < G; ++j) acc[j] = T(0);
        for (int o = 1; o <= r; ++o) {
          const T* pl = planes + ppad + (int64_t)(o - 1) * pstride;
          T own[G], mir[G];
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const int i = tid + (j0 + j) * nt, ic = i < n ? i : 0;
            own[j] = pl[ic];
            mir[j] = pl[ic - o];
          }
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const int i = tid + (j0 + j) * nt;
            if (i < n) {
              const T ui = u[i];
              const T uo = i + o < n ? u[i + o] : T(0);
              const T um = i - o >= 0 ? u[i - o] : T(0);
              acc[j] = fma(own[j], ui - uo, acc[j]);
              acc[j] = fma(mir[j], ui - um, acc[j]);
            }
          }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) q[j0 + j] = is[j0 + j] * acc[j];
      }
    }
  };
  for (int i = tid; i < kSmallWaves * 4; i += nt) part_q[0][0][i] = part_r[0][0][i] = part_r[1][0][i] = 0.0;
  if (tid < kCgPad) {
    ubuf[tid] = T(0);
    u[n + tid] = T(0);
  }
  double zz = 0.0, rho = 0.0;
#pragma unroll
  for (int j = 0; j < PTS; ++j) {
    const int i = tid + j * nt;
    is[j] = i < n ? isqd[i] : T(0);
    p[j] = i < n ? x0[i] * sqd[i] : T(0);
    zr(j) = p[j];
    if constexpr (RW > 0) {
#pragma unroll
      for (int o = 1; o <= RW; ++o) {
        const T* pl = planes + ppad + (int64_t)(o - 1) * pstride;
        wo[o - 1][j] = o <= r && i < n ? pl[i] : T(0);
        wm[o - 1][j] = o <= r && i < n ? pl[i - o] : T(0);
      }
    }
    zz += (double)p[j] * (double)p[j];
  }
  const double tol = init.tol, tau = init.tau;
  apply(p);
#pragma unroll
  for (int j = 0; j < PTS; ++j) {
    rv[j] = -q[j];
    rho += (double)rv[j] * (double)rv[j];
  }
  {
    double t[2] = {rho, zz};
    post_rows<2>(t, part_r);
    __syncthreads();
    take_totals<2>(t, part_r);
    rho = t[0];
    zz = t[1];
  }
  const double floor = tau * tau * zz;
  const double tol2 = tol > 0.0 ? tol * tol * rho : -1.0;
  const double rho0 = rho;
  int status = GSF_OK, active = 1, iters = 0;
  if (!(__builtin_isfinite(rho) && rho > floor)) {
    status = GSF_EBREAKDOWN;
    active = 0;
  } else if (tol2 > 0.0 && rho <= tol2) {
    active = 0;
  }
  double beta = 0.0;
  for (int k = 1; k <= kmax && active; ++k) {
#pragma unroll
    for (int j = 0; j < PTS; ++j) p[j] = k == 1 ? rv[j] : rv[j] + (T)beta * p[j];
    // (a barrier lies between the last apply's reads of u and its new values:
    // those of the sums)
    apply(p);
    double t[1] = {0.0};
#pragma unroll
    for (int j = 0; j < PTS; ++j) t[0] += (double)p[j] * (double)q[j];
    post_rows<1>(t, part_q);
    __syncthreads();
    take_totals<1>(t, part_q);
    const double pq = t[0];
    if (!(__builtin_isfinite(pq) && pq > 0.0)) {
      status = GSF_EBREAKDOWN;
      active = 0;
      break;
    }
    const T alpha = (T)(rho / pq);
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < PTS; ++j) {
      zr(j) += alpha * p[j];
      const T ro = rv[j];
      const T rn = ro - alpha * q[j];
      rv[j] = rn;
      s[0] += (double)rn * (double)rn;
      s[1] += (double)rn * (double)ro;
    }
    post_rows<2>(s, part_r);
    __syncthreads();
    take_totals<2>(s, part_r);
    beta = (s[0] - s[1]) / rho;
    rho = s[0];
    iters = k;
    if (!(__builtin_isfinite(rho) && rho > floor)) {
      status = GSF_EBREAKDOWN;
      active = 0;
    } else if (tol2 > 0.0 && rho <= tol2) {
      active = 0;
    }
  }
#pragma unroll
  for (int j = 0; j < PTS; ++j) {
    const int i = tid + j * nt;
    if (i < n) xout[i] = zr(j) / sqd[i];
  }
  if (tid == 0) {
    init.rho = rho;
    init.rho0 = rho0;
    init.res0 = sqrt(rho0 > 0.0 ? rho0 : 0.0);
    init.floor = floor;
    init.tol2 = tol2;
    init.iters = iters;
    init.k = iters + 1;
    init.status = status;
    init.active = active;
    *st = init;
  }
}

template <typename T, int PTS, int RW>
void launch_cg1d(const Operator& op, const void* x0, void* x_out, int kmax, const CgState& init, CgState* st,
                 hipStream_t s) {
  // as few waves as hold the points; at eight points per thread at least three per
  // SIMD, whose apply reads weights and neighbours (4097 samples, FP32, 10 steps,
  // r = 8: 99 us, 109 with nine waves, 102 with sixteen; r = 1 35, 36, 40)
  constexpr int kLeast = PTS < 8 ? 64 : 768;
  const int per = (int)((op.n + PTS - 1) / PTS), full = (per + 63) / 64 * 64, threads = full < kLeast ? kLeast : full;
  cg1d_small_kernel<T, PTS, RW><<<1, threads, 0, s>>>((const T*)op.planes, op.pstride, op.ppad, op.desc.radius,
                                                      (const T*)op.diag, (const T*)op.sqd, (const T*)x0,
                                                      (T*)x_out, (int)op.n, kmax, init, st);
}

// The fewest points per thread that 1024 threads hold; the weights in
// registers as long as 16 waves' registers have room for them (2048 samples,
// FP64: r = 5 in registers 44 us, r = 8 read in every step 118).
template <typename T>
void launch_cg1d_t(const Operator& op, const void* x0, void* x_out, int kmax, const CgState& init, CgState* st,
                   hipStream_t s) {
  const int r = op.desc.radius;
  const int64_t per = (op.n + kSmallThreads - 1) / kSmallThreads;
  if (per <= 1) {
    if (r <= 2) launch_cg1d<T, 1, 2>(op, x0, x_out, kmax, init, st, s);
    else launch_cg1d<T, 1, 8>(op, x0, x_out, kmax, init, st, s);
  } else if (per <= 2) {
    if (r <= 2) launch_cg1d<T, 2, 2>(op, x0, x_out, kmax, init, st, s);
    else if (r <= 5) launch_cg1d<T, 2, 5>(op, x0, x_out, kmax, init, st, s);
    else launch_cg1d<T, 2, 0>(op, x0, x_out, kmax, init, st, s);
  } else if (per <= 4) {
    if (r <= 2) launch_cg1d<T, 4, 2>(op, x0, x_out, kmax, init, st, s);
    else launch_cg1d<T, 4, 0>(op, x0, x_out, kmax, init, st, s);
  } else {
    launch_cg1d<T, 8, 0>(op, x0, x_out, kmax, init, st, s);
  }
}

}  // namespace

// One-launch re-guided BF power filter for a 1D signal that fits in LDS;
// false (nothing launched) when the descriptor is not of that kind.
bool launch_rg_power_small(const gsf_operator_desc& d, const void* x0, void* x_out, int kmax, hipStream_t s) {
  const int64_t n = d.dims[0];
  if (d.kind != GSF_BF || d.ndim != 1 || desc_channels(d) != 1 || kmax < 1) return false;
  const double cs = inv_two_sigma2(d.sigma_d), cr = inv_two_sigma2(d.sigma_r);
  const int diagl = d.norm == GSF_NORM_DIAGL ? 1 : 0;
  if (d.prec == GSF_F32) {
    if (n > SmallMax<float>::n) return false;
    rg_power1d_small_kernel<float><<<1, kSmallThreads, 0, s>>>((const float*)x0, (float*)x_out, (int)n, kmax,
                                                               d.radius, cs, cr, diagl);
  } else {
    if (n > SmallMax<double>::n) return false;
    rg_power1d_small_kernel<double><<<1, kSmallThreads, 0, s>>>((const double*)x0, (double*)x_out, (int)n, kmax,
                                                                d.radius, cs, cr, diagl);
  }
  return true;
}

// One-launch CG filter of a built 1D BF operator whose signal fits in one
// workgroup (n <= 8192); false (nothing launched) otherwise.  init: the state
// with tol and tau; the kernel writes *st whole, so that no launch sets it first
// (500 samples, 20 steps: 21.5 us per call, 21.8 with one).
bool launch_cg_small(const Operator& op, const void* x0, void* x_out, int kmax, const CgState& init, CgState* st,
                     hipStream_t s) {
  if (op.desc.kind != GSF_BF || op.desc.ndim != 1 || op.n > kCgSmallMax) return false;
  if (op.desc.prec == GSF_F32)
    launch_cg1d_t<float>(op, x0, x_out, kmax, init, st, s);
  else
    launch_cg1d_t<double>(op, x0, x_out, kmax, init, st, s);
  return true;
}

}  // namespace gsf

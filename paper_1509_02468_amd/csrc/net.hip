// Learned preconditioner T for block LOBPCG (the preconditioner slot of
// Algorithm 3): a 3-layer 3x3 convolutional network
//   x = (bf16(r / s), bf16(g)),  a1 = bf16(relu(conv(x; W1))),  2 -> 16
//   a2 = bf16(relu(conv(a1; W2))),  16 -> 16,   y = conv(a2; W3),  16 -> 1
// with zero padding, no biases, s = RMS(r), T(r) = s * y.  BF16 weights and
// activations, FP32 accumulation.  Flat weight layout: W1[o][c][ky][kx]
// (offset 0), W2[o][c][ky][kx] (offset 288), W3[c][ky][kx] (offset 2592).
//
// Training (loss and weight gradient) is in net_train.hip, Adam here;
// inference inside LOBPCG runs on one fused kernel per 30x30 output tile that
// keeps the whole receptive field in LDS and does the three convolutions as
// implicit GEMMs on bf16 MFMA, 16 output channels x 16 pixels per instruction
// (layers 1 and 2 v_mfma_f32_16x16x32_bf16; layer 3 v_mfma_f32_16x16x16bf16_1k,
// as 9 per-tap 1x1 products summed over the taps).
#include <cmath>

#include "net_common.h"
#include "solver_state.h"

namespace gsf {

int vec_blocks(int64_t n);

namespace {

// FP32 -> BF16, round to nearest, ties to even (NaN stays NaN).
__device__ __forceinline__ uint32_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
// FP64 -> BF16 with a single rounding: the FP32 conversion can create an
// exact BF16 tie that the FP64 value does not have; then the FP32 value is
// moved one unit towards the FP64 value, so the tie breaks the right way.
__device__ __forceinline__ uint32_t d2bf(double d) {
  const float f = (float)d;
  uint32_t u = __float_as_uint(f);
  if ((u & 0xffffu) == 0x8000u && (double)f != d && __builtin_isfinite(f))
    u = fabs(d) > fabs((double)f) ? u + 1u : u - 1u;
  return f2bf(__uint_as_float(u));
}

// ---------------------------------------------------------------------------
// optimiser (the training pass is in net_train.hip)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) net_adam_kernel(int64_t count, float b1, float b2, float eps,
                                                            float step, float bc1, float bc2, float* __restrict__ w,
                                                            float* __restrict__ mom, float* __restrict__ vel,
                                                            const float* __restrict__ grad,
                                                            uint16_t* __restrict__ wb) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const float g = grad[i];
    const float m = b1 * mom[i] + (1.0f - b1) * g;
    const float v = b2 * vel[i] + (1.0f - b2) * g * g;
    mom[i] = m;
    vel[i] = v;
    const float wn = w[i] - step * (m / bc1) / (sqrtf(v / bc2) + eps);
    w[i] = wn;
    wb[i] = (uint16_t)f2bf(wn);
  }
}

__global__ void __launch_bounds__(kThreads) net_to_bf16_kernel(int64_t count, const float* __restrict__ w,
                                                               uint16_t* __restrict__ wb) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    wb[i] = (uint16_t)f2bf(w[i]);
}

// ---------------------------------------------------------------------------
// fused inference
// ---------------------------------------------------------------------------
// A tile of 30 x 30 outputs keeps the region each layer needs in LDS: the
// input (36 x 36), a1 (34 x 34) and the nine per-tap products of layer 3 over
// the 32 x 32 pixels of a2, which themselves stay in registers (64 groups of
// 16 pixels, so that layer 2 needs no division for a pixel's row).
constexpr int kOT = 30;             // output tile side
constexpr int kA2 = kOT + 2;        // layer-2 output region side (32)
constexpr int kA1 = kOT + 4;        // layer-1 output region side (34)
constexpr int kXS = kOT + 6;        // input region side (36)
constexpr int kA2N = kA2 * kA2;
constexpr int kA1N = kA1 * kA1;
constexpr int kXN = kXS * kXS;
constexpr int kA1G = (kA1N + 15) / 16, kA2G = kA2N / 16;  // groups of 16 pixels
constexpr int kA1P = kA1G * 16;     // pixels of an a1 plane
constexpr int kC3P = kA2N + 4;      // pitch of a tap's products: lane groups q store taps 4q.. 16 banks apart

struct NetInferArgs {
  const uint16_t* w;       // BF16 weights (flat layout)
  const void* R;           // n x m, point-major
  void* Z;                 // n x m output T(R)
  const void* g;           // guidance, n values
  const void* sqd;         // sqrt(d) (constraint dots), or nullptr
  const double* colnorm;   // ||R_j||
  const LobpcgState* st;   // LOBPCG state (skip when inactive; Y norm), or nullptr
  int64_t rows, cols, n;
  int m;
  int tiles_x, ntiles;
  double* partials;        // [tile][3m]: r_j.w_j, y.w_j, non-finite count
};

__device__ __forceinline__ floatx4_t mfma_bf16(short4_t a, short4_t b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

constexpr int kNetThreads = 512;    // 8 waves per tile
constexpr int kNetWaves = kNetThreads / 64;
constexpr int kXIter = (kXN + kNetThreads - 1) / kNetThreads;
constexpr int kOIter = (kOT * kOT + kNetThreads - 1) / kNetThreads;

// One tile of all m columns.  Per column two phases, with one barrier between:
//   layer 2 of column j (a1 -> c3, the layer-3 products) and the input of
//   column j + 1 (R / s to BF16);   output of column j and layer 1 of j + 1.
// Layers 1 and 2 run on v_mfma_f32_16x16x32_bf16: K = 32 holds all nine taps
// of the two inputs, and two taps of the 16 channels (bitwise the sum of two
// K = 16 products in order).  The ninth tap takes a K = 32 product with a zero
// half too: a K = 16 product that accumulates onto a K = 32 result right after
// it delivers later than the wait before its use allows for (outputs differed
// from run to run), so that the two forms are never chained.
// Bound by vector instructions (conversions, addresses, the FP64 scaling) at
// four waves per SIMD.  An m = 4 block at 2048^2, FP32: 287 us per call, 717
// with 28 x 28 tiles, K = 16 products only, 64-bit coordinates, FP64
// divisions, BF16 rounding by integer operations, the guidance converted
// again for every column and six barriers per column.
struct NetInferShared {
  uint32_t xs[kXN + 4];                       // (r/s, g) as a BF16 pair per pixel, and a zero
  __align__(16) char a1[2 * kA1P * 16];       // layer-1 output [channel half][pixel][8]
  float c3[9 * kC3P];                         // layer-3 products [tap][pixel]
  double red[kMaxBlock * 3 * kNetWaves];
};

// INNER: the tile and its halo lie on the image.
template <typename T, bool INNER>
__device__ __forceinline__ void net_infer_tile(const NetInferArgs& a, NetInferShared& sh, int ty, int tx) {
  uint32_t* xs = sh.xs;
  char* a1s = sh.a1;
  float* c3 = sh.c3;
  double* red = sh.red;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, l16 = lane & 15, half = q & 1, sel = q >> 1;
  const int rows = (int)a.rows, cols = (int)a.cols;
  const int y0 = ty * kOT, x0 = tx * kOT;
  auto on_image = [&](int gy, int gx) { return INNER || ((unsigned)gy < (unsigned)rows && (unsigned)gx < (unsigned)cols); };

  const T* R = (const T*)a.R;
  T* Z = (T*)a.Z;
  const T* G = (const T*)a.g;
  const T* sqd = (const T*)a.sqd;
  const double yinv = (a.st != nullptr && sqd != nullptr) ? a.st->ynorm_inv : 0.0;
  const double rn = sqrt((double)a.n);
  const int m = a.m;

  // the thread's input pixels: offset (or -1) and guidance, alike for every column
  int64_t xi[kXIter];
  uint32_t gv[kXIter];
  T rv[kXIter];
  auto load_r = [&](int j) {
#pragma unroll
    for (int k = 0; k < kXIter; ++k) rv[k] = R[(xi[k] >= 0 ? xi[k] : 0) + j];
  };
  T g0[kXIter];
#pragma unroll
  for (int k = 0; k < kXIter; ++k) {
    const int e = tid + k * kNetThreads;
    const int ey = div_px<kXS, kXIter * kNetThreads>(e), gy = y0 - 3 + ey, gx = x0 - 3 + e - __mul24(ey, kXS);
    const bool in = e < kXN && on_image(gy, gx);
    const int64_t i = in ? (int64_t)gy * cols + gx : -1;
    xi[k] = i >= 0 ? i * m : -1;
    g0[k] = G[i >= 0 ? i : 0];
  }
  load_r(0);
  // The weights, through LDS (the products' space): every lane of eight waves
  // takes 52 of them, and from memory those loads of two bytes, far apart, took
  // as long as two columns' work (2048^2, FP32: m = 1 200 -> 116 us, m = 4
  // 371 -> 287).
  uint16_t* ws = (uint16_t*)c3;
  {
    constexpr int kWIter = (kNetWeights + kNetThreads - 1) / kNetThreads;
    uint16_t wv[kWIter];
#pragma unroll
    for (int k = 0; k < kWIter; ++k) {
      const int e = tid + k * kNetThreads;
      wv[k] = a.w[e < kNetWeights ? e : 0];
    }
#pragma unroll
    for (int k = 0; k < kWIter; ++k)
      if (tid + k * kNetThreads < kNetWeights) ws[tid + k * kNetThreads] = wv[k];
  }
  lds_barrier();
  // MFMA A operands (weights): lane holds A[row = l16][k]; k = 8q + i (K = 32), 4q + i (K = 16)
  uint4_t w1, w2[5];
  short4_t w3a;
  {
    auto pack = [](const uint32_t (&v)[8]) {
      return uint4_t{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
    };
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int tap = 4 * q + (i >> 1);
      v[i] = tap < 9 ? ws[kOffW1 + l16 * 18 + (i & 1) * 9 + tap] : 0u;
    }
    w1 = pack(v);
#pragma unroll
    for (int t = 0; t < 5; ++t) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[i] = 2 * t + sel < 9 ? ws[kOffW2 + l16 * 144 + (8 * half + i) * 9 + 2 * t + sel] : 0u;
      w2[t] = pack(v);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w3a[i] = l16 < 9 ? (short)ws[kOffW3 + (4 * q + i) * 9 + l16] : (short)0;
    }
  }
  // layer-1 B operand: the lane's taps 4q + i, past the last one the zero word
  int xo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tap = 4 * q + i;
    xo[i] = tap < 9 ? (tap / 3) * kXS + tap % 3 : -1;
  }

#pragma unroll
  for (int k = 0; k < kXIter; ++k) gv[k] = xi[k] >= 0 ? d2bf((double)g0[k]) << 16 : 0u;
  auto put_x = [&](int j) {
    const double s = a.colnorm[j] / rn, inv = s > 0.0 ? 1.0 / s : 0.0;
#pragma unroll
    for (int k = 0; k < kXIter; ++k) {
      const int e = tid + k * kNetThreads;
      const uint32_t v = xi[k] >= 0 ? (s > 0.0 ? d2bf((double)rv[k] * inv) : 0u) | gv[k] : 0u;
      if (e < kXN) xs[e] = v;
    }
  };
  // the groups of 16 pixels of a1 and the rows of a2 that are worked on: all of
  // them, or, in a tile with less than half of its rows on the image, those; the
  // others' a1 and layer-3 products are zeros (1 x 100000, m = 4: 232 -> 152 us)
  const int top = y0 < 2 ? 2 - y0 : 0, bottom = rows - y0 + 2 < kA1 ? rows - y0 + 2 : kA1;
  const bool thin = !INNER && 2 * (bottom - top) < kA1;
  const int ga = thin ? top * kA1 / 16 : 0, gb = thin ? (bottom * kA1 + 15) / 16 : kA1G;
  const int pa = thin && top > 1 ? top - 1 : 0, pb = thin && bottom - 1 < kA2 ? bottom - 1 : kA2;
  if (thin) {
    const uint4_t zero4 = {0u, 0u, 0u, 0u};
    for (int e = tid; e < 2 * kA1P; e += kNetThreads) *(uint4_t*)(a1s + 16 * e) = zero4;
  }
  auto layer1 = [&]() {
#pragma unroll 5
    for (int g = ga + wave; g < gb; g += kNetWaves) {
      const int p = g * 16 + l16, pc = p < kA1N ? p : kA1N - 1;
      const int py = div_px<kA1, kA1P>(pc), px = pc - __mul24(py, kA1);
      const int base = __mul24(py, kXS) + px;
      uint4_t b;
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] = xs[xo[i] >= 0 ? base + xo[i] : kXN];
      const floatx4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
      const floatx4_t c = mfma_bf16_k32(w1, b, zero);
      const bool in = on_image(y0 - 2 + py, x0 - 2 + px);
      uint2 u;
      u.x = in ? pack2(relu(c[0]), relu(c[1])) : 0u;
      u.y = in ? pack2(relu(c[2]), relu(c[3])) : 0u;
      *(uint2*)(a1s + (sel * kA1P + p) * 16 + half * 8) = u;
    }
  };

  if (tid == 0) xs[kXN] = 0u;
  put_x(0);
  lds_barrier();
  if (thin)
    for (int e = tid; e < 9 * kC3P; e += kNetThreads) c3[e] = 0.0f;
  if (m > 1) load_r(1);
  layer1();
  lds_barrier();
#pragma unroll 1
  for (int j = 0; j < m; ++j) {
    // R at the output pixels, for r . w: asked for here, used after layer 2
    T ro[kOIter];
#pragma unroll
    for (int k = 0; k < kOIter; ++k) {
      const int e = tid + k * kNetThreads;
      const int oy = div_px<kOT, kOIter * kNetThreads>(e), gy = y0 + oy, gx = x0 + e - __mul24(oy, kOT);
      const bool in = e < kOT * kOT && (INNER || (gy < rows && gx < cols));
      ro[k] = R[in ? ((int64_t)gy * cols + gx) * m + j : 0];
    }
    // layer 2 (16 -> 16 channels, two taps per product) and layer 3 as nine
    // per-tap products c3[tap][p] = sum_c W3[c][tap] a2[p][c]
#pragma unroll 4
    for (int g = 2 * pa + wave; g < 2 * pb; g += kNetWaves) {
      const int py = g >> 1, px = (g & 1) * 16 + l16;
      const char* b = a1s + (half * kA1P + py * kA1 + px) * 16;
      const char* b1 = b + sel * 16;              // taps (0, 1), (4, 5), (6, 7)
      const char* b2 = b + sel * (kA1 - 2) * 16;  // taps (2, 3)
      floatx4_t c = {0.0f, 0.0f, 0.0f, 0.0f};
      c = mfma_bf16_k32(w2[0], *(const uint4_t*)b1, c);
      c = mfma_bf16_k32(w2[1], *(const uint4_t*)(b2 + 2 * 16), c);
      c = mfma_bf16_k32(w2[2], *(const uint4_t*)(b1 + (kA1 + 1) * 16), c);
      c = mfma_bf16_k32(w2[3], *(const uint4_t*)(b1 + 2 * kA1 * 16), c);
      const uint4_t zero4 = {0u, 0u, 0u, 0u};
      const uint4_t last = *(const uint4_t*)(b + (2 * kA1 + 2) * 16);
      c = mfma_bf16_k32(w2[4], sel ? zero4 : last, c);
      const bool in = on_image(y0 - 1 + py, x0 - 1 + px);
      uint2 u;
      u.x = in ? pack2(relu(c[0]), relu(c[1])) : 0u;
      u.y = in ? pack2(relu(c[2]), relu(c[3])) : 0u;
      const floatx4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
      const floatx4_t t = mfma_bf16(w3a, __builtin_bit_cast(short4_t, u), zero);
      float* o = c3 + 4 * q * kC3P + g * 16 + l16;
      if (q < 3) o[0] = t[0];
      if (q < 2) {
        o[kC3P] = t[1];
        o[2 * kC3P] = t[2];
        o[3 * kC3P] = t[3];
      }
    }
    if (j + 1 < m) put_x(j + 1);
    lds_barrier();
    // output: y[o] = sum_tap c3[tap][o + off(tap)], w = s y
    if (j + 2 < m) load_r(j + 2);
    const double s = a.colnorm[j] / rn;
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kOIter; ++k) {
      const int e = tid + k * kNetThreads;
      const int oy = div_px<kOT, kOIter * kNetThreads>(e), ox = e - __mul24(oy, kOT);
      const int gy = y0 + oy, gx = x0 + ox;
      if (e >= kOT * kOT || (!INNER && (gy >= rows || gx >= cols))) continue;
      const float* cp = c3 + oy * kA2 + ox;
      float yv = 0.0f;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) yv += cp[tap * kC3P + (tap / 3) * kA2 + tap % 3];
      const int64_t i = (int64_t)gy * cols + gx;
      const T wt = (T)(s * (double)yv);
      const double r = (double)ro[k];
      Z[i * m + j] = wt;
      const double wd = (double)wt;
      v[0] += r * wd;
      if (sqd != nullptr) v[1] += (double)sqd[i] * yinv * wd;
      if (!__builtin_isfinite(wd)) v[2] += 1.0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k == 1 && sqd == nullptr) continue;
      const double t = wave_sum(v[k]);
      if (lane == 0) red[(3 * j + k) * kNetWaves + wave] = t;
    }
    if (j + 1 < m) layer1();
    lds_barrier();
  }
  // the waves' sums in wave order
  if (tid < 3 * m) {
    double t = 0.0;
    if (sqd != nullptr || tid % 3 != 1)
      for (int wv = 0; wv < kNetWaves; ++wv) t += red[tid * kNetWaves + wv];
    a.partials[(size_t)blockIdx.x * 3 * m + tid] = t;
  }
}

template <typename T>
__global__ void __launch_bounds__(kNetThreads) __attribute__((amdgpu_waves_per_eu(4)))
net_infer_kernel(NetInferArgs a) {
  __shared__ NetInferShared sh;
  if (a.st != nullptr && !a.st->active) return;
  const int tile = xcd_tile(blockIdx.x, a.ntiles);
  const int ty = tile / a.tiles_x, tx = tile - (tile / a.tiles_x) * a.tiles_x;
  const int y0 = ty * kOT, x0 = tx * kOT;
  if (y0 >= 3 && x0 >= 3 && y0 + kOT + 3 <= a.rows && x0 + kOT + 3 <= a.cols)
    net_infer_tile<T, true>(a, sh, ty, tx);
  else
    net_infer_tile<T, false>(a, sh, ty, tx);
}

// LOBPCG: per column, use T(r) unless it has a non-finite entry or
// r^T T(r) <= 0 (then T = I); Y^T T(r) for the constraint projection.
__global__ void __launch_bounds__(kThreads) net_final_kernel(const double* __restrict__ partials, int nparts, int m,
                                                             LobpcgState* st) {
  __shared__ double red[16 * 3];
  if (!st->active) return;
  for (int j = 0; j < m; ++j) {
    double t[3];
    reduce_partials<3>(partials + 3 * j, nparts, 3 * m, t, red);
    if (threadIdx.x == 0) {
      const bool use = t[2] == 0.0 && __builtin_isfinite(t[0]) && t[0] > 0.0 && st->res[j] > 0.0;
      st->tuse[j] = use ? 1 : 0;
      st->yz[j] = t[1];
      if (!use) st->fallbacks += 1;
    }
  }
}

// W <- T(R) or R per column (W holds R on entry), minus its Y component
template <typename T>
__global__ void __launch_bounds__(kThreads) net_select_kernel(T* __restrict__ W, const T* __restrict__ Z,
                                                              const T* __restrict__ sqd, int64_t n, int m,
                                                              int constraint, const LobpcgState* st) {
  if (!st->active) return;
  const double yinv = st->ynorm_inv;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double yi = constraint ? (double)sqd[i] * yinv : 0.0;
    for (int j = 0; j < m; ++j) {
      const bool use = st->tuse[j] != 0;
      double v = use ? (double)Z[i * m + j] : (double)W[i * m + j];
      if (constraint) v -= yi * (use ? st->yz[j] : st->yx[j]);
      W[i * m + j] = (T)v;
    }
  }
}

// Partials of the fallback test for a preconditioner output Z computed
// outside the network kernel: per column r^T z, (Y^T z with Y = sqrt(d) /
// ||sqrt(d)||, when sqd != nullptr) and the count of non-finite entries, in
// the layout net_final_kernel reads (3 values per column, 3m per workgroup).
template <typename T>
__global__ void __launch_bounds__(kThreads) tz_partials_kernel(const T* __restrict__ R, const T* __restrict__ Z,
                                                               const T* __restrict__ sqd, int64_t n, int m,
                                                               const LobpcgState* st, double* __restrict__ partials) {
  __shared__ double red[16 * 3 * kMaxBlock];
  double v[3 * kMaxBlock];
#pragma unroll
  for (int k = 0; k < 3 * kMaxBlock; ++k) v[k] = 0.0;
  const double yinv = sqd != nullptr ? st->ynorm_inv : 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double yi = sqd != nullptr ? (double)sqd[i] * yinv : 0.0;
#pragma unroll
    for (int j = 0; j < kMaxBlock; ++j)
      if (j < m) {
        const double z = (double)Z[i * m + j];
        v[3 * j] += (double)R[i * m + j] * z;
        v[3 * j + 1] += yi * z;
        if (!__builtin_isfinite(z)) v[3 * j + 2] += 1.0;
      }
  }
  block_sum<3 * kMaxBlock>(v, red);
  if (threadIdx.x == 0)
    for (int k = 0; k < 3 * m; ++k) partials[(size_t)blockIdx.x * 3 * m + k] = v[k];
}

// dst[i * ldd] = src[i * lds]
template <typename T>
__global__ void __launch_bounds__(kThreads) col_copy_kernel(const T* __restrict__ src, int64_t lds, T* __restrict__ dst,
                                                            int64_t ldd, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i * ldd] = src[i * lds];
}

// ||R_j||^2 partials of an n x m block
template <typename T>
__global__ void __launch_bounds__(kThreads) colnorm_kernel(const T* __restrict__ R, int64_t n, int m,
                                                           int64_t ld, double* __restrict__ partials) {
  __shared__ double red[16 * kMaxBlock];
  double v[kMaxBlock];
#pragma unroll
  for (int j = 0; j < kMaxBlock; ++j) v[j] = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
#pragma unroll
    for (int j = 0; j < kMaxBlock; ++j)
      if (j < m) {
        const double r = (double)R[i * ld + j];
        v[j] += r * r;
      }
  }
  block_sum<kMaxBlock>(v, red);
  if (threadIdx.x == 0)
    for (int j = 0; j < kMaxBlock; ++j) partials[(size_t)blockIdx.x * kMaxBlock + j] = v[j];
}

__global__ void __launch_bounds__(kThreads) colnorm_final_kernel(const double* __restrict__ partials, int nparts,
                                                                 double* __restrict__ out) {
  __shared__ double red[16 * kMaxBlock];
  double t[kMaxBlock];
  reduce_partials<kMaxBlock>(partials, nparts, kMaxBlock, t, red);
  if (threadIdx.x == 0)
    for (int j = 0; j < kMaxBlock; ++j) out[j] = sqrt(t[j]);
}

// training pair: inputs = (r/s, g), targets = y/s with s = ||r|| / sqrt(n)
template <typename T>
__global__ void __launch_bounds__(kThreads) net_pair_kernel(const T* __restrict__ r, int64_t ldr,
                                                            const T* __restrict__ y, int64_t ldy,
                                                            const T* __restrict__ g, int64_t n,
                                                            const double* __restrict__ norm, float* __restrict__ in,
                                                            float* __restrict__ tg) {
  const double s = norm[0] / sqrt((double)n);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double rs = s > 0.0 ? (double)r[i * ldr] / s : 0.0;
    const double ys = s > 0.0 ? (double)y[i * ldy] / s : 0.0;
    in[2 * i] = (float)rs;
    in[2 * i + 1] = (float)g[i];
    tg[i] = (float)ys;
  }
}

struct Theta8 {
  double v[kMaxBlock];
};

template <typename T>
__global__ void __launch_bounds__(kThreads) residual_kernel(const T* __restrict__ X, T* __restrict__ R, int64_t n,
                                                            int m, Theta8 th) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    for (int j = 0; j < m; ++j) R[i * m + j] = (T)((double)R[i * m + j] - th.v[j] * (double)X[i * m + j]);
}

// ---- shifted CG: (L_sym + alpha I) y = b ---------------------------------
template <typename T>
__global__ void __launch_bounds__(kThreads) scg_init_kernel(const T* __restrict__ b, int64_t ldb,
                                                            T* __restrict__ y, T* __restrict__ r, int64_t n,
                                                            double* __restrict__ partials) {
  __shared__ double red[16];
  double v[1] = {0.0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const T bi = b[i * ldb];
    y[i] = (T)0;
    r[i] = bi;
    v[0] += (double)bi * (double)bi;
  }
  block_sum<1>(v, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

__global__ void __launch_bounds__(kThreads) scg_init_final_kernel(const double* __restrict__ partials, int nparts,
                                                                  CgState* st) {
  __shared__ double red[16];
  double t[1];
  reduce_partials<1>(partials, nparts, 1, t, red);
  if (threadIdx.x == 0) {
    const double rho = t[0];
    st->rho = rho;
    st->rho0 = rho;
    st->res0 = sqrt(rho);
    st->floor = -1.0;  // no breakdown floor: the right-hand side is given
    st->tol2 = st->tol * st->tol * rho;
    st->iters = 0;
    st->k = 1;
    st->beta = 0.0;
    st->status = GSF_OK;
    st->active = (__builtin_isfinite(rho) && rho > st->tol2) ? 1 : 0;
    if (!__builtin_isfinite(rho)) st->status = GSF_EBREAKDOWN;
  }
}

// q += alpha_shift p; partials of p^T q
template <typename T>
__global__ void __launch_bounds__(kThreads) scg_shift_kernel(const T* __restrict__ p, T* __restrict__ q, int64_t n,
                                                             double shift, double* __restrict__ partials,
                                                             const CgState* st) {
  __shared__ double red[16];
  if (!st->active) return;
  double v[1] = {0.0};
  const T sh = (T)shift;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const T pi = p[i];
    const T qi = q[i] + sh * pi;
    q[i] = qi;
    v[0] += (double)pi * (double)qi;
  }
  block_sum<1>(v, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = v[0];
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int px_blocks(int64_t total) {
  int64_t b = (total + kThreads - 1) / kThreads;
  if (b > 4096) b = 4096;
  return (int)(b < 1 ? 1 : b);
}

gsf_status net_adam(int64_t count, int t, double lr, double b1, double b2, double eps, float* w, float* mom,
                    float* vel, const float* grad, uint16_t* wb, hipStream_t s) {
  const float bc1 = (float)(1.0 - std::pow(b1, t)), bc2 = (float)(1.0 - std::pow(b2, t));
  net_adam_kernel<<<px_blocks(count), kThreads, 0, s>>>(count, (float)b1, (float)b2, (float)eps, (float)lr, bc1, bc2,
                                                        w, mom, vel, grad, wb);
  return launch_status();
}

gsf_status net_to_bf16(int64_t count, const float* w, uint16_t* wb, hipStream_t s) {
  net_to_bf16_kernel<<<px_blocks(count), kThreads, 0, s>>>(count, w, wb);
  return launch_status();
}

int net_tiles(int64_t rows, int64_t cols) {
  return (int)(((rows + kOT - 1) / kOT) * ((cols + kOT - 1) / kOT));
}

// Partials that the workspaces hold room for: one per 28 x 28 tile, the sizes
// that callers have always been asked for; at least the tiles of a launch.
int net_partials(int64_t rows, int64_t cols) {
  static_assert(kOT >= 28, "no more tiles than partials");
  return (int)(((rows + 27) / 28) * ((cols + 27) / 28));
}

gsf_status net_infer(int prec, const uint16_t* w, int64_t rows, int64_t cols, int m, const void* R, void* Z,
                     const void* g, const void* sqd, const double* colnorm, const LobpcgState* st, double* partials,
                     hipStream_t s) {
  NetInferArgs a{};
  a.w = w;
  a.R = R;
  a.Z = Z;
  a.g = g;
  a.sqd = sqd;
  a.colnorm = colnorm;
  a.st = st;
  a.rows = rows;
  a.cols = cols;
  a.n = rows * cols;
  a.m = m;
  a.tiles_x = (int)((cols + kOT - 1) / kOT);
  a.ntiles = net_tiles(rows, cols);
  a.partials = partials;
  if (prec == GSF_F32)
    net_infer_kernel<float><<<a.ntiles, kNetThreads, 0, s>>>(a);
  else
    net_infer_kernel<double><<<a.ntiles, kNetThreads, 0, s>>>(a);
  return launch_status();
}

gsf_status net_lob_select(int prec, int64_t rows, int64_t cols, int m, int constraint, void* W, const void* Z,
                          const void* sqd, const double* partials, int nparts, LobpcgState* st, hipStream_t s) {
  const int64_t n = rows * cols;
  net_final_kernel<<<1, kThreads, 0, s>>>(partials, nparts, m, st);
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    net_select_kernel<float><<<nb, kThreads, 0, s>>>((float*)W, (const float*)Z, (const float*)sqd, n, m, constraint,
                                                     st);
  else
    net_select_kernel<double><<<nb, kThreads, 0, s>>>((double*)W, (const double*)Z, (const double*)sqd, n, m,
                                                      constraint, st);
  return launch_status();
}

int tz_blocks(int64_t rows, int64_t cols) {
  const int a = vec_blocks(rows * cols), b = net_partials(rows, cols);
  return a < b ? a : b;
}

gsf_status launch_tz_partials(int prec, const void* R, const void* Z, const void* sqd, int64_t rows, int64_t cols,
                              int m, const LobpcgState* st, double* partials, hipStream_t s) {
  const int nb = tz_blocks(rows, cols);
  const int64_t n = rows * cols;
  if (prec == GSF_F32)
    tz_partials_kernel<float><<<nb, kThreads, 0, s>>>((const float*)R, (const float*)Z, (const float*)sqd, n, m, st,
                                                      partials);
  else
    tz_partials_kernel<double><<<nb, kThreads, 0, s>>>((const double*)R, (const double*)Z, (const double*)sqd, n, m,
                                                       st, partials);
  return launch_status();
}

gsf_status launch_col_copy(int prec, const void* src, int64_t lds, void* dst, int64_t ldd, int64_t n, hipStream_t s) {
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    col_copy_kernel<float><<<nb, kThreads, 0, s>>>((const float*)src, lds, (float*)dst, ldd, n);
  else
    col_copy_kernel<double><<<nb, kThreads, 0, s>>>((const double*)src, lds, (double*)dst, ldd, n);
  return launch_status();
}

gsf_status launch_colnorm(int prec, const void* R, int64_t n, int m, int64_t ld, double* partials, double* out,
                          hipStream_t s) {
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    colnorm_kernel<float><<<nb, kThreads, 0, s>>>((const float*)R, n, m, ld, partials);
  else
    colnorm_kernel<double><<<nb, kThreads, 0, s>>>((const double*)R, n, m, ld, partials);
  colnorm_final_kernel<<<1, kThreads, 0, s>>>(partials, nb, out);
  return launch_status();
}

gsf_status launch_net_pair(int prec, const void* r, int64_t ldr, const void* y, int64_t ldy, const void* g,
                           int64_t n, const double* norm, float* in, float* tg, hipStream_t s) {
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    net_pair_kernel<float><<<nb, kThreads, 0, s>>>((const float*)r, ldr, (const float*)y, ldy, (const float*)g, n,
                                                   norm, in, tg);
  else
    net_pair_kernel<double><<<nb, kThreads, 0, s>>>((const double*)r, ldr, (const double*)y, ldy, (const double*)g,
                                                    n, norm, in, tg);
  return launch_status();
}

gsf_status launch_residual(int prec, const void* X, void* R, int64_t n, int m, const double* theta, hipStream_t s) {
  Theta8 th{};
  for (int j = 0; j < m; ++j) th.v[j] = theta[j];
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    residual_kernel<float><<<nb, kThreads, 0, s>>>((const float*)X, (float*)R, n, m, th);
  else
    residual_kernel<double><<<nb, kThreads, 0, s>>>((const double*)X, (double*)R, n, m, th);
  return launch_status();
}

gsf_status launch_scg_init(int prec, const void* b, int64_t ldb, void* y, void* r, int64_t n, double* partials,
                           CgState* st, hipStream_t s) {
  const int nb = vec_blocks(n);
  if (prec == GSF_F32)
    scg_init_kernel<float><<<nb, kThreads, 0, s>>>((const float*)b, ldb, (float*)y, (float*)r, n, partials);
  else
    scg_init_kernel<double><<<nb, kThreads, 0, s>>>((const double*)b, ldb, (double*)y, (double*)r, n, partials);
  scg_init_final_kernel<<<1, kThreads, 0, s>>>(partials, nb, st);
  return launch_status();
}

gsf_status launch_scg_shift(int prec, const void* p, void* q, int64_t n, double shift, double* partials, int* nparts,
                            const CgState* st, hipStream_t s) {
  const int nb = vec_blocks(n);
  *nparts = nb;
  if (prec == GSF_F32)
    scg_shift_kernel<float><<<nb, kThreads, 0, s>>>((const float*)p, (float*)q, n, shift, partials, st);
  else
    scg_shift_kernel<double><<<nb, kThreads, 0, s>>>((const double*)p, (double*)q, n, shift, partials, st);
  return launch_status();
}

}  // namespace gsf

// Training pass of the learned preconditioner's network (net.hip describes
// the network and its weight layout): loss and weight gradient of a
// mini-batch, or the forward pass alone, in one kernel over 32 x 16 pixel
// tiles, plus a fixed-order reduction of the workgroups' gradients.
//
// One workgroup walks tiles and keeps a tile's whole dependence cone in LDS:
// the input with a 5-pixel halo, a1 with 4, a2 with 3, y and dy with 2,
// dz2 with 1 (131 KB), so that no activation or gradient plane goes to HBM.
//   forward   layers 1 and 2 on v_mfma_f32_16x16x4_f32, which adds its four
//             products to the accumulator one after the other, each rounded as
//             a fused multiply-add (bitwise equal to the chain, checked on the
//             GPU): an activation that lies next to a BF16 rounding boundary
//             then rounds as in a plain FP32 chain over taps and channels.
//             (v_mfma_f32_16x16x32_bf16 would take a fourteenth of the matrix
//             cycles, 512 us in all, but its sums round otherwise: the loss
//             moved by 1.1e-7.)  Layer 3 as FP32 multiply-adds, its weights scalar.
//   dz2, dz1  the FP32 gradients, and
//   dW        K = the 32 pixels of a tile row, one product per tap: on
//             v_mfma_f32_16x16x32_bf16.  An FP32 gradient operand is split
//             exactly into three BF16 parts (8 + 8 + 8 significant bits); a
//             weight or an activation is BF16 already, so the products are
//             exact and the sums FP32.
// Pixel-major operands of the weight gradients come from LDS by transposing
// reads (ds_read_b64_tr_b16: four pixels of one channel per lane).  The
// gradients are summed in FP32 over the two rows a wave takes of a tile and in
// FP64 from there (across tiles, waves and workgroups, in fixed order).
//
// Channel blocks are stored as two planes of 8 channels (16 bytes per pixel),
// so that a wave's 16-byte operand reads are contiguous.  The channels of a1
// are stored in the order of the layer-2 operand (position 4q + i holds
// channel 4i + q: the four values lane group q feeds to one tap's products).
#include <cmath>

#include "net_common.h"

namespace gsf {
namespace {

constexpr int kT = 512;               // threads: 8 waves
constexpr int kWaves = kT / 64;
constexpr int TH = 16, TW = 32;       // own pixels of a tile: two rows per wave
constexpr int XH = TH + 10, XW = TW + 10, XN = XH * XW;
constexpr int A1H = TH + 8, A1W = TW + 8, A1N = A1H * A1W;
constexpr int A2H = TH + 6, A2W = TW + 6, A2N = A2H * A2W;
constexpr int YH = TH + 4, YW = TW + 4, YN = YH * YW;
constexpr int DH = TH + 2, DW = TW + 2, DN = DH * DW;
constexpr int A1G = (A1N + 15) / 16, A2G = (A2N + 15) / 16, DG = (DN + 15) / 16;  // groups of 16 pixels
constexpr int A1P = A1G * 16, A2P = A2G * 16, DP = DG * 16;                        // pixels of a plane
constexpr int kA1Bytes = 2 * A1P * 16, kA2Bytes = 2 * A2P * 16, kDzBytes = 6 * DP * 16;
static_assert(TW == 32 && TH == 2 * kWaves, "a wave owns two rows of 32 pixels");
constexpr int kXIter = (XN + kT - 1) / kT;
static_assert(YH % 2 == 0 && YN / 2 <= kT, "two pixels of y per thread");

// Operand packs: one 16-byte word per lane, four FP32 or eight BF16 weights
enum {
  OP_L1 = 0,       // layer 1, A: 16 channels x (9 taps x 2 inputs), FP32 (two packs, K = 20 padded)
  OP_F2 = 2,       // layer 2, A: 16 channels x 16 channels of tap t, FP32
  OP_B3 = 11,      // dz2, A: 16 channels x (9 taps x 3 parts)
  OP_B2 = 12,      // dz1, B: tap t for the parts 0 and 1
  OP_B2L = 21,     // dz1, B: tap pairs (0,1) (3,4) (6,7) (2,5) (8,-) for part 2
  kOps = 26
};
constexpr int kPackWords = kOps * 64 + 36;  // then the 144 weights of layer 3, FP32, tap by tap

// channel at position m of a1's storage order (its own inverse)
__device__ __forceinline__ int a1_channel(int m) { return 4 * (m & 3) + (m >> 2); }

struct NetTrainArgs {
  const uint4_t* ops;     // [kPackWords]
  const int32_t* idx;     // sample of each batch position
  int rows, cols;
  int64_t hw;
  const float* inputs;    // [sample][hw][2]
  const float* targets;   // [sample][hw]
  float* y;               // [batch position][hw] (forward only)
  double* partials;       // [workgroup][kNetWeights]
  double* loss_part;      // [workgroup]
  float dscale;           // 2 / (batch * hw)
  int tiles_x, tiles_per_sample;
  int64_t ntiles;
};

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// f = h + m + l exactly, each part's bits the upper half of a word: the two
// remainders of a truncation to 8 significant bits are exact (16, then 8 bits)
struct Split {
  uint32_t h, m, l;
};
__device__ __forceinline__ Split split3(float f) {
  Split s;
  s.h = __float_as_uint(f) & 0xffff0000u;
  const float hf = __uint_as_float(s.h);
  const float r = hf == f ? 0.0f : f - hf;  // an infinity stays in h
  s.m = __float_as_uint(r) & 0xffff0000u;
  s.l = __float_as_uint(r - __uint_as_float(s.m));
  return s;
}
// two BF16 values (upper halves of a and b) as one word, a first
__device__ __forceinline__ uint32_t join(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Transposing LDS read: lane i of a group of 16 gets channel i of four
// consecutive pixels (lane i's address: pixel i / 4, channels 4 (i % 4)..).
__device__ __forceinline__ uint2 read_tr(const char* p) {
  return __builtin_bit_cast(
      uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)p));
}
__device__ __forceinline__ uint4_t read_tr8(const char* p) {  // pixels p..p+3 and p+4..p+7
  const uint2 a = read_tr(p), b = read_tr(p + 4 * 16);
  return uint4_t{a.x, a.y, b.x, b.y};
}

// MFMA operand packs of the BF16 weights (one thread per lane and pack)
__global__ void __launch_bounds__(kThreads) net_pack_kernel(const uint16_t* __restrict__ w,
                                                            uint4_t* __restrict__ ops) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= kPackWords) return;
  const int op = t >> 6, lane = t & 63, q = lane >> 4, l16 = lane & 15;
  const int ch = 8 * (q & 1), sel = q >> 1;
  if (op < OP_B3 || op == kOps) {
    uint4_t v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int at;
      if (op == kOps) {
        const int e = 4 * lane + i;  // 16 tap + channel
        at = kOffW3 + (e & 15) * 9 + (e >> 4);
      } else if (op < OP_F2) {
        const int k = 16 * op + 4 * i + q;  // 2 tap + input
        at = k < 18 ? a1_channel(l16) * 18 + (k & 1) * 9 + (k >> 1) : -1;
      } else {
        at = kOffW2 + l16 * 144 + (4 * i + q) * 9 + op - OP_F2;
      }
      v[i] = at >= 0 ? (uint32_t)w[at] << 16 : 0u;
    }
    ops[t] = v;
    return;
  }
  auto pair_tap = [&](int j) { return j < 3 ? 3 * j + sel : (j == 3 ? 2 + 3 * sel : (sel ? -1 : 8)); };
  uint32_t v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int at = -1;
    if (op == OP_B3) {
      const int tap = i < 3 ? 2 * q : (i < 6 ? 2 * q + 1 : 8);
      at = i < 6 || q == 0 || (q == 1 && i == 6) ? kOffW3 + l16 * 9 + tap : -1;
    } else {
      const int tap = op < OP_B2L ? op - OP_B2 : pair_tap(op - OP_B2L);
      at = tap >= 0 ? kOffW2 + (ch + i) * 144 + a1_channel(l16) * 9 + tap : -1;
    }
    v[i] = at >= 0 ? w[at] : 0u;
  }
  ops[t] = uint4_t{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
}

// The training pass (GRAD) or the forward pass (y of every pixel).
template <bool GRAD>
__global__ void __launch_bounds__(kT) net_train_kernel(NetTrainArgs a) {
  __shared__ float2 xs[XN + 1];                         // (r/s, g) rounded to BF16, per pixel (one pad)
  __shared__ __align__(16) char a1s[kA1Bytes];          // [channel half][pixel][8]
  __shared__ __align__(16) char a2s[kA2Bytes];          // [channel half][pixel][8]
  __shared__ __align__(16) char dzs[kDzBytes];          // dz2 [part][channel half][pixel][8]
  __shared__ float dys[YN];                             // dy, 0 off the image
  __shared__ __align__(16) float dyo[TH * TW];          // dy of the own pixels
  __shared__ double red[16];

  // The thread index is made opaque at the top of every stage: what follows
  // from it (pixel coordinates, LDS addresses) is then recomputed there
  // instead of being kept in registers over all tiles.
  auto opaque = [](int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
  };
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

  double dw2[9][4], dw1[2][4], dw3[3][4];
  double loss = 0.0;
  if (GRAD) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int t = 0; t < 9; ++t) dw2[t][i] = 0.0;
      dw1[0][i] = dw1[1][i] = 0.0;
      dw3[0][i] = dw3[1][i] = dw3[2][i] = 0.0;
    }
  }

  struct Tile {
    int b, y0, x0;
  };
  auto tile_at = [&](int64_t t) {
    Tile r;
    r.b = (int)(t / a.tiles_per_sample);
    const int l = (int)(t - (int64_t)r.b * a.tiles_per_sample);
    const int ty = l / a.tiles_x;
    r.y0 = ty * TH;
    r.x0 = (l - ty * a.tiles_x) * TW;
    return r;
  };
  // `inner`: the tile and its whole halo lie on the image
  auto on_image = [&](int gy, int gx) { return (unsigned)gy < (unsigned)a.rows && (unsigned)gx < (unsigned)a.cols; };
  auto load_x = [&](const Tile& t, float2 (&v)[kXIter]) {
    const int tid = opaque(threadIdx.x);
    const float* in = a.inputs + (size_t)a.idx[t.b] * a.hw * 2;
#pragma unroll
    for (int k = 0; k < kXIter; ++k) {
      const int e = tid + k * kT;
      const int ey = div_px<XW, kXIter * kT>(e), gy = t.y0 - 5 + ey, gx = t.x0 - 5 + e - __mul24(ey, XW);
      v[k] = make_float2(0.0f, 0.0f);
      if (e < XN && on_image(gy, gx)) v[k] = *(const float2*)(in + ((size_t)gy * a.cols + gx) * 2);
    }
  };

  float2 xv[kXIter];
  int64_t tt = blockIdx.x;
  if (tt < a.ntiles) load_x(tile_at(tt), xv);
  for (; tt < a.ntiles; tt += gridDim.x) {
    const Tile t = tile_at(tt);
    const int y0 = t.y0, x0 = t.x0;
    // opaque per tile, so that the operand packs are loaded where they are
    // used (L1 hits) instead of being kept in registers over the tiles, which
    // spilled 238 of them
    const uint4_t* ops = a.ops;
    const bool inner = y0 >= 5 && x0 >= 5 && y0 + TH + 5 <= a.rows && x0 + TW + 5 <= a.cols;
    __asm__ volatile("" : "+s"(ops));
    lds_barrier();  // the previous tile's reads of LDS are done
    const int tid = opaque(threadIdx.x);
    // forward only: a tile with less than half of its rows of a1 on the image
    // works on the groups of 16 pixels that hold them; the others' activations are
    // zeros (a signal of 100000 samples: 73 us, 189 without; in the training pass
    // the runtime bounds cost 0.4% of a mini-batch of images)
    const int top = y0 < 4 ? 4 - y0 : 0, bottom = a.rows - y0 + 4 < A1H ? a.rows - y0 + 4 : A1H;
    const bool thin = !GRAD && 2 * (bottom - top) < A1H;
    const int ga1 = thin ? top * A1W / 16 : 0, gb1 = thin ? (bottom * A1W + 15) / 16 : A1G;
    const int ga2 = thin && top > 1 ? (top - 1) * A2W / 16 : 0;
    const int gb2 = thin && bottom - 1 < A2H ? ((bottom - 1) * A2W + 15) / 16 : A2G;
    if (thin) {
      const uint4_t none = {0u, 0u, 0u, 0u};
      for (int e = tid; e < 2 * A1P; e += kT) *(uint4_t*)(a1s + 16 * e) = none;
      for (int e = tid; e < 2 * A2P; e += kT) *(uint4_t*)(a2s + 16 * e) = none;
    }
#pragma unroll
    for (int k = 0; k < kXIter; ++k) {
      const int e = tid + k * kT;
      const uint32_t u = pack2(xv[k].x, xv[k].y);
      if (e < XN) xs[e] = make_float2(bf_lo(u), bf_hi(u));
    }
    float tv[2] = {0.0f, 0.0f};  // targets of this thread's two pixels
    if (GRAD && tid < YN / 2) {
      const float* tg = a.targets + (size_t)a.idx[t.b] * a.hw;
      const int gy = y0 - 2 + 2 * (tid / YW), gx = x0 - 2 + tid % YW;
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (on_image(gy + u, gx)) tv[u] = tg[(size_t)(gy + u) * a.cols + gx];
    }
    const int ln = opaque(threadIdx.x & 63);

    // layer 1
    {
      const int lane = ln, q = lane >> 4, l16 = lane & 15, half = q & 1, sel = q >> 1;
      const floatx4_t w0 = __builtin_bit_cast(floatx4_t, ops[OP_L1 * 64 + lane]);
      const float w4 = __builtin_bit_cast(floatx4_t, ops[(OP_L1 + 1) * 64 + lane])[0];
      lds_barrier();
#pragma unroll 1
      for (int g0 = ga1 + wave; g0 < gb1; g0 += 4 * kWaves) {  // four groups at a time (four accumulator chains)
        float v[4][5];
        floatx4_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = g0 + u * kWaves < gb1 ? g0 + u * kWaves : g0;
          const int p = g * 16 + l16, py = div_px<A1W, A1P>(p), px = p - __mul24(py, A1W);
          // product 4j + q: tap 2j + q / 2, input q % 2
          const float* xp = (const float*)(xs + __mul24(py, XW) + px + sel) + half;
          const float* xw = (const float*)(xs + __mul24(py, XW) + px + sel * (XW - 2)) + half;
          v[u][0] = xp[0];                               // taps 0, 1
          v[u][1] = xw[4];                               // taps 2, 3
          v[u][2] = xp[2 * (XW + 1)];                    // taps 4, 5
          v[u][3] = xp[4 * XW];                          // taps 6, 7
          v[u][4] = sel ? 0.0f : xp[2 * (2 * XW + 2)];   // tap 8
          c[u] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 5; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            c[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(j < 4 ? w0[j] : w4, v[u][j], c[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = g0 + u * kWaves;
          if (g >= gb1) break;
          const int p = g * 16 + l16, py = div_px<A1W, A1P>(p), px = p - __mul24(py, A1W);
          const bool in = inner || on_image(y0 - 4 + py, x0 - 4 + px);
          uint2 w;
          w.x = in ? pack2(relu(c[u][0]), relu(c[u][1])) : 0u;
          w.y = in ? pack2(relu(c[u][2]), relu(c[u][3])) : 0u;
          *(uint2*)(a1s + (sel * A1P + p) * 16 + half * 8) = w;
        }
      }
    }

    // layer 2: two groups of 16 pixels at a time (two accumulator chains)
    {
      const int lane = opaque(threadIdx.x & 63), q = lane >> 4, l16 = lane & 15, half = q & 1, sel = q >> 1;
      floatx4_t w[9];
#pragma unroll
      for (int t = 0; t < 9; ++t) w[t] = __builtin_bit_cast(floatx4_t, ops[(OP_F2 + t) * 64 + lane]);
      lds_barrier();
#pragma unroll 1
      for (int g0 = ga2 + 2 * wave; g0 < gb2; g0 += 2 * kWaves) {
        const char* b[2];
        int pv[2];
        bool in[2];
        floatx4_t c[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          pv[u] = (g0 + u) * 16 + l16;
          const int p = pv[u] < A2N ? pv[u] : A2N - 1;
          const int py = div_px<A2W, A2P>(p), px = p - __mul24(py, A2W);
          b[u] = a1s + (sel * A1P + __mul24(py, A1W) + px) * 16 + half * 8;
          in[u] = inner || on_image(y0 - 3 + py, x0 - 3 + px);
          c[u] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
        // per tap: the next tap's reads, this tap's eight operands, then the
        // products of the two chains in turn (left to itself the compiler put
        // each operand's conversion between two dependent products, with waits)
        uint2 nv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) nv[u] = *(const uint2*)b[u];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          float f[4][2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const uint2 v = nv[u];
            if (t < 8) nv[u] = *(const uint2*)(b[u] + (((t + 1) / 3) * A1W + (t + 1) % 3) * 16);
            f[0][u] = bf_lo(v.x);
            f[1][u] = bf_hi(v.x);
            f[2][u] = bf_lo(v.y);
            f[3][u] = bf_hi(v.y);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) c[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[t][j], f[j][u], c[u], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          uint2 v;
          v.x = in[u] ? pack2(relu(c[u][0]), relu(c[u][1])) : 0u;
          v.y = in[u] ? pack2(relu(c[u][2]), relu(c[u][3])) : 0u;
          if (pv[u] < A2P) *(uint2*)(a2s + (sel * A2P + pv[u]) * 16 + half * 8) = v;
        }
      }
    }
    lds_barrier();

    // y (layer 3, one FP32 chain over taps and channels), the loss and dy:
    // two rows of pixels per thread share the rows of a2 between them.  The
    // weights are scalar loads, one tap column at a time (unrolled over the
    // columns the compiler kept them all and spilled).
    if (tid < YN / 2) {
      typedef const __attribute__((address_space(4))) float* cptr;
      const cptr w3 = (cptr)(uintptr_t)(ops + kOps * 64);
      const int ty = div_px<YW, kT>(tid), py = 2 * ty, px = tid - __mul24(ty, YW);
      const char* ap = a2s + (__mul24(py, A2W) + px) * 16;
      float yv[2] = {0.0f, 0.0f};
      const int gy0 = y0 - 2 + py;
      const bool rows_off = !GRAD && (gy0 + 1 < 0 || gy0 >= a.rows);  // (both; y is not used there)
      if (!rows_off) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll 1
          for (int kx = 0; kx < 3; ++kx) {
            const uint4_t v0 = *(const uint4_t*)(ap + (r * A2W + kx) * 16);
            const uint4_t v1 = *(const uint4_t*)(ap + (A2P + r * A2W + kx) * 16);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const uint32_t v = i < 8 ? v0[i >> 1] : v1[(i >> 1) - 4];
              const float x = (i & 1) ? bf_hi(v) : bf_lo(v);
              if (r < 3) yv[0] = fmaf(w3[(3 * r + kx) * 16 + i], x, yv[0]);
              if (r > 0) yv[1] = fmaf(w3[(3 * (r - 1) + kx) * 16 + i], x, yv[1]);
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int gy = y0 - 2 + py + u, gx = x0 - 2 + px;
        const bool in = inner || on_image(gy, gx);
        const bool own = (unsigned)(py + u - 2) < (unsigned)TH && (unsigned)(px - 2) < (unsigned)TW;
        if (GRAD) {
          const float er = yv[u] - tv[u], d = in ? a.dscale * er : 0.0f;
          dys[(py + u) * YW + px] = d;
          if (own) {
            dyo[(py + u - 2) * TW + px - 2] = d;
            if (in) loss += (double)er * (double)er;
          }
        } else if (own && in) {
          a.y[(size_t)t.b * a.hw + (size_t)gy * a.cols + gx] = yv[u];
        }
      }
    }
    if (!GRAD) {
      if (tt + gridDim.x < a.ntiles) load_x(tile_at(tt + gridDim.x), xv);
      continue;
    }

    // dz2[p][c] = [a2[p][c] > 0] sum_tap W3[c][tap] dy[p - off(tap)]
    {
      const int lane = opaque(threadIdx.x & 63), q = lane >> 4, l16 = lane & 15, half = q & 1, sel = q >> 1;
      const uint4_t w = ops[OP_B3 * 64 + lane];
      lds_barrier();
      const int t0 = 2 * q, t1 = 2 * q + 1;
      const int o0 = (2 - t0 / 3) * YW + 2 - t0 % 3, o1 = (2 - t1 / 3) * YW + 2 - t1 % 3;
#pragma unroll
      for (int k = 0; k < (DG + kWaves - 1) / kWaves; ++k) {
        const int g = wave + kWaves * k;
        if (g >= DG) break;
        const int pv = g * 16 + l16, p = pv < DN ? pv : DN - 1;
        const int py = div_px<DW, DP>(p), px = p - __mul24(py, DW);
        const float* d = dys + __mul24(py, YW) + px;
        const Split s0 = split3(d[o0]), s1 = split3(d[o1]), s8 = split3(d[0]);
        const floatx4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
        const floatx4_t c = mfma_bf16_k32(w, uint4_t{join(s0.h, s0.m), join(s0.l, s1.h), join(s1.m, s1.l),
                                              join(q == 1 ? s8.l : s8.h, s8.m)}, zero);
        const uint2 act = *(const uint2*)(a2s + (sel * A2P + __mul24(py + 2, A2W) + px + 2) * 16 + half * 8);
        const Split d0 = split3(bf_lo(act.x) > 0.0f ? c[0] : 0.0f), d1 = split3(bf_hi(act.x) > 0.0f ? c[1] : 0.0f);
        const Split d2 = split3(bf_lo(act.y) > 0.0f ? c[2] : 0.0f), d3 = split3(bf_hi(act.y) > 0.0f ? c[3] : 0.0f);
        char* o = dzs + (sel * DP + pv) * 16 + half * 8;
        *(uint2*)o = make_uint2(join(d0.h, d1.h), join(d2.h, d3.h));
        *(uint2*)(o + 2 * DP * 16) = make_uint2(join(d0.m, d1.m), join(d2.m, d3.m));
        *(uint2*)(o + 4 * DP * 16) = make_uint2(join(d0.l, d1.l), join(d2.l, d3.l));
      }
    }
    lds_barrier();
    if (tt + gridDim.x < a.ntiles) load_x(tile_at(tt + gridDim.x), xv);

    // weight gradients of layers 2 and 3 over this wave's two rows
    {
      const int lane = opaque(threadIdx.x & 63), q = lane >> 4, l16 = lane & 15;
      // this lane's pixel and channel quarter of a transposing read
      const int trp = l16 >> 2, trc = (l16 >> 1) & 1, trb = (l16 & 1) * 8;
      floatx4_t g2[9], g3[3];
#pragma unroll
      for (int k = 0; k < 9; ++k) g2[k] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 3; ++k) g3[k] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
      for (int rr = 0; rr < 2; ++rr) {
        const int y = 2 * wave + rr;
        const char* dp = dzs + (trc * DP + (y + 1) * DW + 1 + 8 * q + trp) * 16 + trb;
        const uint4_t z0 = read_tr8(dp), z1 = read_tr8(dp + 2 * DP * 16), z2 = read_tr8(dp + 4 * DP * 16);
        const char* ap = a1s + (trc * A1P + (y + 3) * A1W + 3 + 8 * q + trp) * 16 + trb;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const uint4_t b = read_tr8(ap + ((tap / 3) * A1W + tap % 3) * 16);
          g2[tap] = mfma_bf16_k32(z0, b, g2[tap]);
          g2[tap] = mfma_bf16_k32(z1, b, g2[tap]);
          g2[tap] = mfma_bf16_k32(z2, b, g2[tap]);
        }
        // dW3[c][tap] = sum_p dy[p] a2[p + off(tap)][c]: rows 3 kx + part of
        // the tile hold the three parts' sums for tap column kx
        const float* dq = dyo + y * TW + 8 * q;
        uint32_t pt[8];
        const int part = l16 % 3;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const Split s = split3(dq[i]);
          pt[i] = part == 0 ? s.h : (part == 1 ? s.m : s.l);
        }
        const uint4_t pa = {join(pt[0], pt[1]), join(pt[2], pt[3]), join(pt[4], pt[5]), join(pt[6], pt[7])};
        const uint4_t none = {0u, 0u, 0u, 0u};
        const char* bp = a2s + (trc * A2P + (y + 2) * A2W + 2 + 8 * q + trp) * 16 + trb;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
          const uint4_t b = read_tr8(bp + ((tap / 3) * A2W + tap % 3) * 16);
          g3[tap / 3] = mfma_bf16_k32(l16 / 3 == tap % 3 ? pa : none, b, g3[tap / 3]);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int k = 0; k < 9; ++k) dw2[k][i] += (double)g2[k][i];
#pragma unroll
        for (int k = 0; k < 3; ++k) dw3[k][i] += (double)g3[k][i];
      }
    }

    // dz1[p][c] = [a1[p][c] > 0] sum_tap sum_o W2[o][c][tap] dz2[p - off(tap)][o]
    // as D[pixel][channel]: its lane layout is the A operand (channel x
    // pixels) of the weight gradient of layer 1
    {
      const int lane = opaque(threadIdx.x & 63), q = lane >> 4, l16 = lane & 15, half = q & 1, sel = q >> 1;
      // this lane's pixel and channel quarter of a transposing read
      const int trp = l16 >> 2, trc = (l16 >> 1) & 1, trb = (l16 & 1) * 8;
      // the wave's four groups of 16 pixels (two rows) side by side
      floatx4_t c[4], e[4];
      const char* pb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        c[u] = e[u] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
        pb[u] = dzs + ((2 * wave + (u >> 1) + 2) * DW + 16 * (u & 1) + l16 + 2) * 16;
      }
      const int o01 = (sel * 2 + half) * DP * 16, o2 = (4 + half) * DP * 16;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const uint4_t w = ops[(OP_B2 + tap) * 64 + lane];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          c[u] = mfma_bf16_k32(*(const uint4_t*)(pb[u] + o01 - ((tap / 3) * DW + tap % 3) * 16), w, c[u]);
      }
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const uint4_t w = ops[(OP_B2L + j) * 64 + lane];
        const int off = j < 3 ? j * DW + sel : (j == 3 ? 2 + sel * DW : 2 * DW + 2);
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = mfma_bf16_k32(*(const uint4_t*)(pb[u] + o2 - off * 16), w, e[u]);
      }
      floatx4_t g1[2];
      g1[0] = g1[1] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
      const int xtap = l16 < 9 ? l16 : 8;
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        const int y = 2 * wave + rr;
        uint2 zp[3][2];
        uint2 xc[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const floatx4_t d = c[2 * rr + h] + e[2 * rr + h];
          const uint2 act = read_tr(a1s + (trc * A1P + (y + 4) * A1W + 16 * h + 4 + 4 * q + trp) * 16 + trb);
          const Split s0 = split3(bf_lo(act.x) > 0.0f ? d[0] : 0.0f), s1 = split3(bf_hi(act.x) > 0.0f ? d[1] : 0.0f);
          const Split s2 = split3(bf_lo(act.y) > 0.0f ? d[2] : 0.0f), s3 = split3(bf_hi(act.y) > 0.0f ? d[3] : 0.0f);
          zp[0][h] = make_uint2(join(s0.h, s1.h), join(s2.h, s3.h));
          zp[1][h] = make_uint2(join(s0.m, s1.m), join(s2.m, s3.m));
          zp[2][h] = make_uint2(join(s0.l, s1.l), join(s2.l, s3.l));
          const float2* xp = xs + (y + 4 + div_px<3, 9>(xtap)) * XW + 16 * h + 4 * q + 4 + xtap % 3;
          const float2 v0 = xp[0], v1 = xp[1], v2 = xp[2], v3 = xp[3];
          auto bits = [](float f) { return __float_as_uint(f); };
          xc[0][h] = make_uint2(join(bits(v0.x), bits(v1.x)), join(bits(v2.x), bits(v3.x)));
          xc[1][h] = make_uint2(join(bits(v0.y), bits(v1.y)), join(bits(v2.y), bits(v3.y)));
        }
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
          const uint4_t b = {xc[ch][0].x, xc[ch][0].y, xc[ch][1].x, xc[ch][1].y};
#pragma unroll
          for (int k = 0; k < 3; ++k)
            g1[ch] = mfma_bf16_k32(uint4_t{zp[k][0].x, zp[k][0].y, zp[k][1].x, zp[k][1].y}, b, g1[ch]);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dw1[0][i] += (double)g1[0][i];
        dw1[1][i] += (double)g1[1][i];
      }
    }
  }
  if (!GRAD) return;

  // the eight waves' sums in wave order, in LDS (weights of layers 1 and 2 at
  // their place, layer 3 as [ky][3 kx + part][c]), then the workgroup's partial
  const int tid = threadIdx.x, q = (tid & 63) >> 4, l16 = tid & 15;
  constexpr int kDw3 = kOffW3;
  static_assert((kDw3 + 3 * 16 * 16) * 8 <= kA1Bytes, "the gradient sums take the space of a1");
  double* sum = (double*)a1s;
  for (int wv = 0; wv < kWaves; ++wv) {
    __syncthreads();
    if (wave != wv) continue;
    auto put = [&](int at, double v) { sum[at] = wv == 0 ? v : sum[at] + v; };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 4 * q + i;
#pragma unroll
      for (int k = 0; k < 9; ++k) put(kOffW2 + m * 144 + a1_channel(l16) * 9 + k, dw2[k][i]);
      if (l16 < 9) {
        put(a1_channel(m) * 18 + l16, dw1[0][i]);
        put(a1_channel(m) * 18 + 9 + l16, dw1[1][i]);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) put(kDw3 + (k * 16 + m) * 16 + l16, dw3[k][i]);
    }
  }
  double v[1] = {loss};
  block_sum<1>(v, red);  // (its barriers order the sums above as well)
  if (tid == 0) a.loss_part[blockIdx.x] = v[0];
  double* out = a.partials + (size_t)blockIdx.x * kNetWeights;
  for (int e = tid; e < kNetWeights; e += kT) {
    if (e < kOffW3) {
      out[e] = sum[e];
    } else {
      const int c = (e - kOffW3) / 9, tap = (e - kOffW3) - 9 * c;
      const double* s = sum + kDw3 + ((tap / 3) * 16 + 3 * (tap % 3)) * 16 + c;
      out[e] = s[0] + s[16] + s[32];
    }
  }
}

// grad[w] = sum of the workgroups' partials: 32 weights per workgroup, eight
// slices of the partials summed side by side, then in slice order; the first
// workgroup also closes the loss.
__global__ void __launch_bounds__(kThreads) net_grad_reduce_kernel(const double* __restrict__ partials,
                                                                   const double* __restrict__ loss_part, int nparts,
                                                                   double inv_count, float* __restrict__ grad,
                                                                   double* __restrict__ loss) {
  __shared__ double s[8][32];
  __shared__ double red[16];
  const int wl = threadIdx.x & 31, slice = threadIdx.x >> 5;
  const int w = blockIdx.x * 32 + wl;
  const int per = (nparts + 7) / 8, b1 = (slice + 1) * per < nparts ? (slice + 1) * per : nparts;
  double v = 0.0;
  if (w < kNetWeights)
#pragma unroll 8
    for (int b = slice * per; b < b1; ++b) v += partials[(size_t)b * kNetWeights + w];
  s[slice][wl] = v;
  __syncthreads();
  if (slice == 0 && w < kNetWeights) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) t += s[k][wl];
    grad[w] = (float)t;
  }
  if (blockIdx.x != 0) return;
  double t[1];
  reduce_partials<1>(loss_part, nparts, 1, t, red);
  if (threadIdx.x == 0) *loss = t[0] * inv_count;
}

// workgroups of the training pass: one per CU (its LDS), each walking tiles
constexpr int kNetGrid = 256;

int64_t train_tiles(int batch, int64_t rows, int64_t cols) {
  return (int64_t)batch * ((rows + TH - 1) / TH) * ((cols + TW - 1) / TW);
}

}  // namespace

// The pass needs the operand packs and the loss and gradient partials (the
// tiles' planes stay in LDS).  The entry points ask for what they always did,
// room for a whole batch's planes (the activations of both hidden layers in
// BF16, their gradients in FP32, y and dy) beside the partials of 1024
// workgroups, so that the sizes callers hold and the calls they see refused
// stay the same.
size_t net_train_bytes(int batch, int64_t hw) {
  constexpr size_t used = (size_t)kPackWords * 16 + (size_t)kNetGrid * (1 + kNetWeights) * 8 + 3 * 256;
  constexpr size_t partials = (size_t)1024 * kNetWeights * 8;
  static_assert(used <= partials, "the pass fits whatever the batch");
  const size_t px = (size_t)batch * (size_t)hw;
  return align_up(kNetWeights * 4, 256) + 2 * align_up(px * 32, 256) + 2 * align_up(px * 4, 256) +
         2 * align_up(px * 64, 256) + align_up(1024 * 8, 256) + align_up(partials, 256);
}

gsf_status net_forward_train(const uint16_t* w, int batch, const int32_t* idx, int64_t rows, int64_t cols,
                             const float* inputs, const float* targets, float* y_out, float* grad, double* loss,
                             void* ws, hipStream_t s) {
  char* p = (char*)ws;
  NetTrainArgs a{};
  a.ops = (const uint4_t*)p;
  p += align_up((size_t)kPackWords * 16, 256);
  a.loss_part = (double*)p;
  p += align_up((size_t)kNetGrid * 8, 256);
  a.partials = (double*)p;
  a.idx = idx;
  a.rows = (int)rows;
  a.cols = (int)cols;
  a.hw = rows * cols;
  a.inputs = inputs;
  a.targets = targets;
  a.y = y_out;
  const double count = (double)batch * (double)a.hw;
  a.dscale = (float)(2.0 / count);
  a.tiles_x = (int)((cols + TW - 1) / TW);
  a.ntiles = train_tiles(batch, rows, cols);
  a.tiles_per_sample = (int)(a.ntiles / batch);
  const int nb = a.ntiles < kNetGrid ? (int)a.ntiles : kNetGrid;
  net_pack_kernel<<<(kPackWords + kThreads - 1) / kThreads, kThreads, 0, s>>>(w, (uint4_t*)ws);
  if (targets == nullptr) {
    net_train_kernel<false><<<nb, kT, 0, s>>>(a);
    return launch_status();
  }
  net_train_kernel<true><<<nb, kT, 0, s>>>(a);
  net_grad_reduce_kernel<<<(kNetWeights + 31) / 32, kThreads, 0, s>>>(a.partials, a.loss_part, nb, 1.0 / count, grad,
                                                                     loss);
  return launch_status();
}

}  // namespace gsf

// mlp.hip -- the surrogate network of log L: 17 -> 256 -> 256 -> 256 -> 1, SiLU.
//
// Matrix products run on the matrix cores with bfloat16 operands and float32
// accumulation (v_mfma_f32_16x16x32_bf16). Operands are rounded to bfloat16
// (nearest even) at fixed points: normalised input, weights, activations H and
// back-propagated dZ; everything else is float32.
//
// The work is small (0.8 MFLOP a row and direction) and was bound by launches,
// by reads and writes of every layer's Z and H, and, in the weight gradients, by
// 16 blocks that each walked all rows with strided two-byte loads. So:
//   mlp_rows_kernel   a block takes 16, 32 or 64 rows through all layers, and in
//                     training back again. Activations and dZ pass between the
//                     layers in LDS, Z stays in registers, the weights come from
//                     L2 in the lanes' operand layout, one layer ahead. For the
//                     weight gradients it also writes H and dZ transposed (rows
//                     contiguous) and its own column sums (bias gradients, dW4).
//   mlp_dw_kernel     dW_l = dZ_l^T H_{l-1}: a wave takes a 64 x 64 (64 x 32 for
//                     W1) piece over a part of the rows, both operands straight
//                     from the transposed copies.
//   mlp_sum_kernel    adds the parts in a fixed order and writes the gradient, or
//                     applies Adam to it.
// One Adam step at 4096 rows: 1959 us with one kernel per layer and reduction, 49 us
// so (rows 27, weight gradients 13, sums 6, weight conversion 5 us, of which a
// launch is about 4 each); predictions for 16384 rows 154 -> 30 us. What is left
// is latency: 12.6 million SiLUs are 6 us of vector work, the products 4 us.
//
// Flat parameter layout (float32): W1 [256][17], b1 [256], W2 [256][256], b2,
// W3 [256][256], b3, W4 [1][256], b4 [1]. Normalisation block: x_shift [17],
// x_scale [17], y_shift, y_scale.
#include <stdint.h>

#include <cmath>
#include <type_traits>

#include "internal.h"
#include "kernels.h"
#include "mlp.h"

namespace lensed {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// n / d for d in [1, inf]: the steps of a correctly rounded division that need no
// scaling for d up to 8e37 (the compiler's general division takes half again as many
// instructions, and these divisions are most of the vector work here). Past that the
// quotient, below 1e-35 for every n that can come with it, is off by at most itself:
// the corrections take d as 8e37, which leaves a reciprocal of 0 at 0. d = inf gives
// n x 0, as the division does for finite n (0) and for n = -inf (NaN); n = +inf with
// d = 1 stands as the largest float32, which rounds to inf in bfloat16.
__device__ __forceinline__ float div_unscaled(float n, float d) {
  const float dc = fminf(d, 8e37f);
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-dc, r, 1.0f), r, r);
  float q = n * r;
  q = fmaf(fmaf(-dc, q, n), r, q);
  return fmaf(fmaf(-dc, q, n), r, q);
}
__device__ __forceinline__ float silu(float z) { return div_unscaled(fminf(z, 3.402823466e38f), 1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = div_unscaled(1.0f, 1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p) { return __builtin_bit_cast(bf16x8, *(const u16x8*)p); }
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// bfloat16 copies of the weights: W1 padded to [256][32], W2, W3 [256][256], W4
// [256], and, with `transposes`, W2 and W3 transposed. A block takes a 64 x 64
// piece of W2 or W3 (blocks 0..31) or a share of the rest.
constexpr int CONVERT_BLOCKS = 34;
__global__ __launch_bounds__(256) void convert_weights_kernel(const float* __restrict__ p, uint16_t* __restrict__ wb,
                                                              int transposes) {
  const int t = (int)threadIdx.x, b = (int)blockIdx.x;
  if (b >= 32) {
    for (int i = (b - 32) * 256 + t; i < MLP_H * MLP_KPAD; i += 512) {
      const int o = i / MLP_KPAD, k = i - o * MLP_KPAD;
      wb[i] = k < MLP_IN ? f2bf(p[MLP_OFF_W1 + o * MLP_IN + k]) : (uint16_t)0;
    }
    if (b == 32) wb[MLP_WB_W4 + t] = f2bf(p[MLP_OFF_W4 + t]);
    return;
  }
  __shared__ uint16_t tile[64][66];
  const int r0 = (b & 15) / 4 * 64, c0 = (b & 3) * 64;
  const float* __restrict__ W = p + (b < 16 ? MLP_OFF_W2 : MLP_OFF_W3);
  uint16_t* __restrict__ o = wb + (b < 16 ? MLP_WB_W2 : MLP_WB_W3);
  uint16_t* __restrict__ oT = wb + (b < 16 ? MLP_WB_W2T : MLP_WB_W3T);
  const int c = t & 63;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = (t >> 6) + 4 * k;
    const uint16_t h = f2bf(W[(r0 + r) * MLP_H + c0 + c]);
    o[(r0 + r) * MLP_H + c0 + c] = h;
    tile[r][c] = h;
  }
  if (!transposes) return;   // uniform
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = (t >> 6) + 4 * k;
    oT[(c0 + r) * MLP_H + r0 + c] = tile[c][r];
  }
}

struct RowArgs {
  const float* p;       // parameters
  const float* norm;
  const float* x;
  const float* yt;      // targets (training)
  const uint16_t* wb;
  float* y;             // predictions (forward)
  int B;
  long ld;              // distance of two rows of the transposed buffers
  uint16_t *X0T, *HT0, *HT1, *dZT0, *dZT1, *dZT2;
  float *d, *sq, *cols;
};

// MT x 16 rows per block, NW waves of 16 NT columns each. Lane l of a 16x16x32 MFMA
// holds A[m = l % 16][k = 8 (l / 16) + j] and B[k = 8 (l / 16) + j][n = l % 16],
// j = 0..7, and receives D[m = 4 (l / 16) + j][n = l % 16], j = 0..3. In training A is
// the activations (a lane receives four rows of a column, for the transposed
// copies and the column sums); otherwise A is the weights (four columns of a row,
// one 8-byte write to LDS). The sums over k are the same. Rows past B compute with
// x = 0; their H and dZ are written as zeros.
constexpr int LDH = MLP_H + 8;   // 16 rows fall into different banks
template <int MT, int NW, bool TRAIN>
__global__ __launch_bounds__(64 * NW, 1) void mlp_rows_kernel(RowArgs a) {
  constexpr int NT = 16 / NW;
  __shared__ __align__(16) uint16_t buf[2][16 * MT][LDH];
  __shared__ float dl[16 * MT];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int c = lane & 15, g = lane >> 4, wn = wave * 16 * NT;
  const int row0 = (int)blockIdx.x * 16 * MT;
  const float* __restrict__ p = a.p;

  bf16x8 wf[8][NT];   // the lane's pieces of one 256 x 256 layer
  auto load_w = [&](long off) {
    const uint16_t* __restrict__ w = a.wb + off + (long)(wn + c) * MLP_H + 8 * g;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int t = 0; t < NT; ++t) wf[ks][t] = frag(w + (long)16 * t * MLP_H + 32 * ks);
  };
  auto mul = [&](bf16x8 h, bf16x8 w, f32x4 acc) { return TRAIN ? mfma(h, w, acc) : mfma(w, h, acc); };
  auto gemm = [&](const uint16_t (*h)[LDH], f32x4 (&acc)[MT][NT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf16x8 hv = frag(&h[16 * mt + c][32 * ks + 8 * g]);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mt][t] = mul(hv, wf[ks][t], acc[mt][t]);
      }
  };
  // H = bf16(silu(z)) into LDS, and (training) transposed into HT, zero past B
  auto activate = [&](f32x4 (&z)[MT][NT], int off_b, uint16_t (*h)[LDH], uint16_t* HT) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = p[off_b + wn + 16 * t + (TRAIN ? c : 4 * g + j)];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        u16x4 hv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          z[mt][t][j] += b[j];
          hv[j] = f2bf(silu(z[mt][t][j]));
        }
        if (!TRAIN) {
          *(u16x4*)&h[16 * mt + c][wn + 16 * t + 4 * g] = hv;
          continue;
        }
        const int n = wn + 16 * t + c, r = 16 * mt + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) h[r + j][n] = hv[j];
        if (HT) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (row0 + r + j >= a.B) hv[j] = 0;
          *(u16x4*)(HT + n * a.ld + row0 + r) = hv;
        }
      }
    }
  };

  load_w(MLP_WB_W2);
  f32x4 z1[MT][NT], z2[MT][NT], z3[MT][NT];
  {   // layer 1: x normalised and rounded in the operand layout
    bf16x8 w1[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) w1[t] = frag(a.wb + (wn + 16 * t + c) * MLP_KPAD + 8 * g);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = row0 + 16 * mt + c;
      u16x8 xv;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = 8 * g + j;
        xv[j] = k < MLP_IN && row < a.B ? f2bf((a.x[(long)row * MLP_IN + k] - a.norm[k]) * a.norm[MLP_IN + k])
                                        : (uint16_t)0;
        if (TRAIN && wave == 0) a.X0T[k * a.ld + row] = xv[j];
      }
      const bf16x8 hv = __builtin_bit_cast(bf16x8, xv);
#pragma unroll
      for (int t = 0; t < NT; ++t) z1[mt][t] = mul(hv, w1[t], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
    }
  }
  activate(z1, MLP_OFF_B1, buf[0], a.HT0);
  __syncthreads();
  gemm(buf[0], z2);
  load_w(MLP_WB_W3);
  activate(z2, MLP_OFF_B2, buf[1], a.HT1);
  __syncthreads();
  gemm(buf[1], z3);
  if (TRAIN) load_w(MLP_WB_W3T);
  activate(z3, MLP_OFF_B3, buf[0], nullptr);
  __syncthreads();

  // head: out = H3 . W4 + b4, one row per wave at a time
  float w4[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) w4[j] = bf2f(a.wb[MLP_WB_W4 + lane + 64 * j]);
  for (int r = wave; r < 16 * MT; r += NW) {
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) s = fmaf(bf2f(buf[0][r][lane + 64 * j]), w4[j], s);
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    const int row = row0 + r;
    if (lane == 0) {
      const float out = s + p[MLP_OFF_B4];
      if (!TRAIN) {
        if (row < a.B) a.y[row] = a.norm[2 * MLP_IN] + a.norm[2 * MLP_IN + 1] * out;
      } else {
        float dv = 0.0f;
        if (row < a.B) {
          const float t = (a.yt[row] - a.norm[2 * MLP_IN]) / a.norm[2 * MLP_IN + 1];
          const float e = out - t;
          dv = 2.0f * e / (float)a.B;
          a.d[row] = dv;
          a.sq[row] = e * e;
        }
        dl[r] = dv;
      }
    }
  }
  if (!TRAIN) return;
  __syncthreads();

  float* __restrict__ cols = a.cols + (long)blockIdx.x * MLP_COLS;
  // the sum of v over the block's rows of column n, from the 16 lanes' four rows each
  auto column_sum = [&](float v, int slot) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (g == 0) cols[slot] = v;
  };
  // dZ in bfloat16 into LDS and transposed into dZT; its column sums in float32
  auto propagate = [&](const f32x4 (&dz)[MT][NT], uint16_t (*h)[LDH], uint16_t* dZT, int slot) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = wn + 16 * t + c;
      float s = 0.0f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        u16x4 hv;
        const int r = 16 * mt + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = row0 + r + j < a.B ? dz[mt][t][j] : 0.0f;
          s += v;
          hv[j] = f2bf(v);
          if (h) h[r + j][n] = hv[j];
        }
        *(u16x4*)(dZT + n * a.ld + row0 + r) = hv;
      }
      column_sum(s, slot + n);
    }
  };

  // layer 4: dW4[n] = sum_m d[m] H3[m][n]; dZ3 = d W4 silu'(Z3)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int n = wn + 16 * t + c;
    const float w = bf2f(a.wb[MLP_WB_W4 + n]);
    float s = 0.0f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 16 * mt + 4 * g + j;
        if (row0 + r < a.B) s += dl[r] * bf2f(buf[0][r][n]);
        z3[mt][t][j] = dl[r] * w * dsilu(z3[mt][t][j]);
      }
    column_sum(s, 3 * MLP_H + n);
  }
  propagate(z3, buf[1], a.dZT2, 2 * MLP_H);
  __syncthreads();
  gemm(buf[1], z3);   // dZ3 W3
  load_w(MLP_WB_W2T);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) z2[mt][t][j] = z3[mt][t][j] * dsilu(z2[mt][t][j]);
  propagate(z2, buf[0], a.dZT1, MLP_H);
  __syncthreads();
  gemm(buf[0], z2);   // dZ2 W2
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) z1[mt][t][j] = z2[mt][t][j] * dsilu(z1[mt][t][j]);
  propagate(z1, nullptr, a.dZT0, 0);
}

// dW_l[o][i] = sum_b dZ_l[b][o] H_{l-1}[b][i] over one part of the rows. Wave item
// (part, piece): pieces 0..15 of W3, 16..31 of W2 (64 x 64 each), 32..35 of W1
// (64 x 32, columns past 17 dropped). Both operands are rows of the transposed
// copies, 16 bytes per lane.
constexpr int DW_PIECES = 36;
template <int NT>
__device__ __forceinline__ void dw_piece(const uint16_t* __restrict__ A, const uint16_t* __restrict__ Bm, long ld,
                                         int k0, int k1, float* __restrict__ out, int ldo, int n_cols) {
  const int lane = (int)threadIdx.x & 63, c = lane & 15, g = lane >> 4;
  f32x4 acc[4][NT];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const uint16_t* __restrict__ pa = A + (long)c * ld + 8 * g;
  const uint16_t* __restrict__ pb = Bm + (long)c * ld + 8 * g;
  // U steps of 32 rows: all their loads first
  auto steps = [&](int k, auto uc) {
    constexpr int U = decltype(uc)::value;
    bf16x8 av[U][4], bv[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) av[u][i] = frag(pa + 16 * i * ld + k + 32 * u);
#pragma unroll
      for (int j = 0; j < NT; ++j) bv[u][j] = frag(pb + 16 * j * ld + k + 32 * u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = mfma(av[u][i], bv[u][j], acc[i][j]);
  };
  int k = k0;
  for (; k + 128 <= k1; k += 128) steps(k, std::integral_constant<int, 4>{});
  for (; k < k1; k += 32) steps(k, std::integral_constant<int, 1>{});
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (16 * j + c < n_cols) out[(long)(16 * i + 4 * g + r) * ldo + 16 * j + c] = acc[i][j][r];
}

__global__ __launch_bounds__(64) void mlp_dw_kernel(MlpScratch s, long ld, int Bp, int rows_per_part) {
  const int part = (int)blockIdx.x / DW_PIECES, piece = (int)blockIdx.x - part * DW_PIECES;
  const int k0 = part * rows_per_part, k1 = min(k0 + rows_per_part, Bp);
  float* __restrict__ out = s.dw + (long)part * MLP_NPARAM;
  if (piece < 32) {
    const int l = piece < 16 ? 2 : 1, o = (piece & 15) / 4 * 64, i = (piece & 3) * 64;
    dw_piece<4>(s.dZT[l] + o * ld, s.HT[l - 1] + i * ld, ld, k0, k1,
                out + (l == 2 ? MLP_OFF_W3 : MLP_OFF_W2) + (long)o * MLP_H + i, MLP_H, 64);
  } else {
    const int o = (piece - 32) * 64;
    dw_piece<2>(s.dZT[0] + o * ld, s.X0T, ld, k0, k1, out + MLP_OFF_W1 + (long)o * MLP_IN, MLP_IN, MLP_IN);
  }
}

// Adam (Kingma & Ba 2015): m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// p -= lr (m / bc1) / (sqrt(v / bc2) + eps), bc = 1 - b^t. The factors 1 - b
// and the bias corrections come from the host in float64 (1 - b2 rounded from a
// float b2 would carry a 1e-5 relative error).
__device__ __forceinline__ void adam_update(float* __restrict__ p, float gi, float* __restrict__ m,
                                            float* __restrict__ v, int i, const AdamStep& a) {
  const float mi = fmaf(a.beta1, m[i], a.omb1 * gi);
  const float vi = fmaf(a.beta2, v[i], a.omb2 * gi * gi);
  m[i] = mi;
  v[i] = vi;
  p[i] -= a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
}

__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int n, AdamStep a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) adam_update(p, g[i], m, v, i, a);
}

// The gradient from its parts, each sum in a fixed order, and (ADAM) the update.
// Blocks 0 .. SUM_COL_BLOCKS - 1: 64 column sums each (the biases and W4), four
// threads per column over the row blocks; the next: db4 and the loss; the rest:
// 256 weights each over the parts. The slow sums come first.
constexpr int SUM_COL_BLOCKS = MLP_COLS / 64;
constexpr int SUM_W = MLP_H * MLP_IN + 2 * MLP_H * MLP_H;
static_assert(SUM_W % 256 == 0, "whole blocks of weights");
constexpr int SUM_BLOCKS = SUM_COL_BLOCKS + 1 + SUM_W / 256;
template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_sum_kernel(MlpScratch s, int B, int row_blocks, int parts,
                                                      float* __restrict__ grad, float* __restrict__ loss,
                                                      float* __restrict__ p, float* __restrict__ m,
                                                      float* __restrict__ v, AdamStep a) {
  __shared__ float red[2][256];
  const int t = (int)threadIdx.x, b = (int)blockIdx.x;
  auto put = [&](int i, float gi) {
    if (ADAM)
      adam_update(p, gi, m, v, i, a);
    else
      grad[i] = gi;
  };
  if (b < SUM_COL_BLOCKS) {
    const int slot = b * 64 + (t & 63);
    float acc = 0.0f;
#pragma unroll 8
    for (int r = t >> 6; r < row_blocks; r += 4) acc += s.cols[(long)r * MLP_COLS + slot];
    red[0][t] = acc;
    __syncthreads();
    if (t < 64) {
      const float gi = (red[0][t] + red[0][t + 64]) + (red[0][t + 128] + red[0][t + 192]);
      const int l = slot / MLP_H, n = slot - l * MLP_H;
      put((l == 0 ? MLP_OFF_B1 : l == 1 ? MLP_OFF_B2 : l == 2 ? MLP_OFF_B3 : MLP_OFF_W4) + n, gi);
    }
    return;
  }
  if (b == SUM_COL_BLOCKS) {
    float sd = 0.0f, sl = 0.0f;
#pragma unroll 4
    for (int r = t; r < B; r += 256) {
      sd += s.d[r];
      sl += s.sq[r];
    }
    red[0][t] = sd;
    red[1][t] = sl;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
      if (t < k) {
        red[0][t] += red[0][t + k];
        red[1][t] += red[1][t + k];
      }
      __syncthreads();
    }
    if (t == 0) {
      put(MLP_OFF_B4, red[0][0]);
      loss[0] = red[1][0] / (float)B;
    }
    return;
  }
  const int e = (b - SUM_COL_BLOCKS - 1) * 256 + t;
  const int i = e < MLP_H * MLP_IN ? MLP_OFF_W1 + e
                : e < MLP_H * MLP_IN + MLP_H * MLP_H ? MLP_OFF_W2 + (e - MLP_H * MLP_IN)
                                                     : MLP_OFF_W3 + (e - MLP_H * MLP_IN - MLP_H * MLP_H);
  float gi = 0.0f;
#pragma unroll 8
  for (int k = 0; k < parts; ++k) gi += s.dw[(long)k * MLP_NPARAM + i];
  put(i, gi);
}

hipError_t convert_weights(const float* params, const MlpScratch& s, bool transposes, hipStream_t st) {
  hipLaunchKernelGGL(convert_weights_kernel, dim3(CONVERT_BLOCKS), dim3(256), 0, st, params, s.wb, transposes ? 1 : 0);
  return hipGetLastError();
}

// Rows per block: 16 while that leaves compute units idle otherwise, more for larger
// batches, so that a block's weights serve more rows (training keeps Z of three
// layers in registers: 32 at most). Eight waves hide the loads and the serial
// parts of 16 rows better than four.
template <int MT, bool TRAIN>
hipError_t launch_rows(const RowArgs& a, int Bp, hipStream_t st) {
  constexpr int NW = 8;
  hipLaunchKernelGGL((mlp_rows_kernel<MT, NW, TRAIN>), dim3((unsigned)(Bp / (16 * MT))), dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

// Everything but the last sums: the rows forward and back, and the parts of dW.
hipError_t grad_parts(const float* params, const float* norm, const float* x, const float* yt, int B,
                      const MlpScratch& s, int* row_blocks, int* parts, hipStream_t st) {
  hipError_t e = convert_weights(params, s, true, st);
  if (e != hipSuccess) return e;
  const int Bp = mlp_padded_rows(B);
  RowArgs a{};
  a.p = params, a.norm = norm, a.x = x, a.yt = yt, a.wb = s.wb;
  a.B = B, a.ld = mlp_transposed_stride(B);
  a.X0T = s.X0T, a.HT0 = s.HT[0], a.HT1 = s.HT[1];
  a.dZT0 = s.dZT[0], a.dZT1 = s.dZT[1], a.dZT2 = s.dZT[2];
  a.d = s.d, a.sq = s.sq, a.cols = s.cols;
  const bool two = Bp > 8192;
  *row_blocks = Bp / (two ? 32 : 16);
  if ((e = two ? launch_rows<2, true>(a, Bp, st) : launch_rows<1, true>(a, Bp, st)) != hipSuccess) return e;
  // parts of at least 128 rows (four matrix steps), whole 32-row steps
  int n = Bp / 128;
  n = n < 1 ? 1 : n > MLP_MAX_SPLITS ? MLP_MAX_SPLITS : n;
  const int rows = ((Bp + n - 1) / n + 31) / 32 * 32;
  *parts = (Bp + rows - 1) / rows;
  hipLaunchKernelGGL(mlp_dw_kernel, dim3((unsigned)(*parts * DW_PIECES)), dim3(64), 0, st, s, a.ld, Bp, rows);
  return hipGetLastError();
}

}  // namespace

hipError_t mlp_forward(const float* params, const float* norm, const float* x, float* y, int B, const MlpScratch& s,
                       hipStream_t st) {
  if (B <= 0) return hipSuccess;
  const hipError_t e = convert_weights(params, s, false, st);
  if (e != hipSuccess) return e;
  RowArgs a{};
  a.p = params, a.norm = norm, a.x = x, a.wb = s.wb, a.y = y;
  a.B = B;
  const int Bp = mlp_padded_rows(B);
  if (Bp <= 8192) return launch_rows<1, false>(a, Bp, st);
  return Bp <= 16384 ? launch_rows<2, false>(a, Bp, st) : launch_rows<4, false>(a, Bp, st);
}

hipError_t mlp_grad(const float* params, const float* norm, const float* x, const float* yt, int B, float* grad,
                    float* loss, const MlpScratch& s, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  int row_blocks = 0, parts = 0;
  const hipError_t e = grad_parts(params, norm, x, yt, B, s, &row_blocks, &parts, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((mlp_sum_kernel<false>), dim3(SUM_BLOCKS), dim3(256), 0, st, s, B, row_blocks, parts, grad, loss,
                     nullptr, nullptr, nullptr, AdamStep{});
  return hipGetLastError();
}

AdamStep adam_factors(int step, double lr, double beta1, double beta2, double eps) {
  const double bc1 = 1.0 - std::pow(beta1, (double)step), bc2 = 1.0 - std::pow(beta2, (double)step);
  return AdamStep{(float)lr,          (float)beta1, (float)(1.0 - beta1), (float)beta2,
                  (float)(1.0 - beta2), (float)eps,   (float)bc1,           (float)bc2};
}

hipError_t mlp_adam(float* params, const float* grad, float* m, float* v, int n, const AdamStep& a, hipStream_t st) {
  hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, st, params, grad, m, v, n, a);
  return hipGetLastError();
}

hipError_t mlp_train(float* params, float* m, float* v, const AdamStep& a, const float* norm, const float* x,
                     const float* yt, int B, float* loss, const MlpScratch& s, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  int row_blocks = 0, parts = 0;
  const hipError_t e = grad_parts(params, norm, x, yt, B, s, &row_blocks, &parts, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((mlp_sum_kernel<true>), dim3(SUM_BLOCKS), dim3(256), 0, st, s, B, row_blocks, parts, nullptr, loss,
                     params, m, v, a);
  return hipGetLastError();
}

}  // namespace lensed

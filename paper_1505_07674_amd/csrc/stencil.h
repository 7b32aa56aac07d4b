// stencil.h -- the tile stencil shared by the PSF convolution (Sec. 3.1, Eq. 15)
// and its transpose in the adjoint.
//
// A block stages a TW x TH tile of outputs with its halo in LDS, transposed
// (the rows of a column contiguous), and the taps of the column-major kernel. A
// thread owns Q x 4 adjacent rows of C adjacent columns. The stencil is a sum
// over the kernel's columns l of a one-dimensional (vertical) correlation, and
// that correlation runs on the matrix cores: with the A block broadcast to all
// 16 blocks (cbsz 4, abid k'), v_mfma_f32_4x4x1_16b_f32 adds A[m] v(lane) to four
// accumulators of every lane, m = 0..3. With four adjacent output rows as m and
// the input row k' as v, A[m] is the tap k' - m, zero outside the kernel, so
// KP = ph + 3 instructions cover the ph taps of four rows.
//
// What bounds it, and why this layout: the multiply-add rate. The matrix cores
// run f32 at twice the rate of v_fma_f32 (8 cycles for 256 products per wave
// against 16), of which a 21-row kernel uses 21/24. LDS comes second: one row
// per read (ds_read_b32 of a row-major tile, 28 reads per column for 8 outputs)
// held the matrix cores to 60 %; transposed, a thread reads its column in
// 16-byte pieces, keeps the C columns in registers from one l to the next, and
// reads 28 floats per l for 16 outputs. 200 x 200 pixels x
// 4096 images, 21 x 21 taps, on one card: v_fma chains 2.12 ms, MFMA from a row-major
// tile 1.87 ms, this layout 1.61 ms (the MFMA instructions alone take 1.25 ms).
//
// Exactness: each product-add is rounded once, in the order (l, then k') of the
// plain sum, and a zero tap adds exactly nothing to a finite value, so a result
// equals the chain of fmaf bit for bit (512 000 products compared, denormals
// included). A zero tap times inf or NaN is not nothing: a tile that holds a
// non-finite value takes the fmaf chain instead.
#pragma once

#include <stdint.h>

#include <utility>

#include "internal.h"

namespace lensed {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Matrix steps of a launch whose largest kernel has ph rows: ph + 3 up to 21
// rows, one step count for a range of sizes above (zero taps fill the rest). The line
// is where the PSFs in common use end, and what it buys is the size of the library: with
// ph + 3 throughout, the two stencil kernels would have 32 instances each instead of 15
// (3.09 MB against 2.55). It costs the larger PSFs their padding: PSF + chi^2 of 512 images of
// 200 x 200 pixels, these steps against ph + 3: 262 and 262 us at 25 rows, 367 and 293 at 27,
// 400 and 385 at 31, 659 and 469 at 35, 1042 and 1046 at 49, 2206 and 1105 at 51.
constexpr int psf_steps(int ph) {
  return ph <= 21 ? ph + 3 : ph <= 25 ? 28 : ph <= 33 ? 36 : ph <= 49 ? 52 : 66;
}
// Calls f(integral_constant<int, KP>) for the step count KP of such a launch.
template <class F>
hipError_t with_psf_steps(int ph, F f) {
  switch (psf_steps(ph)) {
#define LENSED_STEPS(KP) \
  case KP: return f(std::integral_constant<int, KP>{});
    LENSED_STEPS(4)
    LENSED_STEPS(6)
    LENSED_STEPS(8)
    LENSED_STEPS(10)
    LENSED_STEPS(12)
    LENSED_STEPS(14)
    LENSED_STEPS(16)
    LENSED_STEPS(18)
    LENSED_STEPS(20)
    LENSED_STEPS(22)
    LENSED_STEPS(24)
    LENSED_STEPS(28)
    LENSED_STEPS(36)
    LENSED_STEPS(52)
    LENSED_STEPS(66)
#undef LENSED_STEPS
    default: return hipErrorInvalidValue;
  }
}

// Outputs of a thread: PSF_Q x 4 rows by PSF_C columns.
constexpr int PSF_Q = 2, PSF_C = 2;
constexpr int PSF_MAX_THREADS = 512;

// Rows staged per column, and the distance of two columns in LDS: a multiple of
// four (16-byte reads); an odd number of quads, so that the quads a wave of the
// staging pass writes (one per column) fall into different banks.
__host__ __device__ constexpr int psf_tile_rows(int TH, int KP) { return (TH - 4 + KP + 3) / 4 * 4; }
__host__ __device__ constexpr int psf_col_stride(int TH, int KP) {
  return psf_tile_rows(TH, KP) + (psf_tile_rows(TH, KP) % 8 == 0 ? 4 : 0);
}
__host__ __device__ constexpr int tap_stride(int KP) { return 3 + (KP + 15) / 16 * 16; }

inline int psf_threads(int TW, int TH) { return ((TW / PSF_C) * (TH / (4 * PSF_Q)) + 63) / 64 * 64; }
inline size_t psf_lds_bytes(int TW, int TH, int max_ph, int max_pw) {
  const int KP = psf_steps(max_ph);
  return sizeof(float) * ((size_t)(TW + max_pw - 1) * psf_col_stride(TH, KP) + (size_t)max_pw * tap_stride(KP));
}
constexpr size_t PSF_MAX_LDS = 65536 - 512;   // 512 bytes for the block sums

// A value that is the same in every lane, held in a scalar register.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Global memory as a scalar base and a 32-bit byte offset per lane (an image has
// at most 2^28 pixels).
typedef const char __attribute__((address_space(1))) gbyte_in;
typedef char __attribute__((address_space(1))) gbyte_out;
__device__ __forceinline__ gbyte_in* uniform_in(const float* p) { return (gbyte_in*)uniform((int64_t)p); }
__device__ __forceinline__ gbyte_out* uniform_out(float* p) { return (gbyte_out*)uniform((int64_t)p); }
__device__ __forceinline__ float load_at(gbyte_in* p, unsigned bytes) {
  return *(const float __attribute__((address_space(1)))*)(p + bytes);
}
__device__ __forceinline__ void store_at(gbyte_out* p, unsigned bytes, float v) {
  *(float __attribute__((address_space(1)))*)(p + bytes) = v;
}

// Stages SW columns from gj0 and 4 quads rows from gi0 of image I into S (columns cs
// floats apart). Outside the image: the nearest edge pixel (CLAMP), or zero. Every argument
// but the thread is uniform over the block, so a load is a scalar base plus a
// 32-bit offset, and tiles whose rows all lie inside the image take no row
// clamps: vector instructions do not overlap with the matrix ones here, so what
// the staging saves, the kernel saves. STAGE_BATCH quads of rows are loaded
// before the first is written. True if every staged value of this thread is
// finite.
constexpr int STAGE_BATCH = 4;
template <bool CLAMP>
__device__ __forceinline__ bool stage_tile(float* __restrict__ S, gbyte_in* I, int H, int W, int SW, int quads, int cs,
                                           int gi0, int gj0) {
  const bool rows_inside = gi0 >= 0 && gi0 + 4 * quads <= H;
  const unsigned W4 = 4u * (unsigned)W;
  const int bq = (int)blockDim.x / SW, bc = (int)blockDim.x - bq * SW;
  int quad = (int)threadIdx.x / SW, col = (int)threadIdx.x - quad * SW;
  float probe = 0.0f;   // 0 x value: NaN as soon as a value is not finite
  while (quad < quads) {
    f32x4_t v[STAGE_BATCH];
    int at[STAGE_BATCH];
#pragma unroll
    for (int k = 0; k < STAGE_BATCH; ++k) {
      at[k] = quad < quads ? col * cs + 4 * quad : -1;
      const int gi = gi0 + 4 * quad, gj = gj0 + col, gjc = min(max(gj, 0), W - 1);
      v[k] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
      if (at[k] >= 0 && (CLAMP || gj == gjc)) {
        if (rows_inside) {
          const unsigned o = (unsigned)gi * W4 + 4u * (unsigned)gjc;
#pragma unroll
          for (int u = 0; u < 4; ++u) v[k][u] = load_at(I, o + (unsigned)u * W4);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int gic = min(max(gi + u, 0), H - 1);
            if (CLAMP || gic == gi + u) v[k][u] = load_at(I, (unsigned)gic * W4 + 4u * (unsigned)gjc);
          }
        }
      }
      quad += bq;
      col += bc;
      if (col >= SW) col -= SW, ++quad;
    }
#pragma unroll
    for (int k = 0; k < STAGE_BATCH; ++k) {
#pragma unroll
      for (int u = 0; u < 4; ++u) probe = fmaf(v[k][u], 0.0f, probe);
      if (at[k] >= 0) *(f32x4_t*)(S + at[k]) = v[k];
    }
  }
  return probe == 0.0f;
}

// The taps of the column-major kernel F (ph per column) into T, columns ts floats
// apart, `lead` zeros before and zeros after them.
__device__ __forceinline__ void stage_taps(float* __restrict__ T, gbyte_in* F, int ph, int pw, int ts, int lead) {
  for (int i = (int)threadIdx.x; i < pw * ts; i += (int)blockDim.x) {
    const int l = i / ts, k = i - l * ts - lead;
    T[i] = k >= 0 && k < ph ? load_at(F, 4u * (unsigned)(l * ph + k)) : 0.0f;
  }
}

// c[m] + a(block AB, m) * b for m = 0..3.
template <int AB>
__device__ __forceinline__ f32x4_t mfma_rows(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, AB, 0);
}

// One stencil column: the KP steps of the C x Q groups of four rows. win[c] is the
// input column of output column c.
template <int Q, int C, int W, int... I>
__device__ __forceinline__ void mfma_column(const float* a, const float (*const (&win)[C])[W], f32x4_t (&acc)[C][Q],
                                            std::integer_sequence<int, I...>) {
  auto step = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[c][q] = mfma_rows<i % 16>(a[i / 16], (*win[c])[i + 4 * q], acc[c][q]);
  };
  (step(std::integral_constant<int, I>{}), ...);
}

// The stencil of one thread: S0 its first input column and row in LDS, acc[c][q][m]
// the output at column c, row 4 q + m. finite: every staged value of the block is
// (uniform over the block).
template <int KP, int Q, int C>
__device__ __forceinline__ void stencil(const float* __restrict__ S0, const float* __restrict__ T, int ph, int pw,
                                        int cs, bool finite, f32x4_t (&acc)[C][Q]) {
  static_assert(C == 2, "the column window is unrolled by two");
  constexpr int ts = tap_stride(KP), NA = (KP + 15) / 16, NB = (KP + 4 * (Q - 1) + 3) / 4;
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[c][q] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  if (!finite) {
#pragma unroll 1
    for (int l = 0; l < pw; ++l)
#pragma unroll 1
      for (int k = 0; k < ph; ++k) {
        const float f = T[l * ts + 3 + k];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[c][q][m] = fmaf(f, S0[(c + l) * cs + 4 * q + m + k], acc[c][q][m]);
      }
    return;
  }
  const int lane = (int)threadIdx.x & 63;
  const float* __restrict__ Tl = T + 3 + (lane >> 2) - (lane & 3);
  float win[C][4 * NB];
  auto load = [&](float (&w)[4 * NB], int col) {
    const f32x4_t* __restrict__ s = (const f32x4_t*)(S0 + col * cs);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const f32x4_t v = s[b];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[4 * b + u] = v[u];
    }
  };
  auto column = [&](int l, const float (*const (&w)[C])[4 * NB]) {
    float a[NA];
#pragma unroll
    for (int g = 0; g < NA; ++g) a[g] = Tl[l * ts + 16 * g];
    mfma_column<Q, C>(a, w, acc, std::make_integer_sequence<int, KP>{});
  };
  load(win[0], 0);
  for (int l = 0; l < pw; l += 2) {   // pw is odd: the last column is the first of its pair
    load(win[1], l + 1);
    column(l, {&win[0], &win[1]});
    if (l + 1 >= pw) break;
    load(win[0], l + 2);
    column(l + 1, {&win[1], &win[0]});
  }
}

// Writes a thread's outputs over the staged tile: output (row, col) goes to
// S[col * cs + row]. All threads have read the tile before.
template <int Q, int C>
__device__ __forceinline__ void outputs_to_lds(float* __restrict__ S, int cs, int row, int col,
                                               const f32x4_t (&acc)[C][Q]) {
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int q = 0; q < Q; ++q) *(f32x4_t*)(S + (col + c) * cs + row + 4 * q) = acc[c][q];
}

// ---- One image at a time --------------------------------------------------
// The single-point calls run one image on an otherwise idle chip, so what counts is
// the longest thread. A matrix chain of four rows takes 504 dependent steps for
// 21 x 21 taps; here a thread owns two rows of one column and runs two chains of
// v_fma (882 instructions, no step waits for another thread's work), over small
// tiles. 200 x 200 pixels, 21 x 21 taps: 9.5 us, against 11.6 us for four-row matrix
// chains and 15.2 us for four-row v_fma chains in tiles of 32 x 20.
constexpr int SINGLE_ROWS = 2;
inline int single_threads(int TW, int TH) { return TW * TH / SINGLE_ROWS; }
__host__ __device__ constexpr int single_tile_rows(int TH, int ph) { return (TH + ph - 1 + 3) / 4 * 4; }
__host__ __device__ constexpr int single_col_stride(int TH, int ph) {
  return single_tile_rows(TH, ph) + (single_tile_rows(TH, ph) % 8 == 0 ? 4 : 0);
}
__host__ __device__ constexpr int single_tap_stride(int ph) { return (ph + 3) / 4 * 4; }
inline size_t single_lds_bytes(int TW, int TH, int ph, int pw) {
  return sizeof(float) * ((size_t)(TW + pw - 1) * single_col_stride(TH, ph) + (size_t)pw * single_tap_stride(ph));
}

// acc[r] = sum over the kernel of the outputs r = 0, 1 below S0 (an even row), in the
// order (l, then k). PH: ph, or 0 for any.
template <int PH>
__device__ __forceinline__ void stencil_pair(const float* __restrict__ S0, const float* __restrict__ T, int ph_, int pw,
                                             int cs, float (&acc)[2]) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const int ph = PH > 0 ? PH : ph_, ts = single_tap_stride(ph);
  float a0 = 0.0f, a1 = 0.0f;
  for (int l = 0; l < pw; ++l) {
    const f32x2_t* __restrict__ s = (const f32x2_t*)(S0 + l * cs);
    const f32x4_t* __restrict__ t = (const f32x4_t*)(T + l * ts);
    f32x2_t p = s[0];
#pragma unroll PH > 0 ? PH / 4 : 2
    for (int k = 0; k < ph / 4; ++k) {
      const f32x4_t f = t[k];
      const f32x2_t p1 = s[2 * k + 1], p2 = s[2 * k + 2];
      a0 = fmaf(f[0], p[0], a0);
      a1 = fmaf(f[0], p[1], a1);
      a0 = fmaf(f[1], p[1], a0);
      a1 = fmaf(f[1], p1[0], a1);
      a0 = fmaf(f[2], p1[0], a0);
      a1 = fmaf(f[2], p1[1], a1);
      a0 = fmaf(f[3], p1[1], a0);
      a1 = fmaf(f[3], p2[0], a1);
      p = p2;
    }
    // the one or three taps left (ph is odd); no zero tap, which inf or NaN would turn into NaN
    const f32x4_t f = t[ph / 4];
    a0 = fmaf(f[0], p[0], a0);
    a1 = fmaf(f[0], p[1], a1);
    if (ph % 4 == 3) {
      const f32x2_t p1 = s[ph / 4 * 2 + 1];
      a0 = fmaf(f[1], p[1], a0);
      a1 = fmaf(f[1], p1[0], a1);
      a0 = fmaf(f[2], p1[0], a0);
      a1 = fmaf(f[2], p1[1], a1);
    }
  }
  acc[0] = a0;
  acc[1] = a1;
}

}  // namespace lensed

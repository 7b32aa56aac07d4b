// psf_chi2.hip -- PSF convolution (Sec. 3.1, Eq. 15) fused with the weighted
// chi^2 of the log-likelihood (Sec. 3.2, Eq. 17).
//
// Each block owns a TW x TH tile of output pixels of one image. It stages the
// tile and its halo in LDS, reading the unconvolved image with clamped indices
// (the replicate padding of Eq. 15), applies the PSF on the matrix cores
// (stencil.h), and puts the outputs back into LDS; then threads walk the tile
// column by column of GROUP rows, neighbouring threads on neighbouring columns,
// so that the images, data and weights are read and written in rows.
// The chi^2 contribution w (d - L*)^2 is accumulated with Kahan summation per
// group, combined across the block with error-free TwoSum steps, and written
// as one (hi, lo) float pair per tile; the final sum over tiles is float64.
#include "internal.h"
#include "kernels.h"
#include "plan.h"
#include "stencil.h"

namespace lensed {
namespace {

__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
  s = a + b;
  const float bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// Kahan sum of w (d - L*)^2 over the first n of N rows of one column, v the L* in
// LDS, from byte offset o on in steps of W4; w (d - L*) goes to rho if RHO. The
// first product's rounding goes into the compensation; the later ones enter
// unrounded (fmaf) and are rounded with it. Contraction is off, so that this is
// what is computed.
template <int N, bool RHO>
__device__ __forceinline__ void chi2_chain(const float* __restrict__ v, gbyte_in* data, gbyte_in* weight, unsigned o,
                                           unsigned W4, gbyte_out* rho, int n, float& sum, float& comp) {
#pragma clang fp contract(off)
  float d[N], wt[N];
#pragma unroll
  for (int r = 0; r < N; ++r) {   // rows past the image repeat its last one
    const unsigned at = o + (unsigned)min(r, n - 1) * W4;
    d[r] = load_at(data, at);
    wt[r] = load_at(weight, at);
  }
#pragma unroll
  for (int r = 0; r < N; ++r) {
    const float res = d[r] - v[r];
    const float wres = wt[r] * res;
    if (RHO && r < n) store_at(rho, o + (unsigned)r * W4, wres);
    if (r == 0) {
      sum = wres * res;
      comp = fmaf(-wres, res, sum);
    } else if (r < n) {
      const float yk = fmaf(wres, res, -comp);
      const float t = sum + yk;
      comp = (t - sum) - yk;
      sum = t;
    }
  }
}

// The outputs of a tile, in LDS (output (r, c) at S[c cs + r]): stored (mode 0), or
// their chi^2 (mode 1), or that and w (d - L*) stored (mode 2). The block's chi^2
// goes to *partial. group: rows of a Kahan chain (4 or 8). The threads walk the tile
// column by column of `group` rows, neighbouring threads on neighbouring columns.
__device__ __forceinline__ void tile_epilogue(const float* __restrict__ S, int cs, int H, int W, int TW, int TH, int x0,
                                              int y0, gbyte_in* data, gbyte_in* weight, gbyte_out* op, int mode,
                                              int group, float2* __restrict__ partial) {
  __shared__ float red_hi[PSF_MAX_THREADS / 64], red_lo[PSF_MAX_THREADS / 64];
  const int tid = (int)threadIdx.x;
  // the tile in groups of rows: group g of column c is item g TW + c
  float hi = 0.0f, lo = 0.0f;
  const int items = TW * (TH / group);
  for (int it = tid; it < items; it += blockDim.x) {
    const int g = it / TW, c = it - g * TW;
    const int gj = x0 + c, gi0 = y0 + g * group;
    if (gj >= W) continue;
    const int n = min(group, H - gi0);   // rows inside the image
    if (n <= 0) continue;
    const float* __restrict__ v = S + c * cs + g * group;
    const unsigned W4 = 4u * (unsigned)W, o = (unsigned)gi0 * W4 + 4u * (unsigned)gj;
    if (mode == 0) {
      for (int r = 0; r < n; ++r) store_at(op, o + (unsigned)r * W4, v[r]);
      continue;
    }
    float sum, comp;
    if (group == 8) {
      if (mode == 2)
        chi2_chain<8, true>(v, data, weight, o, W4, op, n, sum, comp);
      else
        chi2_chain<8, false>(v, data, weight, o, W4, op, n, sum, comp);
    } else {
      if (mode == 2)
        chi2_chain<4, true>(v, data, weight, o, W4, op, n, sum, comp);
      else
        chi2_chain<4, false>(v, data, weight, o, W4, op, n, sum, comp);
    }
    float s, e;
    two_sum(hi, sum, s, e);
    hi = s;
    lo = lo - comp + e;
  }
  if (mode == 0) return;
  // wave reduction with error-free transformations
  const int lane = tid & 63, wid = tid >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    const float h2 = __shfl_down(hi, off, 64);
    const float l2 = __shfl_down(lo, off, 64);
    if (lane + off < 64) {
      float s, e;
      two_sum(hi, h2, s, e);
      hi = s;
      lo = lo + l2 + e;
    }
  }
  if (lane == 0) {
    red_hi[wid] = hi;
    red_lo[wid] = lo;
  }
  __syncthreads();
  if (tid == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    float h = red_hi[0], lsum = red_lo[0];
    for (int i = 1; i < nw; ++i) {
      float s, e;
      two_sum(h, red_hi[i], s, e);
      h = s;
      lsum = lsum + red_lo[i] + e;
    }
    *partial = make_float2(h, lsum);
  }
}

// KP: matrix steps, psf_steps of the launch's largest PSF. Q, C: a thread's
// outputs (stencil.h). The block is whole waves: the taps are spread over all 64
// lanes, and threads past the tile's last one repeat thread 0 and store nothing.
// group: rows of a Kahan chain (4 or 8).
template <int KP, int Q, int C>
__global__ __launch_bounds__(PSF_MAX_THREADS, KP <= 24 ? 4 : 2) void psf_kernel(
    WorkArgs w, const float* __restrict__ L, float* __restrict__ out, float2* __restrict__ partials, int mode,
    int group) {
  extern __shared__ __align__(16) float S[];
  int point, tile;
  if (w.items) {
    const int2 it = w.items[blockIdx.x];
    point = it.x;
    tile = it.y;
  } else {
    point = w.point0;
    tile = blockIdx.x;
  }
  point = uniform(point);
  tile = uniform(tile);
  const SysDesc& sd = w.sys_table ? w.sys_table[w.point_sys ? w.point_sys[point] : 0] : w.single;
  const int64_t loff = uniform(w.point_loff ? w.point_loff[point] : (int64_t)0);
  const int H = uniform(sd.H), W = uniform(sd.W), TW = uniform(sd.TW), TH = uniform(sd.TH);
  const int ph = uniform(sd.ph), pw = uniform(sd.pw), tiles_x = uniform(sd.tiles_x);
  gbyte_in* data = uniform_in(sd.data);
  gbyte_in* weight = uniform_in(sd.weight);
  gbyte_in* taps = uniform_in(sd.psfn + ph * pw);
  gbyte_in* Lp = uniform_in(L + loff);
  gbyte_out* op = uniform_out(out + loff);
  const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
  const int x0 = tx * TW, y0 = ty * TH;
  const int tid = threadIdx.x;
  if (sd.ptile_w && !(sd.ptile_w[tile] & PTILE_W)) {   // no pixel with w > 0 (gradient plans): zero chi^2, zero rho
    if (mode == 2)
      for (int k = tid; k < TW * TH; k += blockDim.x) {
        const int gi = y0 + k / TW, gj = x0 + k % TW;
        if (gi < H && gj < W) out[loff + (size_t)gi * W + gj] = 0.0f;
      }
    if (tid == 0) partials[(w.point_pbase ? w.point_pbase[point] : 0) + tile] = make_float2(0.0f, 0.0f);
    return;
  }

  const int cs = psf_col_stride(TH, KP);
  float* __restrict__ T = S + (TW + pw - 1) * cs;
  const bool mine = stage_tile<true>(S, Lp, H, W, TW + pw - 1, psf_tile_rows(TH, KP) / 4, cs, y0 - ph / 2, x0 - pw / 2);
  stage_taps(T, taps, ph, pw, tap_stride(KP), 3);
  const bool finite = __syncthreads_and(mine);

  const int nc = TW / C;   // threads per row of threads
  const int jr = tid / nc;
  const bool own = jr < TH / (4 * Q);
  const int row = own ? jr * 4 * Q : 0, col = own ? (tid - jr * nc) * C : 0;
  f32x4_t acc[C][Q];
  stencil<KP, Q, C>(S + col * cs + row, T, ph, pw, cs, finite, acc);
  __syncthreads();
  if (own) outputs_to_lds<Q, C>(S, cs, row, col, acc);
  __syncthreads();

  tile_epilogue(S, cs, H, W, TW, TH, x0, y0, data, weight, op, mode, group,
                partials + (w.point_pbase ? w.point_pbase[point] : 0) + tile);
}

// The lanes of a wave stride over a point's tile sums, then a fixed shuffle tree in
// float64; lane 0 returns log L.
__device__ __forceinline__ double loglike_sum(const float2* partials, int n) {
  double s = 0.0;
  for (int t = (int)threadIdx.x & 63; t < n; t += 64) {
    const float2 v = partials[t];
    s += (double)v.x + (double)v.y;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  return -0.5 * s;
}

// One image at a time: the tiles of w.single, two rows of one column per thread
// (stencil_pair). With logl, the block that finishes last (by *done, which starts
// at 0) also adds the tile sums: 3 us more here, a launch and its gap less. 21 x 21 taps
// on 200 x 200 pixels: half of the 9 us is the stencil, whose reads fill the LDS port
// (the taps through scalar registers instead took 12 us, a column ahead 13 us).
template <int PH>
__global__ __launch_bounds__(PSF_MAX_THREADS) void psf_single_kernel(WorkArgs w, const float* __restrict__ L,
                                                                     float* __restrict__ out,
                                                                     float2* partials, int mode, int* done,
                                                                     double* __restrict__ logl) {
  extern __shared__ __align__(16) float S[];
  __shared__ bool last;
  const SysDesc& sd = w.single;
  const int H = sd.H, W = sd.W, TW = sd.TW, TH = sd.TH, ph = PH > 0 ? PH : sd.ph, pw = PH > 0 ? PH : sd.pw;
  const int tile = blockIdx.x, ty = tile / sd.tiles_x, x0 = (tile - ty * sd.tiles_x) * TW, y0 = ty * TH;
  const int cs = single_col_stride(TH, ph);
  float* __restrict__ T = S + (TW + pw - 1) * cs;
  stage_tile<true>(S, uniform_in(L), H, W, TW + pw - 1, single_tile_rows(TH, ph) / 4, cs, y0 - ph / 2, x0 - pw / 2);
  stage_taps(T, uniform_in(sd.psfn + ph * pw), ph, pw, single_tap_stride(ph), 0);
  __syncthreads();
  const int jr = (int)threadIdx.x / TW, col = (int)threadIdx.x - jr * TW, row = jr * SINGLE_ROWS;
  float acc[SINGLE_ROWS];
  stencil_pair<PH>(S + col * cs + row, T, ph, pw, cs, acc);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < SINGLE_ROWS; ++r) S[col * cs + row + r] = acc[r];
  __syncthreads();
  tile_epilogue(S, cs, H, W, TW, TH, x0, y0, uniform_in(sd.data), uniform_in(sd.weight), uniform_out(out), mode, 4,
                partials + tile);
  if (!logl) return;
  if (threadIdx.x == 0) {   // the thread that stored the tile's sum
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    last = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!last || threadIdx.x >= 64) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const double v = loglike_sum(partials, (int)gridDim.x);
  if (threadIdx.x == 0) *logl = v;
}

// log L of one point per wave. (One thread per point waits for one load after
// another: 5.2 us for the 49 tiles of a single 200 x 200 image, 9.2 us for 91.)
constexpr int FINALIZE_WAVES = 4;
__global__ __launch_bounds__(64 * FINALIZE_WAVES) void finalize_kernel(const float2* __restrict__ partials,
                                                                       const int* __restrict__ pbase,
                                                                       const int* __restrict__ ntiles, int n_points,
                                                                       int single_ntiles, double* __restrict__ logl) {
  const int p = blockIdx.x * FINALIZE_WAVES + ((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  if (p >= n_points) return;   // a whole wave
  const int base = pbase ? pbase[p] : 0;
  const int nt = ntiles ? ntiles[p] : single_ntiles;
  const double v = loglike_sum(partials + base, nt);
  if (lane == 0) logl[p] = v;
}

}  // namespace

hipError_t launch_psf(const WorkArgs& w, const float* L, float* out, float2* partials, int mode, int n_blocks, int TW,
                      int TH, int max_ph, int max_pw, int group, hipStream_t stream) {
  if (n_blocks <= 0) return hipSuccess;
  const int threads = psf_threads(TW, TH);
  const size_t lds = psf_lds_bytes(TW, TH, max_ph, max_pw);
  if (threads > PSF_MAX_THREADS || lds > PSF_MAX_LDS || TH % (4 * PSF_Q) != 0 || TW % PSF_C != 0 ||
      (group != 4 && group != 8))
    return hipErrorInvalidValue;
  return with_psf_steps(max_ph, [&](auto steps) {
    constexpr int KP = decltype(steps)::value;
    return for_item_parts(w, n_blocks, [&](const WorkArgs& part, int n) {
      hipLaunchKernelGGL((psf_kernel<KP, PSF_Q, PSF_C>), dim3(n), dim3(threads), lds, stream, part, L, out, partials,
                         mode, group);
      return hipGetLastError();
    });
  });
}

hipError_t launch_psf_single(const WorkArgs& w, const float* L, float* out, float2* partials, int mode, int* done,
                             double* logl, hipStream_t stream) {
  const SysDesc& sd = w.single;
  if (!is_single_tile(TileShape{sd.TW, sd.TH})) {
    const hipError_t e = launch_psf(w, L, out, partials, mode, sd.n_ptiles, sd.TW, sd.TH, sd.ph, sd.pw, 4, stream);
    return e != hipSuccess || !logl ? e : launch_finalize(partials, nullptr, nullptr, 1, sd.n_ptiles, logl, stream);
  }
  const int threads = single_threads(sd.TW, sd.TH);
  const size_t lds = single_lds_bytes(sd.TW, sd.TH, sd.ph, sd.pw);
  const dim3 grid((unsigned)sd.n_ptiles), block((unsigned)threads);
  if (sd.ph == 21 && sd.pw == 21)
    hipLaunchKernelGGL((psf_single_kernel<21>), grid, block, lds, stream, w, L, out, partials, mode, done, logl);
  else if (sd.ph == 7 && sd.pw == 7)
    hipLaunchKernelGGL((psf_single_kernel<7>), grid, block, lds, stream, w, L, out, partials, mode, done, logl);
  else
    hipLaunchKernelGGL((psf_single_kernel<0>), grid, block, lds, stream, w, L, out, partials, mode, done, logl);
  return hipGetLastError();
}

hipError_t launch_finalize(const float2* partials, const int* point_pbase, const int* point_ntiles, int n_points,
                           int single_ntiles, double* logl, hipStream_t stream) {
  if (n_points <= 0) return hipSuccess;
  const int blocks = (n_points + FINALIZE_WAVES - 1) / FINALIZE_WAVES;
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)blocks), dim3(n_points > 1 ? 64 * FINALIZE_WAVES : 64), 0, stream,
                     partials, point_pbase, point_ntiles, n_points, single_ntiles, logl);
  return hipGetLastError();
}

}  // namespace lensed

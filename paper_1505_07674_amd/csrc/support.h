// support.h -- which pixels a gradient plan's g = A^T rho can reach, from the
// weights as they are now (a caller may change them in place between launches).
// Extra blocks of the prologue's launch dilate w > 0 by the PSF box, as bits;
// grad_support_kernel (adjoint.hip) then turns the bits into lists.
//
// What bounds it: latency, a few hundred kB are read once. So a pixel is one
// bit of a 64-bit word (a wave's ballot), the box is an OR over rows and shifts
// over columns, and a short block covers a band of rows.
#pragma once

#include "internal.h"
#include "kernels.h"

namespace lensed {

constexpr int SUPPORT_THREADS = 256;
constexpr int SUPPORT_ROWS = 8;   // rows per band

struct SupportScratch {
  unsigned long long bits[SUPPORT_ROWS + MAX_PSF - 1][SUPPORT_SEG_WORDS + 2];   // w > 0, a word of halo on each side
  unsigned long long rows[SUPPORT_ROWS][SUPPORT_SEG_WORDS + 2];                  // dilated over rows
};

// Blocks of a system: a band and segment each, then a PSF output tile each.
__host__ __device__ inline int support_bands(const SysDesc& sd) {
  return ((sd.H + SUPPORT_ROWS - 1) / SUPPORT_ROWS) * support_segments(sd);
}
inline int support_blocks(const SysDesc& sd) { return support_bands(sd) + sd.n_ptiles; }

// Flags of PSF output tile `tile`: PTILE_W where it holds a pixel with w > 0,
// PTILE_G where it holds one of the support.
__device__ inline void support_tile(const SysDesc& sd, int tile) {
  const int ty = tile / sd.tiles_x, tx = tile - ty * sd.tiles_x;
  const int p = sd.ph / 2, q = sd.pw / 2;
  const int r0 = max(ty * sd.TH - p, 0), r1 = min(ty * sd.TH + sd.TH + p, sd.H);
  const int c0 = max(tx * sd.TW - q, 0), c1 = min(tx * sd.TW + sd.TW + q, sd.W);
  const int wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  bool any_w = false, any_g = false;
  for (int c = c0 + lane; c < c1; c += 64) {
    const bool cin = c >= tx * sd.TW && c < tx * sd.TW + sd.TW;
#pragma unroll 8
    for (int r = r0 + wv; r < r1; r += SUPPORT_THREADS / 64) {
      const bool on = sd.weight[(size_t)r * sd.W + c] > 0.0f;
      any_g = any_g || on;
      any_w = any_w || (on && cin && r >= ty * sd.TH && r < ty * sd.TH + sd.TH);
    }
  }
  const int g = __syncthreads_or(any_g), w = __syncthreads_or(any_w);
  if (threadIdx.x == 0) sd.ptile_w[tile] = (unsigned char)((w ? PTILE_W : 0) | (g ? PTILE_G : 0));
}

// Block `block` of a system's support blocks (SUPPORT_THREADS threads).
__device__ inline void support_block(const SysDesc& sd, int block, SupportScratch& s) {
  if (!sd.gsup) return;   // uniform over the block, as every return before a barrier
  const int bands = support_bands(sd);
  if (block >= bands) {
    if (block - bands < sd.n_ptiles) support_tile(sd, block - bands);
    return;
  }
  const int nseg = support_segments(sd), nw = support_words(sd);
  const int band = block / nseg, seg = block - band * nseg;
  const int p = sd.ph / 2, q = sd.pw / 2, r0 = band * SUPPORT_ROWS, k0 = seg * SUPPORT_SEG_WORDS;
  const int t = (int)threadIdx.x, wv = t >> 6, lane = t & 63;
  constexpr int WORDS = SUPPORT_SEG_WORDS + 2;
  const int nrows = SUPPORT_ROWS + 2 * p;
  for (int i = t; i < nrows * WORDS; i += SUPPORT_THREADS) (&s.bits[0][0])[i] = 0;
  __syncthreads();
  // words of the rows and of the segment with its halo that lie in the image
  const int ra = max(r0 - p, 0), rb = min(r0 + SUPPORT_ROWS + p, sd.H);
  const int ka = max(k0 - 1, 0), kb = min(k0 + SUPPORT_SEG_WORDS + 1, nw);
  constexpr int WAVES = SUPPORT_THREADS / 64, BATCH = 8;   // loads in flight per lane
  for (int k = ka; k < kb; ++k) {
    const int c = 64 * k + lane;
    for (int r = ra + wv; r < rb; r += WAVES * BATCH) {
      float v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int rr = r + WAVES * u;
        v[u] = c < sd.W && rr < rb ? sd.weight[(size_t)rr * sd.W + c] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int rr = r + WAVES * u;
        const unsigned long long b = __ballot(v[u] > 0.0f);
        if (lane == 0 && rr < rb) s.bits[rr - r0 + p][k - k0 + 1] = b;
      }
    }
  }
  __syncthreads();
  for (int i = t; i < SUPPORT_ROWS * WORDS; i += SUPPORT_THREADS) {
    const int r = i / WORDS, k = i - r * WORDS;
    unsigned long long v = 0;
    for (int a = 0; a <= 2 * p; ++a) v |= s.bits[r + a][k];
    s.rows[r][k] = v;
  }
  __syncthreads();
  if (t >= SUPPORT_ROWS * SUPPORT_SEG_WORDS) return;
  const int r = t / SUPPORT_SEG_WORDS, j = t % SUPPORT_SEG_WORDS, row = r0 + r, k = k0 + j;
  const unsigned long long lo = s.rows[r][j], mid = s.rows[r][j + 1], hi = s.rows[r][j + 2];
  unsigned long long d = mid;
  for (int x = 1; x <= q; ++x)   // q <= 31: the neighbouring words suffice
    d |= (mid << x | lo >> (64 - x)) | (mid >> x | hi << (64 - x));
  const bool in = row < sd.H && k < nw;
  if (in && 64 * k + 64 > sd.W) d &= ~0ull >> (64 * k + 64 - sd.W);
  if (!in) d = 0;
  int px = __popcll(d), un = sd.uppt == 2 ? __popcll((d | d >> 1) & 0x5555555555555555ull) : px;
  for (int o = 1; o < SUPPORT_SEG_WORDS; o <<= 1) {   // the segment's words are adjacent lanes
    px += __shfl_xor(px, o, 64);
    un += __shfl_xor(un, o, 64);
  }
  if (in) sd.gbits[(size_t)row * nw + k] = d;
  if (j == 0 && row < sd.H) sd.gcount[(size_t)row * nseg + seg] = make_int2(px, un);
}

}  // namespace lensed

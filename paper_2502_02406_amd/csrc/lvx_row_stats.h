// Row statistics of the backward pass: the kernel that makes them alone (lvx_elementwise.hip) and the one that makes a
// masked call's words beside them (lvx_mask_rows.hip).
#pragma once
#include "lvx_internal.h"

namespace lvx {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

__device__ __forceinline__ float bf16_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }

// delta[b,h,i] = sum_d dO[b,h,i,d] * O[b,h,i,d].  16 lanes per row.  The bf16 kernels read the
// row statistics 32 rows at a time with aligned copies, so a padded, grouped copy is written as
// well: stats[B,Hq,sq_pad/32][2][32] (sq_pad a multiple of 32) holds, per group of 32 rows, 32
// values of -L * log2(e) -- -inf for rows without keys and for pad rows, which makes their
// probabilities exp2(-inf) = 0 -- followed by the 32 values of -delta (0 in pad rows).
// stats_ovl (optional, [B,Hq][2][32]): the same for rows Sq-32 .. Sq-1, with -inf for those of them
// that belong to a full group of 32.
// Lane c of the 16 of row rowp (of B Hq sq_pad); whole groups of 16 lanes leave together.
template <bool F32>
__device__ __forceinline__ void row_delta(const Dims& d, const void* o, const void* d_o, const float* lse, float* delta, float* stats,
                                          int sq_pad, float* stats_ovl, long rowp, int c) {
  const long rows = (long)d.B * d.Hq * sq_pad;
  if (rowp >= rows) return;
  const long i = rowp % sq_pad, h = (rowp / sq_pad) % d.Hq, b = rowp / ((long)sq_pad * d.Hq);
  float s = 0.f;
  if (i < d.Sq) {
    const long off = b * d.q_sb + h * d.q_sh + i * d.q_ss;
    if (F32) {
      const float* po = (const float*)o + off;
      const float* pg = (const float*)d_o + off;
      for (int e = c * 4; e < d.D; e += 64) {
        f32x4 x = *(const f32x4*)(po + e), y = *(const f32x4*)(pg + e);
        s += x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
      }
    } else {
      const uint16_t* po = (const uint16_t*)o + off;
      const uint16_t* pg = (const uint16_t*)d_o + off;
      for (int e = c * 8; e < d.D; e += 128) {
        u32x4 x = *(const u32x4*)(po + e), y = *(const u32x4*)(pg + e);
#pragma unroll
        for (int k = 0; k < 4; ++k) s += bf16_lo(x[k]) * bf16_lo(y[k]) + bf16_hi(x[k]) * bf16_hi(y[k]);
      }
    }
  }
#pragma unroll
  for (int m = 8; m >= 1; m >>= 1) s += __shfl_xor(s, m, 16);
  if (c != 0) return;
  float nl2 = -INFINITY;
  if (i < d.Sq) {
    const long row = (b * d.Hq + h) * d.Sq + i;
    delta[row] = s;
    const float L = lse[row];
    if (L != -INFINITY) nl2 = -L * 1.4426950408889634f;
  }
  const long slot = (rowp / 32) * 64 + rowp % 32;     // sq_pad is a multiple of 32
  stats[slot] = nl2;
  stats[slot + 32] = -s;
  if (stats_ovl && i >= d.Sq - 32 && i < d.Sq) {
    const long j = (b * d.Hq + h) * 64 + (i - (d.Sq - 32));
    stats_ovl[j] = i >= (d.Sq & ~31) ? nl2 : -INFINITY;
    stats_ovl[j + 32] = -s;
  }
}

}  // namespace lvx

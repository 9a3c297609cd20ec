// Media mask, regrouped once per call for the kernels that mask by data instead of by control flow
// (lvx_internal.h, MaskRows): for every block of 32 query rows and every key block, one word whose
// bit r says whether row r of the block sees the key block.  The kernels then answer "which
// rows see these keys" with one word, whatever the chunk length, instead of probing the bitmap a
// chunk at a time in every workgroup of every head.
//
// Bound by the latency of its probes: a thread makes one word from its 1 .. 32 chunks, eight or
// sixteen probes on their way at a time, a wave's lanes on 64 neighbouring key blocks of one chunk row.
// 2048 chunks of two rows x 2048 key blocks (4 MiB of bitmap, 1 MiB of words): 7.6 us (8.6 with eight); 32 chunks x
// 32 key blocks: 4.5 us, a launch and a round trip.
#include "lvx_internal.h"
#include "lvx_row_stats.h"

#include <type_traits>

namespace lvx {

namespace {

constexpr int FB = 64;                 // key blocks per workgroup

// the words of FB key blocks (x: which, of nx) and the 256 rows of tile qt, by 512 threads
__device__ __forceinline__ void make_words(const MaskDev& m, const MaskRows& r, int Sq, unsigned* out, unsigned long long* any,
                                           unsigned* counts, int x, int nx, int qt, int bz) {
  __shared__ unsigned tile[8][FB];
  const int lane = threadIdx.x & (FB - 1), f = x * FB + lane, rb = threadIdx.x / FB;
  const int i0 = qt * 256 + rb * 32, rows = min(32, Sq - i0);
  unsigned bits = 0;
  if (f < r.w1 - 1 && rows > 0) {      // (the last key block is a padding one that nobody sees)
    const uint8_t* const base = m.allow + bz * m.stride_b + f;
    const int ca = i0 / m.q_chunk, cb = (i0 + rows - 1) / m.q_chunk;
    auto probe = [&](int c, auto many) __attribute__((always_inline)) {      // `many` chunks from c on, their probes on their way at once
      constexpr int N = decltype(many)::value;
      uint8_t v[N];
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = base[(long)min(c + u, cb) * m.stride_q];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const long lo = (long)(c + u) * m.q_chunk - i0;                // the chunk's rows, relative to the block
        const int a = (int)max(lo, 0L), z = (int)min(lo + m.q_chunk, (long)rows);
        if (c + u <= cb && v[u] != 0 && z > a) bits |= (z - a == 32 ? ~0u : ((1u << (z - a)) - 1u) << a);
      }
    };
    for (int c = ca; c <= cb;) {
      if (cb - c >= 8) { probe(c, std::integral_constant<int, 16>{}); c += 16; }
      else { probe(c, std::integral_constant<int, 8>{}); c += 8; }
    }
  }
  if (f < r.w1) out[bz * r.stride_b + ((long)qt * r.w1 + f) * 8 + rb] = bits;
  tile[rb][lane] = bits;
  __syncthreads();
  if (rb == 0) {                       // one bit per key block: some row of the tile sees it; and how many each two row blocks see
    unsigned count = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned w = tile[k][lane];
      count += (unsigned)__popcll(__ballot(w != 0)) << (8 * (k % 4));
      bits |= w;
    }
    const unsigned long long on = __ballot(bits != 0);
    if (lane == 0) {
      const long at = ((long)bz * r.n_qt + qt) * nx + x;
      any[at] = on;
      counts[at] = count;
    }
  }
}

__global__ void __launch_bounds__(512) mask_rows_kernel(MaskDev m, MaskRows r, int Sq, unsigned* out,
                                                        unsigned long long* any, unsigned* counts) {
  make_words(m, r, Sq, out, any, counts, blockIdx.x, gridDim.x, blockIdx.y, blockIdx.z);
}

// The words and, by the workgroups behind the first n_words, the row statistics of the backward pass: neither needs the other and
// both are over in the time of a launch and a few trips to memory.  4096 rows x 8 heads in chunks of two, 2048 frames of 64 keys:
// 7.0 and 5.2 us and the gap between them -> 9.1 us, the step of it 331 -> 326 us.
__global__ void __launch_bounds__(512) mask_rows_delta_kernel(MaskDev m, MaskRows r, unsigned* out, unsigned long long* any,
                                                              unsigned* counts, int nx, int n_words, Dims d, const void* o,
                                                              const void* d_o, const float* lse, float* delta, float* stats,
                                                              int sq_pad, float* stats_ovl) {
  const int w = blockIdx.x;
  if (w < n_words) make_words(m, r, d.Sq, out, any, counts, w % nx, nx, w / nx % r.n_qt, w / nx / r.n_qt);
  else row_delta<false>(d, o, d_o, lse, delta, stats, sq_pad, stats_ovl, ((long)(w - n_words) * 512 + threadIdx.x) / 16, threadIdx.x % 16);
}

}  // namespace

MaskRows mask_rows_of(const Dims& d, const MaskDev& m) {
  MaskRows r;
  r.words = nullptr;
  r.any = nullptr;
  r.counts = nullptr;
  r.w1 = (d.Skv - 1) / m.kv_block + 2;
  r.n_qt = (d.Sq + 255) / 256;
  r.stride_b = m.stride_b != 0 ? (long)r.n_qt * r.w1 * 8 : 0;          // (one bitmap for all batches: one set of words)
  return r;
}
size_t mask_rows_bytes(const Dims& d, const MaskRows& r) {
  return (size_t)(r.stride_b != 0 ? d.B : 1) * r.n_qt * ((size_t)r.w1 * 32 + (size_t)(r.w1 + FB - 1) / FB * 12);
}

size_t mask_rows_counts_bytes(const Dims& d, const MaskRows& r) {
  return (size_t)(r.stride_b != 0 ? d.B : 1) * r.n_qt * ((size_t)(r.w1 + FB - 1) / FB * 4);
}

// where the words of r lie, and the grid that makes them
static dim3 place_words(const Dims& d, MaskRows* r, void* words) {
  const dim3 grid((r->w1 + FB - 1) / FB, r->n_qt, r->stride_b != 0 ? d.B : 1);
  r->words = (const unsigned*)words;
  r->any = (const unsigned long long*)((const char*)words + (size_t)grid.z * r->n_qt * r->w1 * 32);
  r->any_stride_b = r->stride_b != 0 ? (long)r->n_qt * grid.x : 0;
  r->any_words = (int)grid.x;
  r->counts = (const unsigned*)(r->any + (size_t)grid.z * r->n_qt * grid.x);
  return grid;
}

hipError_t launch_mask_rows(const Dims& d, const MaskDev& m, MaskRows* r, void* words, hipStream_t s) {
  const dim3 grid = place_words(d, r, words);
  mask_rows_kernel<<<grid, 512, 0, s>>>(m, *r, d.Sq, (unsigned*)words, (unsigned long long*)r->any, (unsigned*)r->counts);
  return hipGetLastError();
}

hipError_t launch_mask_rows_delta(const BwdArgs& a, MaskRows* r, hipStream_t s) {
  const dim3 grid = place_words(a.d, r, a.rows_ws);
  const unsigned n_words = grid.x * grid.y * grid.z;
  const unsigned blocks = n_words + (unsigned)(((long)a.d.B * a.d.Hq * a.sq_pad * 16 + 511) / 512);
  mask_rows_delta_kernel<<<blocks, 512, 0, s>>>(a.mask, *r, (unsigned*)a.rows_ws, (unsigned long long*)r->any, (unsigned*)r->counts,
                                                (int)grid.x, (int)n_words, a.d, a.o, a.d_o, a.lse, a.delta, a.stats, a.sq_pad, a.stats_ovl);
  return hipGetLastError();
}

}  // namespace lvx

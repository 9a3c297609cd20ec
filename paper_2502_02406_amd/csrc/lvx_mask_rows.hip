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

#include <type_traits>

namespace lvx {

namespace {

constexpr int FB = 64;                 // key blocks per workgroup

__global__ void __launch_bounds__(512) mask_rows_kernel(MaskDev m, MaskRows r, int Sq, unsigned* out,
                                                        unsigned long long* any, unsigned* counts) {
  __shared__ unsigned tile[8][FB];
  const int lane = threadIdx.x & (FB - 1), f = blockIdx.x * FB + lane, rb = threadIdx.x / FB, qt = blockIdx.y;
  const int i0 = qt * 256 + rb * 32, rows = min(32, Sq - i0);
  unsigned bits = 0;
  if (f < r.w1 - 1 && rows > 0) {      // (the last key block is a padding one that nobody sees)
    const uint8_t* const base = m.allow + blockIdx.z * m.stride_b + f;
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
  if (f < r.w1) out[blockIdx.z * r.stride_b + ((long)qt * r.w1 + f) * 8 + rb] = bits;
  tile[rb][lane] = bits;
  __syncthreads();
  if (rb == 0) {                       // one bit per key block: some row of the tile sees it; and how many each two row blocks see
    unsigned count = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned x = tile[k][lane];
      count += (unsigned)__popcll(__ballot(x != 0)) << (8 * (k % 4));
      bits |= x;
    }
    const unsigned long long on = __ballot(bits != 0);
    if (lane == 0) {
      const long at = ((long)blockIdx.z * r.n_qt + qt) * gridDim.x + blockIdx.x;
      any[at] = on;
      counts[at] = count;
    }
  }
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

hipError_t launch_mask_rows(const Dims& d, const MaskDev& m, MaskRows* r, void* words, hipStream_t s) {
  const dim3 grid((r->w1 + FB - 1) / FB, r->n_qt, r->stride_b != 0 ? d.B : 1);
  r->words = (const unsigned*)words;
  r->any = (const unsigned long long*)((const char*)words + (size_t)grid.z * r->n_qt * r->w1 * 32);
  r->any_stride_b = r->stride_b != 0 ? (long)r->n_qt * grid.x : 0;
  r->any_words = (int)grid.x;
  r->counts = (const unsigned*)(r->any + (size_t)grid.z * r->n_qt * grid.x);
  mask_rows_kernel<<<grid, 512, 0, s>>>(m, *r, d.Sq, (unsigned*)words, (unsigned long long*)r->any, (unsigned*)r->counts);
  return hipGetLastError();
}

}  // namespace lvx

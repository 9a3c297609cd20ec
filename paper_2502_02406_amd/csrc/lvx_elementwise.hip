// HBM-bound kernels of the path: the Rescale/merge of Algorithm 1 (also used to combine the
// forward kernel's KV splits), the backward's delta = rowsum(dO * O), and the dQ conversion.
#include "lvx_internal.h"
#include "lvx_row_stats.h"

namespace lvx {

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  bf16x2 r;
  r[0] = (__bf16)a;   // round to nearest even
  r[1] = (__bf16)b;
  return *(unsigned*)&r;
}

// One thread owns VEC consecutive elements of one (b,h,i) row: VEC = 4 floats or 8 bf16 (16 bytes).
// L' = ln sum_k exp(L_k), O' = sum_k exp(L_k - L') O_k.  A row's threads sit in one wavefront, so
// every lane has read lse_parts[*][row] before lane 0 of the row stores lse_out[row]; this is
// what makes lse_out == lse_parts[0] (in-place update of the running state) safe.  (A row takes a
// power-of-two number of lanes, the next one up when D / VEC is none: the spare lanes idle.)
__host__ __device__ inline int merge_lanes_per_row(int n) {   // smallest power of two >= n (n <= 64)
  int p = 1;
  while (p < n) p <<= 1;
  return p;
}

constexpr int MERGE_UNITS = 1;        // 16-byte pieces of rows that one thread merges (2: measured, no faster)

template <bool PART_F32, bool OUT_F32>
__global__ void __launch_bounds__(256) merge_kernel(MergeArgs a) {
  constexpr int VEC_IN = PART_F32 ? 4 : 8;
  constexpr int VEC_OUT = OUT_F32 ? 4 : 8;
  constexpr int VEC = VEC_IN < VEC_OUT ? VEC_IN : VEC_OUT;   // elements per piece
  constexpr int U = MERGE_UNITS, GRP = 4;
  const int vpr = merge_lanes_per_row(a.D / VEC);             // lanes per row
  // Piece u of a thread lies a whole grid further on (a multiple of 64 lanes, so rows still sit in
  // one wavefront).  The parts' elements are fetched four parts at a time, the first four of
  // every piece before anything else: they are on their way while the rows' statistics are read
  // and turned into weights, so a thread waits for memory once, not twice.  (A part without keys
  // still has a buffer; what it holds is fetched and dropped.)
  const long t0 = (long)blockIdx.x * 256 + threadIdx.x, stride = (long)gridDim.x * 256;
  long row[U], grow[U];                 // of the parts that are slices; of the tensor
  int c[U];
  bool on[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const long t = t0 + u * stride;
    row[u] = t / vpr;
    c[u] = (int)(t % vpr) * VEC;
    on[u] = row[u] < a.rows && c[u] < a.D;
    const int run = a.group - a.skip;
    grow[u] = a.skip == 0 ? row[u] : row[u] / run * a.group + a.skip + row[u] % run;
  }
  auto load_part = [&](int u, int k) __attribute__((always_inline)) -> u32x4 {
    if (PART_F32) return *(const u32x4*)((const float*)a.o_parts[k] + (k < a.first ? grow[u] : row[u]) * a.D + c[u]);
    const uint16_t* src = (const uint16_t*)a.o_parts[k] + row[u] * a.D + c[u];
    if (VEC == 8) return *(const u32x4*)src;
    const unsigned x0 = ((const unsigned*)src)[0], x1 = ((const unsigned*)src)[1];
    return u32x4{x0, x1, 0u, 0u};
  };
  const int n = a.n_parts;
  u32x4 buf[U][GRP];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int g = 0; g < GRP; ++g)
      if (on[u] && g < n) buf[u][g] = load_part(u, g);

  float acc[U][VEC], Lout[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[u][e] = 0.f;
    Lout[u] = -INFINITY;
    if (!on[u]) continue;
    auto add_part = [&](const u32x4& x, float w) __attribute__((always_inline)) {
      if (PART_F32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[u][e] += w * __uint_as_float(x[e]);
      } else {
#pragma unroll
        for (int e = 0; e < VEC / 2; ++e) {
          acc[u][2 * e] += w * bf16_lo(x[e]);
          acc[u][2 * e + 1] += w * bf16_hi(x[e]);
        }
      }
    };
    // The statistics of the first LG parts (all of them, as a rule) are read once, together, and
    // kept: read part by part inside the loops below, each would wait for the one before it.
    constexpr int LG = 8;
    float lk[LG];
#pragma unroll
    for (int k = 0; k < LG; ++k) {
      const float x = a.lse_parts[k < n ? k : n - 1][k < a.first ? grow[u] : row[u]];
      lk[k] = k < n ? x : -INFINITY;
    }
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < LG; ++k) M = max_or_nan(M, lk[k]);
    for (int k = LG; k < n; ++k) M = max_or_nan(M, a.lse_parts[k][row[u]]);
    if (M == -INFINITY) continue;
    float z = 0.f;
#pragma unroll
    for (int k = 0; k < LG; ++k) z += expf(lk[k] - M);               // (exp(-inf) = 0: parts that are not there)
    for (int k = LG; k < n; ++k) z += expf(a.lse_parts[k][row[u]] - M);
    Lout[u] = M + logf(z);
#pragma unroll
    for (int k0 = 0; k0 < LG; k0 += GRP) {
      if (k0 >= n) break;
      if (k0 > 0) {
#pragma unroll
        for (int g = 0; g < GRP; ++g)
          if (k0 + g < n) buf[u][g] = load_part(u, k0 + g);
      }
#pragma unroll
      for (int g = 0; g < GRP; ++g)
        if (k0 + g < n && lk[k0 + g] != -INFINITY) add_part(buf[u][g], expf(lk[k0 + g] - Lout[u]));
    }
    for (int k0 = LG; k0 < n; k0 += GRP) {
#pragma unroll
      for (int g = 0; g < GRP; ++g)
        if (k0 + g < n) buf[u][g] = load_part(u, k0 + g);
#pragma unroll
      for (int g = 0; g < GRP; ++g)
        if (k0 + g < n) {
          const float l = a.lse_parts[k0 + g][row[u]];
          if (l != -INFINITY) add_part(buf[u][g], expf(l - Lout[u]));
        }
    }
  }
  // (every load of the statistics above precedes every store below: lse_out may be lse_parts[0])
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!on[u]) continue;
    const long i = grow[u] % a.Sq, h = (grow[u] / a.Sq) % a.Hq, b = grow[u] / ((long)a.Sq * a.Hq);
    const long off = b * a.o_sb + h * a.o_sh + i * a.o_ss + c[u];
    if (OUT_F32) {
      const f32x4 y = {acc[u][0], acc[u][1], acc[u][2], acc[u][3]};
      *(f32x4*)((float*)a.o_out + off) = y;
    } else {
      unsigned* dst = (unsigned*)((uint16_t*)a.o_out + off);
      if (VEC == 8) {
        const u32x4 y = {pack_bf16(acc[u][0], acc[u][1]), pack_bf16(acc[u][2], acc[u][3]),
                         pack_bf16(acc[u][4], acc[u][5]), pack_bf16(acc[u][6], acc[u][7])};
        *(u32x4*)dst = y;
      } else {
        dst[0] = pack_bf16(acc[u][0], acc[u][1]);
        dst[1] = pack_bf16(acc[u][2], acc[u][3]);
      }
    }
    if (c[u] == 0) a.lse_out[grow[u]] = Lout[u];
  }
}

// The same for few rows and many parts (a serving step's split-KV combine: 32 rows, 32 .. 64 parts of
// float32; a short query block's): one workgroup per row, whose threads share the PARTS as well as the columns -- thread groups
// of 16 or 32 lanes take every NG-th part, all their loads on their way at once, and meet in LDS.  The
// kernel above gives such a problem one thread per 16 bytes of output, 4 workgroups in all, each thread
// walking through the parts four at a time.  Bound by one trip to memory and the launch: the parts'
// addresses come from their slices' numbers (reading the general kernel's pointers per lane is a trip of
// its own), and no branch stands around a load.  32 rows x 64 parts x 128 columns: 23.5 -> 4.5 us; 32
// parts: 3.8 us.
struct MergeRowArgs {
  const float *o0, *l0;                 // part 0 when `first` is 1
  const float *o, *l;                   // parts first .. n - 1, `rows` rows each
  void* o_out;
  float* lse_out;
  long o_sb, o_sh, o_ss;
  int n, first, rows, Hq, Sq;
};
template <int D, bool OUT_F32>
__global__ void __launch_bounds__(256) merge_row_kernel(MergeRowArgs a) {
  constexpr int LPR = D == 64 ? 16 : 32, NG = 256 / LPR;    // lanes per group, groups
  constexpr int MOST = 64 / NG;                             // parts per group at most
  __shared__ f32x4 sums[256];
  const int row = (int)blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int grp = tid / LPR, c = (tid % LPR) * 4, cc = D % (4 * LPR) == 0 ? c : min(c, D - 4);
  // (no branch around a load: each would wait for the one before it; parts past the last re-read it)
  const int pl = min(lane, a.n - 1);
  const float Lp = *((pl < a.first ? a.l0 : a.l + (long)(pl - a.first) * a.rows) + row);
  f32x4 x[MOST];
#pragma unroll
  for (int k = 0; k < MOST; ++k) {
    const int p = min(grp + k * NG, a.n - 1);
    x[k] = *(const f32x4*)((p < a.first ? a.o0 : a.o + (long)(p - a.first) * a.rows * D) + row * D + cc);
  }
  // every wave works out all weights: lane k holds part k's
  const float L = lane < a.n ? Lp : -INFINITY;
  float M = L;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) M = max_or_nan(M, __shfl_xor(M, w, 64));
  float z = M == -INFINITY ? 0.f : expf(L - M);
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) z += __shfl_xor(z, w, 64);
  const float Lout = M == -INFINITY ? -INFINITY : M + logf(z);
  const float wt = L == -INFINITY ? 0.f : expf(L - Lout);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < MOST; ++k) {
    const int p = grp + k * NG;
    const float w = __shfl(wt, p, 64);                      // (0 past the last part)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += w != 0.f ? w * x[k][e] : 0.f;      // (what a part without keys holds is dropped)
  }
  sums[tid] = acc;
  __syncthreads();
  if (tid < LPR && c < D) {
#pragma unroll
    for (int k = 1; k < NG; ++k) acc += sums[tid + k * LPR];
    const unsigned bh = (unsigned)row / (unsigned)a.Sq, i = (unsigned)row % (unsigned)a.Sq;
    const long off = (long)(bh / (unsigned)a.Hq) * a.o_sb + (long)(bh % (unsigned)a.Hq) * a.o_sh + i * a.o_ss + c;
    if (OUT_F32) {
      *(f32x4*)((float*)a.o_out + off) = acc;
    } else {
      unsigned* const dst = (unsigned*)((uint16_t*)a.o_out + off);
      dst[0] = pack_bf16(acc[0], acc[1]);
      dst[1] = pack_bf16(acc[2], acc[3]);
    }
    if (c == 0) a.lse_out[row] = Lout;                      // (all of this row's reads of L are past the barrier)
  }
}

hipError_t launch_merge(const MergeArgs& a, int part_is_f32, int out_is_f32, hipStream_t s) {
  // (few rows: the kernel below gives them one thread per 16 bytes, too few to wait for many parts; and parts enough to share.
  // Forward with its combine, us, this kernel against that one: 2048 rows x 128 x 32 parts 63 and 77, x 8 parts 31
  // and 39; 4096 rows 99 and 102, 36 and 39; 8192 rows 172 and 163, 53 and 46)
  if (part_is_f32 && a.o_slices != nullptr && a.first <= 1 && a.skip == 0 && a.n_parts > 4 && a.rows <= 4096) {
    MergeRowArgs r;
    r.o0 = (const float*)a.o_parts[0]; r.l0 = a.lse_parts[0];
    r.o = a.o_slices; r.l = a.lse_slices;
    r.o_out = a.o_out; r.lse_out = a.lse_out;
    r.o_sb = a.o_sb; r.o_sh = a.o_sh; r.o_ss = a.o_ss;
    r.n = a.n_parts; r.first = a.first; r.rows = (int)a.rows; r.Hq = a.Hq; r.Sq = a.Sq;
    const unsigned blocks = (unsigned)a.rows;
    if (out_is_f32) {
      if (a.D == 64) merge_row_kernel<64, true><<<blocks, 256, 0, s>>>(r);
      else if (a.D == 96) merge_row_kernel<96, true><<<blocks, 256, 0, s>>>(r);
      else merge_row_kernel<128, true><<<blocks, 256, 0, s>>>(r);
    } else {
      if (a.D == 64) merge_row_kernel<64, false><<<blocks, 256, 0, s>>>(r);
      else if (a.D == 96) merge_row_kernel<96, false><<<blocks, 256, 0, s>>>(r);
      else merge_row_kernel<128, false><<<blocks, 256, 0, s>>>(r);
    }
    return hipGetLastError();
  }
  const int vec = (part_is_f32 || out_is_f32) ? 4 : 8;
  const long threads = a.rows * merge_lanes_per_row(a.D / vec);
  const unsigned blocks = (unsigned)((threads + 256 * MERGE_UNITS - 1) / (256 * MERGE_UNITS));
  if (part_is_f32 && out_is_f32) merge_kernel<true, true><<<blocks, 256, 0, s>>>(a);
  else if (part_is_f32) merge_kernel<true, false><<<blocks, 256, 0, s>>>(a);
  else if (out_is_f32) merge_kernel<false, true><<<blocks, 256, 0, s>>>(a);
  else merge_kernel<false, false><<<blocks, 256, 0, s>>>(a);
  return hipGetLastError();
}

template <bool F32>
__global__ void __launch_bounds__(256) delta_kernel(Dims d, const void* o, const void* d_o,
                                                    const float* lse, float* delta, float* stats,
                                                    int sq_pad, float* stats_ovl) {
  row_delta<F32>(d, o, d_o, lse, delta, stats, sq_pad, stats_ovl, ((long)blockIdx.x * 256 + threadIdx.x) / 16, threadIdx.x % 16);
}

hipError_t launch_delta(const Dims& d, const void* o, const void* d_o, int is_f32, const float* lse,
                        float* delta, float* stats, int sq_pad, float* stats_ovl, hipStream_t s) {
  const long rows = (long)d.B * d.Hq * sq_pad;
  const unsigned blocks = (unsigned)((rows * 16 + 255) / 256);
  if (is_f32) delta_kernel<true><<<blocks, 256, 0, s>>>(d, o, d_o, lse, delta, stats, sq_pad, stats_ovl);
  else delta_kernel<false><<<blocks, 256, 0, s>>>(d, o, d_o, lse, delta, stats, sq_pad, stats_ovl);
  return hipGetLastError();
}

// dq_accum += sum of the KV splits' partial dQ (float32, contiguous; where only the last rows of a group were split,
// `run` of its `group` floats).  One thread per 4 elements.
// LAST: the sum is the result, rounded to bf16 with Q's strides.
template <bool FIRST, bool LAST>
__global__ void __launch_bounds__(256) dq_reduce_kernel(Dims d, const float* parts, int n_parts, long n, long run, long group, float* acc,
                                                        uint16_t* dq) {
  const long i = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  const long at = run != group ? i + (i / run + 1) * (group - run) : i;
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
  if (!FIRST) x = *(const f32x4*)(acc + at);
#pragma unroll 4
  for (int k = 0; k < n_parts; ++k) x += *(const f32x4*)(parts + (long)k * n + i);
  if (!LAST) {
    *(f32x4*)(acc + at) = x;
    return;
  }
  const long row = at / d.D;
  const int c = (int)(at % d.D);
  const long ih = row % d.Sq, h = (row / d.Sq) % d.Hq, b = row / ((long)d.Sq * d.Hq);
  unsigned* const dst = (unsigned*)(dq + b * d.q_sb + h * d.q_sh + ih * d.q_ss + c);
  dst[0] = pack_bf16(x[0], x[1]);
  dst[1] = pack_bf16(x[2], x[3]);
}

hipError_t launch_dq_reduce(const Dims& d, const float* parts, int n_parts, long n, long run, long group, float* dq_accum, bool first,
                            void* dq_last, hipStream_t s) {
  const unsigned blocks = (unsigned)((n / 4 + 255) / 256);
  uint16_t* const dq = (uint16_t*)dq_last;
  if (first && dq) dq_reduce_kernel<true, true><<<blocks, 256, 0, s>>>(d, parts, n_parts, n, run, group, dq_accum, dq);
  else if (first) dq_reduce_kernel<true, false><<<blocks, 256, 0, s>>>(d, parts, n_parts, n, run, group, dq_accum, dq);
  else if (dq) dq_reduce_kernel<false, true><<<blocks, 256, 0, s>>>(d, parts, n_parts, n, run, group, dq_accum, dq);
  else dq_reduce_kernel<false, false><<<blocks, 256, 0, s>>>(d, parts, n_parts, n, run, group, dq_accum, dq);
  return hipGetLastError();
}

// dq (input dtype, Q's strides) = dq_accum (float32, contiguous).  One thread per 8 elements.
template <bool F32>
__global__ void __launch_bounds__(256) dq_finalize_kernel(Dims d, const float* acc, void* dq) {
  const int vpr = d.D / 8;
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  const long row = t / vpr;
  if (row >= (long)d.B * d.Hq * d.Sq) return;
  const int c = (int)(t % vpr) * 8;
  const long i = row % d.Sq, h = (row / d.Sq) % d.Hq, b = row / ((long)d.Sq * d.Hq);
  const long off = b * d.q_sb + h * d.q_sh + i * d.q_ss + c;
  const f32x4 x0 = *(const f32x4*)(acc + row * d.D + c), x1 = *(const f32x4*)(acc + row * d.D + c + 4);
  if (F32) {
    *(f32x4*)((float*)dq + off) = x0;
    *(f32x4*)((float*)dq + off + 4) = x1;
  } else {
    u32x4 y = {pack_bf16(x0[0], x0[1]), pack_bf16(x0[2], x0[3]), pack_bf16(x1[0], x1[1]),
               pack_bf16(x1[2], x1[3])};
    *(u32x4*)((uint16_t*)dq + off) = y;
  }
}

hipError_t launch_dq_finalize(const Dims& d, const float* dq_accum, void* dq, int is_f32,
                              hipStream_t s) {
  const long threads = (long)d.B * d.Hq * d.Sq * (d.D / 8);
  const unsigned blocks = (unsigned)((threads + 255) / 256);
  if (is_f32) dq_finalize_kernel<true><<<blocks, 256, 0, s>>>(d, dq_accum, dq);
  else dq_finalize_kernel<false><<<blocks, 256, 0, s>>>(d, dq_accum, dq);
  return hipGetLastError();
}

}  // namespace lvx

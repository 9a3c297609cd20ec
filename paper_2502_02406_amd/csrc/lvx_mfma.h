// Device helpers shared by the bf16 MFMA kernels (gfx950 only).
//
// Register layouts of v_mfma_f32_32x32x16_bf16 (wave64), lane l, g = l / 32:
//   A (32 x 16): row m = l % 32, k = 8 g + e, e = 0..7   (8 bf16 per lane)
//   B (16 x 32): col n = l % 32, k = 8 g + e
//   C (32 x 32): col n = l % 32, row m = 8 (v / 4) + 4 g + (v % 4), v = 0..15
// All kernels compute TRANSPOSED score tiles S^T = K Q^T, so that a lane holds one query column
// and 16 key rows per 32x32 block: the softmax statistics of a query are per-lane scalars, and
// the C registers, converted to bf16, already ARE the B operand of the next product over keys
// (k index = key), with key order  key = 16 t + 8 (e / 4) + 4 g + (e % 4)  for k-step t, slot e.
// The matching A operand (V^T or K^T) is fetched with the transposing LDS read, two per operand.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lvx {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

#define LVX_LDS(ptr, type) ((type __attribute__((address_space(3)))*)(ptr))

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

// Transposing LDS read.  Within each group of 16 lanes, lane j supplies the address of 4
// consecutive bf16; lane i receives element i of the 4 quads supplied by lanes 4r..4r+3 taken as
// row r, i.e. result[r] = row_r[i].  With lanes 4r..4r+3 pointing at 16 consecutive columns of
// row k0 + r of a row-major tile, lane i gets the column (k0..k0+3, n0 + i).
__device__ __forceinline__ s16x4 lds_read_tr(const void* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(uintptr_t)(p));
}

// A operand (32 rows n x 16 k) of a product over k taken from a ROW-MAJOR LDS tile X[k][n]
// (pitch in bytes): rows n0 + l%32, k slots e -> k = kbase + 8 (e / 4) + 4 g + (e % 4).
__device__ __forceinline__ bf16x8 load_tr_operand(const char* tile, int pitch_b, int kbase, int n0,
                                                  int lane) {
  const int j = lane & 15, half = (lane >> 4) & 1, g = lane >> 5;
  const char* p = tile + (kbase + 4 * g + (j >> 2)) * pitch_b + (n0 + 16 * half + 4 * (j & 3)) * 2;
  s16x4 lo = lds_read_tr(p);
  s16x4 hi = lds_read_tr(p + 8 * pitch_b);
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// Row-interleaved tile: up to 64 logical rows of D bf16 at pitch (D + 8) * 2 bytes, logical row r
// stored in physical row (r % 4) * 20 + r / 4.  With D = 128 (pitch 272 = 16 mod 256) BOTH access
// patterns of a tile are free of LDS bank conflicts and need no address arithmetic beyond an
// immediate offset: b128 reads of one 16-byte column by 16 consecutive logical rows land in 16
// distinct 16-byte bank groups, and a transposing read of 4 consecutive logical rows x 64 bytes
// lands in four disjoint 64-byte groups (20 * 272 = 64 mod 256).
constexpr int ILV_ROWS = 80;                       // physical rows of a 64-row interleaved tile
__device__ __forceinline__ int ilv_row(int r) { return (r & 3) * 20 + (r >> 2); }
// Byte offset of logical row (rc + rl), column col: rc is a compile-time multiple of 4 (so that it
// becomes an immediate offset), rl the lane-dependent part.
template <int D> __device__ __forceinline__ int ilv_off(int rl, int rc, int col) {
  return ilv_row(rl) * ((D + 8) * 2) + (rc >> 2) * ((D + 8) * 2) + col * 2;
}
// A operand via transposing reads from an interleaved tile (same contract as load_tr_operand;
// kbase is the first logical row, a multiple of 16).
template <int D>
__device__ __forceinline__ bf16x8 load_tr_operand_ilv(const char* tile, int kbase, int n0, int lane) {
  const int j = lane & 15, half = (lane >> 4) & 1, g = lane >> 5;
  const char* p = tile + ilv_off<D>(4 * g + (j >> 2), 0, 16 * half + 4 * (j & 3));   // lane part
  s16x4 lo = lds_read_tr(p + ilv_off<D>(0, kbase, n0));
  s16x4 hi = lds_read_tr(p + ilv_off<D>(0, kbase + 8, n0));
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// Direct global -> LDS copy of 16 bytes per lane (no staging registers): lane l's 16 bytes land at
// lds_dst + 16 l, where lds_dst must be wave-uniform.  Completion is tracked by vmcnt; the
// compiler does not order later LDS reads against it, so callers wait with wait_vmcnt<N>() and
// then cross a barrier before reading.
__device__ __forceinline__ void dma16(const void* gsrc, void* lds_dst) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)gsrc,
                                   (void __attribute__((address_space(3)))*)lds_dst, 16, 0, 0);
}
// The same copy written out as an instruction, with a wave-uniform 64-bit base and a 32-bit byte
// offset per lane (dma4s: 4 bytes per lane, landing at lds_dst + 4 l).  The compiler does not see
// a memory instruction here: it neither counts the copy in vmcnt nor lets it force the waits of
// unrelated LDS reads to zero, which it does for the builtin above while any copy is in flight.
// The caller orders everything by hand: wait_vmcnt<N>() + barrier before the data is read, a
// barrier before a stage is overwritten.  m0 (declared clobbered) carries the LDS address; one wait
// state separates its write from the copy.
__device__ __forceinline__ unsigned lds_addr_uniform(void* p) {
  // wave-uniform LDS byte address in a scalar register (a no-op when the compiler already keeps it there)
  return (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)LVX_LDS(p, char));
}
__device__ __forceinline__ const void* ptr_uniform(const void* p) {
  // wave-uniform pointer in scalar registers (a no-op when the compiler already keeps it there)
  const unsigned long long x = (unsigned long long)(uintptr_t)p;
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(x >> 32));
  return (const void*)(uintptr_t)(((unsigned long long)hi << 32) | lo);
}
// (the forms that take an LDS byte address save the null test that a cast from a generic pointer
// carries -- two scalar instructions per copy, which a kernel with one wave per SIMD pays for in
// issue slots; lds_base gives the address of the dynamic LDS array once per kernel)
__device__ __forceinline__ unsigned lds_base(void* smem) { return lds_addr_uniform(smem); }
__device__ __forceinline__ void dma16u(const void* base, unsigned voff, unsigned lds_addr) {
  base = ptr_uniform(base);
  const unsigned l = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_addr);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(base), "s"(l) : "memory", "m0");
}
__device__ __forceinline__ void dma4u(const void* base, unsigned voff, unsigned lds_addr) {
  base = ptr_uniform(base);
  const unsigned l = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_addr);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :: "v"(voff), "s"(base), "s"(l) : "memory", "m0");
}
__device__ __forceinline__ void dma16s(const void* base, unsigned voff, void* lds_dst) {
  base = ptr_uniform(base);
  const unsigned l = lds_addr_uniform(lds_dst);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(base), "s"(l) : "memory", "m0");
}
__device__ __forceinline__ void dma4s(const void* base, unsigned voff, void* lds_dst) {
  base = ptr_uniform(base);
  const unsigned l = lds_addr_uniform(lds_dst);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
               :: "v"(voff), "s"(base), "s"(l) : "memory", "m0");
}
// s_waitcnt vmcnt(N) only (expcnt and lgkmcnt left at "no wait").
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// Workgroup barrier without the memory fences of __syncthreads (which would drain vmcnt and so
// serialise the DMA pipeline).  LDS traffic of the calling wave must already be waited for.
__device__ __forceinline__ void wg_barrier() { __builtin_amdgcn_s_barrier(); }

// Two floats -> packed bf16 (round to nearest even), low half = a.
__device__ __forceinline__ unsigned pack2_bf16(float a, float b) {
  bf16x2 r;
  r[0] = (__bf16)a;
  r[1] = (__bf16)b;
  return __builtin_bit_cast(unsigned, r);
}

// 8 consecutive C registers (v0..v0+7) of one 32x32 block -> B operand of the next product.
__device__ __forceinline__ bf16x8 cvt_operand(const f32x16& c, int v0) {
  u32x4 r = {pack2_bf16(c[v0], c[v0 + 1]), pack2_bf16(c[v0 + 2], c[v0 + 3]),
             pack2_bf16(c[v0 + 4], c[v0 + 5]), pack2_bf16(c[v0 + 6], c[v0 + 7])};
  return __builtin_bit_cast(bf16x8, r);
}

// max / sum across the two half-waves (lanes l and l ^ 32 hold the same query column).
__device__ __forceinline__ float xhalf_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Media-mask classification of the rectangle query rows [i0, i1] x key rows [j0, j1]:
// 0 = nothing visible, 1 = everything visible, 2 = mixed.  Wave-uniform arguments.
__device__ __forceinline__ int mask_rect(const MaskWin& m, int b, int i0, int i1, int j0, int j1) {
  if (!m.allow) return 1;
  const long at = b * m.stride_b - m.first;
  bool any = false, all = true;
  for (int c = i0 / m.q_chunk; c <= i1 / m.q_chunk; ++c)
    for (int f = j0 / m.kv_block; f <= j1 / m.kv_block; ++f) {
      const bool on = m.allow[at + (long)c * m.stride_q + f] != 0;
      any |= on;
      all &= on;
    }
  return all ? 1 : (any ? 2 : 0);
}

// mask_rect for rectangles that may span many chunks (planning: a workgroup's rows against one key
// tile, a different tile in every lane; the loops: a wave's rows when chunks are a few rows): the
// same probes and the same answer, the bitmap's rows taken eight at a time so that their round
// trips overlap when the bitmap is in global memory (the rows past the last chunk repeat the last
// one).
__device__ inline int mask_rect_tall(const MaskWin& m, int b, int i0, int i1, int j0, int j1) {
  if (!m.allow) return 1;
  const long at = b * m.stride_b - m.first;
  const int ca = i0 / m.q_chunk, cb = i1 / m.q_chunk;
  if (cb - ca < 4) return mask_rect(m, b, i0, i1, j0, j1);
  unsigned any = 0, all = 1;
  for (int f = j0 / m.kv_block; f <= j1 / m.kv_block; ++f)
    for (int c = ca; c <= cb; c += 8) {
      uint8_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = m.allow[at + (long)min(c + u, cb) * m.stride_q + f];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        any |= v[u];
        all &= v[u] != 0 ? 1u : 0u;
      }
    }
  return all ? 1 : (any ? 2 : 0);
}

__device__ __forceinline__ bool mask_elem(const MaskWin& m, int b, int i, int j) {
  return m.allow[b * m.stride_b - m.first + (long)(i / m.q_chunk) * m.stride_q + j / m.kv_block] != 0;
}

// ---- media mask, staged for a workgroup -----------------------------------------------------
// Reading the bitmap from global memory costs a round trip per probe, and a workgroup probes it
// once per tile or step.  Two helpers take that off the critical path (every thread of the
// workgroup, nthreads of them, must call them; both end with a barrier):
//  * mask_to_lds copies the window [c0, c1] x [f0, f1] of batch b's bitmap into LDS when it fits
//    in `cap` bytes and returns the copy (mask_rect / mask_elem work
//    unchanged: the pointer is generic); otherwise it returns the mask as it is.
//  * build_bits evaluates pred(i), i in [0, n), with all threads at once and leaves bit i in the
//    word array bits[2 ..] (bits[0] = number of set bits); next_bit then finds the next set bit.
//  * class_of reads a three-way classification back from two such planes: the query-stationary
//    kernels keep one pair per wave, so that inside the loop the class of a (wave, tile) pair is
//    two LDS words away and only mixed tiles ever touch the bitmap.
__device__ inline MaskWin mask_to_lds(const MaskDev& m, int b, int c0, int c1, int f0, int f1,
                                      uint8_t* lds, int cap, int tid, int nthreads) {
  MaskWin r = {m, 0};
  if (!m.allow) return r;
  const int w = f1 - f0 + 1, h = c1 - c0 + 1;
  if (w <= 0 || h <= 0 || (long)w * h > cap) return r;               // workgroup-uniform
  for (int i = tid; i < w * h; i += nthreads)
    lds[i] = m.allow[b * m.stride_b + (long)(c0 + i / w) * m.stride_q + f0 + i % w];
  __syncthreads();
  // (the copy itself, and where it starts: a pointer that many bytes before it would be formed in LDS's 32-bit
  // addresses, wrap there once the window starts further on than the copy lies, and be no address of LDS as
  // a generic one: a memory fault for 1102 rows in chunks of one against 2640 keys in blocks of 16)
  r.allow = lds;
  r.first = (long)c0 * w + f0;
  r.stride_b = 0;
  r.stride_q = w;
  return r;
}
template <typename Pred>
__device__ inline int build_bits(unsigned* bits, int n, int tid, int nthreads, Pred pred) {
  if (tid == 0) bits[0] = 0;
  __syncthreads();
  for (int base = 0; base < n; base += nthreads) {   // workgroup-uniform trip count
    const int i = base + tid;
    const bool on = i < n && pred(i);
    const unsigned long long m = __ballot(on);
    if ((tid & 63) == 0 && i < n) {
      *(unsigned long long*)(bits + 2 + i / 32) = m;
      atomicAdd(&bits[0], (unsigned)__popcll(m));
    }
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane((int)bits[0]);
}
// Class of item i from two bit planes laid out like build_bits' (words from [2]): bit i of `any`
// = something visible, of `all` = everything visible.
__device__ inline int class_of(const unsigned* any, const unsigned* all, int i) {   // wave-uniform i
  const unsigned a = (unsigned)__builtin_amdgcn_readfirstlane((int)any[2 + (i >> 5)]) >> (i & 31);
  const unsigned l = (unsigned)__builtin_amdgcn_readfirstlane((int)all[2 + (i >> 5)]) >> (i & 31);
  return (l & 1) ? 1 : ((a & 1) ? 2 : 0);
}
constexpr __host__ __device__ int bit_plane_words(int n) { return 2 + ((n + 63) / 64) * 2; }   // words one plane of n bits takes
__device__ inline int next_bit(const unsigned* bits, int i, int n) {    // first set bit >= i, or n
  // (wave-uniform argument and result: the words are read through the vector path, so say so)
  while (i < n) {
    const unsigned w = (unsigned)__builtin_amdgcn_readfirstlane((int)bits[2 + (i >> 5)]) >> (i & 31);
    if (w) return __builtin_amdgcn_readfirstlane(min(n, i + __ffs(w) - 1));
    i = (i | 31) + 1;
  }
  return __builtin_amdgcn_readfirstlane(n);
}

__device__ inline int nth_bit(const unsigned* bits, int k, int n) {     // index of the k-th set bit (k >= 0), or n
  for (int w0 = 0; w0 < n; w0 += 32) {
    unsigned w = (unsigned)__builtin_amdgcn_readfirstlane((int)bits[2 + (w0 >> 5)]);
    const int c = __popc(w);
    if (k < c) {
      for (; k > 0; --k) w &= w - 1;
      return __builtin_amdgcn_readfirstlane(min(n, w0 + __ffs(w) - 1));
    }
    k -= c;
  }
  return __builtin_amdgcn_readfirstlane(n);
}

// dK and dV of more than 48 MB go past the caches: what these hold of K and V, which the dQ kernel reads next, stays in them.  Smaller ones
// stay there themselves, for the gradients of the projections (RecomputeLayer), which read both twice.  Backward of a layer of 256 rows, two
// blocks, through the caches -> past them, by the size of dK and dV of a block, us: 4, 8, 17 MB (8 heads of 64) 208 -> 215, 217 -> 224, 246 -> 249;
// 17, 36, 50, 56, 67, 134 MB (16 of 128) 486 -> 517, 826 -> 875, 929 -> 983, 919 -> 923, 999 -> 991, 1756 -> 1749; 67 and 268 MB (32 / 8 of 128, 4096
// features) 1923 -> 1949 and 6983 -> 6969.  Without projections, 16 heads of 128: 17, 50, 67, 134, 268 MB 58.1 -> 56.5, 85.1 -> 81.7, 101 -> 95, 157 -> 152,
// 295 -> 275; 8 heads x 131072 keys, D = 64, of which every row sees 64 (134 MB): the step 353 -> 322.
constexpr long DKDV_PAST = 48l << 20;
inline bool dkdv_past(int heads, int keys, int width) { return (long)heads * keys * width * 4 > DKDV_PAST; }
// (a kernel is compiled for either, since with both forms in its code the compiler arranged other parts differently: 8 heads x 4096 rows x 131072
// keys, D = 64, chunks of two rows that see a frame of 64 each, the step 328 -> 331 us)
template <bool PAST> __device__ __forceinline__ void store_dkdv(void* to, u32x4 y) {
  if constexpr (PAST) __builtin_nontemporal_store(y, (u32x4*)to);
  else *(u32x4*)to = y;
}

// XCD-aware decode of a 1-D grid.  Workgroup ids are dealt round-robin to the 8 XCDs, each with
// its own L2.  All work items that share a K/V head are placed on one XCD (or, when there are
// fewer heads than XCDs, a head is cut into equal parts) so that one HBM fetch of a K/V tile
// feeds every workgroup that needs it.  Returns false for padding workgroups.
struct HeadWork { int head; int item; };
__host__ __device__ inline int xcd_parts(int n_heads) {   // parts a head is cut into
  int g = n_heads % 8 == 0 ? 8 : (n_heads % 4 == 0 ? 4 : (n_heads % 2 == 0 ? 2 : 1));
  return 8 / g;
}
__host__ __device__ inline long xcd_grid(int n_heads, int items_per_head) {
  const int S = xcd_parts(n_heads);
  const int per_vh = (items_per_head + S - 1) / S;
  const long n_vh = (long)n_heads * S;                    // multiple of 8
  return n_vh * per_vh;
}
// interleave: the parts of a head take its items in turn instead of a run each, for items whose
// work falls or rises along the head (key tiles under a causal mask): with runs, one XCD would get
// the long items of a head and another the short ones.
__host__ __device__ __forceinline__ bool xcd_decode(long pid, int n_heads, int items_per_head, HeadWork* w,
                                           bool interleave = false) {
  const int S = xcd_parts(n_heads);
  const int per_vh = (items_per_head + S - 1) / S;
  const int xcd = (int)(pid % 8);
  const long slot = pid / 8;
  const long vh = (slot / per_vh) * 8 + xcd;
  const int item = interleave ? (int)(slot % per_vh) * S + (int)(vh % S)
                              : (int)(vh % S) * per_vh + (int)(slot % per_vh);
  w->head = (int)(vh / S);
  w->item = item;
  return item < items_per_head;
}
// Items of which the first n_whole of a head are long and the n_parts behind them short, the long ones of all heads first: for workgroups of
// which a compute unit holds two.  Head by head, an XCD with two heads starts parts of the first where whole row tiles of the
// second belong, and these then share compute units two by two.  64-wide forward, one workgroup a compute unit, two head by head, two in
// this order, us: 2 x 16 heads x 2805 rows x 7318 keys 262, 240, 177; 2 x 8 x 5404 x 11643 306, 338, 263; 2 x 32 / 8 x 1153 x 5543 137, 157, 122;
// 44 others the same to 2 % or better.  (One workgroup a compute unit, 96- and 128-wide: from 26 % less to 6 % more.)
__host__ __device__ inline long tail_grid(int n_heads, int n_whole, int n_parts) {
  return xcd_grid(n_heads, n_whole) + xcd_grid(n_heads, n_parts);
}
__host__ __device__ __forceinline__ bool tail_decode(long pid, int n_heads, int n_whole, int n_parts, HeadWork* w) {
  const long first = xcd_grid(n_heads, n_whole);          // (a multiple of 8)
  if (pid < first) return xcd_decode(pid, n_heads, n_whole, w, true);
  const bool on = xcd_decode(pid - first, n_heads, n_parts, w, n_whole > 0);
  w->item += n_whole;
  return on;
}
// Entry of a list of `total` that workgroup pid takes when every XCD (pid mod 8) takes a run of the list, no XCD
// one of more than an entry beyond another's; false: none.  The grid has a multiple of 8 workgroups, total or more.
__host__ __device__ __forceinline__ bool xcd_run(long pid, long total, long* entry) {
  const long x = pid % 8;
  *entry = total * x / 8 + pid / 8;
  return *entry < total * (x + 1) / 8;
}
// The same for the tiles of a matrix product (head = row tile, item = column tile), of which there may be any
// number of rows: where the parts above come out uneven, each XCD takes a run of the list (row tile, column tile)
// instead, so that no XCD has more than one tile beyond another (xcd_run) and the column tiles of a row tile still meet in
// one L2 (but for a row tile that two runs share).  An odd number of row tiles with 4 column tiles left four
// XCDs idle: projection of 17958 tokens x 512 features x 1024 columns 63 -> 36 us, its dx 86 -> 35; 60001 x
// 1024 x 1024 263 -> 125 and 237 -> 126 us.  Even parts stay as they are: there runs gain nothing (131072 x 512 x
// 1024: forward 201 us, in runs 207; dx 168 and 174).
__host__ __device__ inline bool tile_runs(int n_rt, int n_ct) { return n_ct % xcd_parts(n_rt) != 0; }
__host__ __device__ inline long tile_grid(int n_rt, int n_ct) {
  return tile_runs(n_rt, n_ct) ? ((long)n_rt * n_ct + 7) / 8 * 8 : xcd_grid(n_rt, n_ct);
}
__host__ __device__ __forceinline__ bool tile_decode(long pid, int n_rt, int n_ct, HeadWork* w) {
  if (!tile_runs(n_rt, n_ct)) return xcd_decode(pid, n_rt, n_ct, w);
  long tile;
  const bool on = xcd_run(pid, (long)n_rt * n_ct, &tile);
  w->head = (int)(tile / n_ct);
  w->item = (int)(tile % n_ct);
  return on;
}

}  // namespace lvx

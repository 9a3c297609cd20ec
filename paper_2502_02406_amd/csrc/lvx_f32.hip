// float32 forward and backward passes, computed in float32 end to end on the float32 matrix
// instructions (v_mfma_f32_32x32x2_f32 and 16x16x4: float32 products and sums, 64 operations per clock and SIMD,
// twice what the vector ALU's multiply-adds reach and without their operand traffic).
//
// Every wave works on one 32 x 32 (or 32 x 16) block of scores at a time, transposed as in the bf16 kernels: the
// stationary side (query rows; in dK/dV keys) is a lane's column, the streamed side its 16 (or 8)
// registers.  A contraction may run in any order both operands agree on, and the orders are chosen so
// that registers are operands as they are:
//  * over the head dim (S, dP): lane group g takes dims 8 i + 4 g + e in step (i, e), so that a lane's
//    operands are 16-byte reads of its row;
//  * over the streamed rows (P V, dS K, ...): register v of a score block holds row
//    8 (v / 4) + 4 g + v % 4 in lane group g, and IS the B operand of a step whose A operand is that
//    row's element of the lane's column.
// Tiles come from memory as whole rows (a lane that fetches its own row makes the memory pipeline walk 64
// lines per instruction: 8 waves spent 8000 of their 22000 clocks on that) into registers a tile
// ahead, and through an LDS tile of the wave's own, from which rows and columns are read.  The waves of a
// workgroup share the stationary side and deal the streamed tiles out among them; their results meet in
// LDS at the end.  All rows of the query heads that share a K/V head are one list of G Sq rows (as in the
// bf16 kernels), so short query blocks fill tiles.
//
// Bound by the matrix instructions where there is work enough (512 rows x 8 heads x 4096 keys x 128:
// forward 0.20 ms = 43 TFLOP/s on the half of the chip its 128 workgroups occupy, backward 0.49 ms; the
// plain multiply-add kernels before took 3.55 ms for the step, now 0.65), by latency on the smallest: the tiny step's
// launches (128 rows x 2 heads x 256 keys x 64) take 7 us forward and 7.5 backward, a chain of one block's
// products and the trip of its operands; with 32 x 32 blocks they took 9.5 and 11 (see narrow()).
#include "lvx_internal.h"
#include "lvx_mfma.h"

namespace lvx {

namespace {

constexpr int waves_of(int D) { return D == 64 ? 8 : 4; }     // (wider heads need more than half of a SIMD's registers per wave)
constexpr int pitch_of(int D) { return D + 4; }               // floats per row of an LDS tile of 32 rows
constexpr int tile_of(int D) { return 32 * pitch_of(D); }

// R: width of the stationary side, one row a lane.  32: blocks of 32 x 32 in 16 registers; 16: blocks of 16 x 16 in 4.
template <int R> struct Block;
template <> struct Block<32> { typedef f32x16 type; };
template <> struct Block<16> { typedef f32x4 type; };
template <int R> using BlockOf = typename Block<R>::type;
template <int R> constexpr int VR = R * R / 64;                  // registers of a block,
template <int R> constexpr int NG = 64 / R;                      // lane groups: lane l is row l % R in group l / R,
template <int R> constexpr int SUB = 32 / R;                     // blocks over the 32 streamed rows
template <int R> __device__ __forceinline__ BlockOf<R> zero_block() {
  BlockOf<R> c;
#pragma unroll
  for (int v = 0; v < VR<R>; ++v) c[v] = 0.f;
  return c;
}
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// streamed row that register v of block `sub` holds, without the lane group's 4 g
template <int R> __device__ __forceinline__ constexpr int reg_u(int sub, int v) { return R * sub + 8 * (v / 4) + v % 4; }
template <int R> __device__ __forceinline__ float groups_max(float x) {
  x = xhalf_max(x);
  return R == 32 ? x : fmaxf(x, __shfl_xor(x, 16, 64));
}
template <int R> __device__ __forceinline__ float groups_sum(float x) {
  x = xhalf_sum(x);
  return R == 32 ? x : x + __shfl_xor(x, 16, 64);
}
// e^x for x <= 0, -infinity included: 2^h (1 + l ln 2) with h + l = x log2(e), h rounded and l what the
// rounding and the constant's own lost (within 2 ulp like the library's, in half its instructions: a
// launch whose waves pass through their code once is bound by fetching it)
__device__ __forceinline__ float exp_neg(float x) {
  x = x < -200.f ? -200.f : x;                     // (e^-200 is 0 in float32; keeps infinities out of l, and a NaN a NaN)
  const float h = x * 1.44269504f;
  const float l = fmaf(x, 1.925963033e-8f, fmaf(x, 1.44269504f, -h));
  const float e = __builtin_amdgcn_exp2f(h);
  return fmaf(e, l * 0.693147181f, e);
}
__device__ __forceinline__ bool visible(const MaskDev& m, int b, int i, int j) {
  return m.allow[b * m.stride_b + (long)(i / m.q_chunk) * m.stride_q + (j / m.kv_block)] != 0;
}
// A tile of 32 rows on its way from memory to LDS: piece it of a lane is 16 bytes of row
// row_of_piece(it, lane).
template <int D> struct Pieces { f32x4 x[D / 8]; };
template <int D> __device__ __forceinline__ int row_of_piece(int it, int lane) { return (64 * it + lane) / (D / 4); }
template <int D> __device__ __forceinline__ int col_of_piece(int it, int lane) { return (64 * it + lane) % (D / 4) * 4; }
// n rows `stride` apart (rows past them re-read the last one)
template <int D> __device__ __forceinline__ Pieces<D> fetch(const float* first, int n, long stride, int lane) {
  Pieces<D> p;
#pragma unroll
  for (int it = 0; it < D / 8; ++it)
    p.x[it] = *(const f32x4*)(first + (long)min(row_of_piece<D>(it, lane), n - 1) * stride + col_of_piece<D>(it, lane));
  return p;
}
template <int D> __device__ __forceinline__ void put_tile(float* tile, const Pieces<D>& p, int lane) {
#pragma unroll
  for (int it = 0; it < D / 8; ++it) *(f32x4*)(tile + row_of_piece<D>(it, lane) * pitch_of(D) + col_of_piece<D>(it, lane)) = p.x[it];
}
// rows `first` .. 31 of a tile in LDS become 0: those past the last row, where something without a weight would be
// multiplied that need not be finite
template <int D> __device__ __forceinline__ void clear_rows(float* tile, int first, int lane) {
#pragma unroll 1
  for (int x = first * (D / 4) + lane; x < 32 * (D / 4); x += 64)
    *(f32x4*)(tile + x / (D / 4) * pitch_of(D) + x % (D / 4) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
}
// a lane's row of the stationary side, 16 bytes per step group i: dims 4 NG i + 4 g ...
template <int D, int R> struct RowOps { f32x4 x[D / (4 * NG<R>)]; };
template <int D, int R> __device__ __forceinline__ RowOps<D, R> row_ops(const float* tile, int lr, int g) {
  RowOps<D, R> r;
#pragma unroll
  for (int i = 0; i < D / (4 * NG<R>); ++i) r.x[i] = *(const f32x4*)(tile + lr * pitch_of(D) + 4 * NG<R> * i + 4 * g);
  return r;
}
// 32 x R products over the head dim: rows of the tile in registers, stationary rows in lanes.  b(i): the stationary
// row's operands of step group i.  Blocks of 16 x 16 are summed in two chains: their scores are half as
// many steps away from their last addition, and everything that follows from them is nearer to float64 (dK of the tiny
// step 3.6e-7, with one chain 4.8e-7, with 32 x 32 blocks 4.2e-7; dQ where keys are eight times the others' 1.7e-6 and
// 2.9e-6); 1.5 us of 62 a step.
template <int R> struct Scores { BlockOf<R> b[SUB<R>]; };
template <int D, int R, typename B> __device__ __forceinline__ Scores<R> products_of(const float* tile, B&& b, int lr, int g) {
  constexpr int CH = R == 16 ? 2 : 1;
  Scores<R> c[CH];
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u) c[h].b[u] = zero_block<R>();
#pragma unroll
  for (int i = 0; i < D / (4 * NG<R>); ++i) {
    const f32x4 bi = b(i);
    f32x4 a[SUB<R>];
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u) a[u] = *(const f32x4*)(tile + (R * u + lr) * pitch_of(D) + 4 * NG<R> * i + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < SUB<R>; ++u) c[e % CH].b[u] = mfma_f32(a[u][e], bi[e], c[e % CH].b[u]);
  }
#pragma unroll
  for (int h = 1; h < CH; ++h)
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u)
#pragma unroll
      for (int v = 0; v < VR<R>; ++v) c[0].b[u][v] += c[h].b[u][v];
  return c[0];
}
template <int D, int R> __device__ __forceinline__ Scores<R> products(const float* tile, const RowOps<D, R>& b, int lr, int g) {
  return products_of<D, R>(tile, [&](int i) __attribute__((always_inline)) -> f32x4 { return b.x[i]; }, lr, g);
}
// ... with the stationary rows in LDS as well
template <int D, int R> __device__ __forceinline__ Scores<R> products(const float* tile, const float* btile, int lr, int g) {
  return products_of<D, R>(tile, [&](int i) __attribute__((always_inline)) -> f32x4 {
    return *(const f32x4*)(btile + lr * pitch_of(D) + 4 * NG<R> * i + 4 * g);
  }, lr, g);
}
// acc += (tile's columns, 32 rows) x b
template <int D, int R>
__device__ __forceinline__ void contract(BlockOf<R> (&acc)[D / R], const float* tile, const Scores<R>& b, int lr, int g) {
#pragma unroll
  for (int u = 0; u < SUB<R>; ++u)
#pragma unroll
    for (int v = 0; v < VR<R>; ++v)
#pragma unroll
      for (int db = 0; db < D / R; ++db)
        acc[db] = mfma_f32(tile[(reg_u<R>(u, v) + 4 * g) * pitch_of(D) + R * db + lr], b.b[u][v], acc[db]);
}
// the (transposed) result block of a wave -> its part of the combine buffer: row lr, columns of D
template <int D, int R> __device__ __forceinline__ void put_block(float* buf, const BlockOf<R> (&acc)[D / R], int lr, int g) {
#pragma unroll
  for (int db = 0; db < D / R; ++db)
#pragma unroll
    for (int q4 = 0; q4 < VR<R> / 4; ++q4) {
      const f32x4 y = {acc[db][4 * q4], acc[db][4 * q4 + 1], acc[db][4 * q4 + 2], acc[db][4 * q4 + 3]};
      *(f32x4*)(buf + lr * pitch_of(D) + R * db + 8 * q4 + 4 * g) = y;
    }
}
// Where the rows of the group's list lie: row r is row r % Sq of head r / Sq of the group.
struct Rows {
  const Dims& d;
  long base;                                       // first element of the group's first head (batch and head offset)
  float inv_sq;
  __device__ __forceinline__ Rows(const Dims& d_, int b, int hk)
      : d(d_), base(b * d_.q_sb + (long)(hk * d_.G) * d_.q_sh), inv_sq(1.f / (float)d_.Sq) {}
  struct At { long off; int i; };                  // element offset of the row, its number in its head
  // (r / Sq in float is off by less than one, the heads of a group being fewer than 2^23)
  __device__ __forceinline__ At operator()(int r) const {
    int h = (int)((float)r * inv_sq), i = r - h * d.Sq;
    if (i < 0) { --h; i += d.Sq; }
    if (i >= d.Sq) { ++h; i -= d.Sq; }
    return {base + (long)h * d.q_sh + (long)i * d.q_ss, i};
  }
};

// Forward: a workgroup's R rows against all keys; its waves take the tiles of 32 keys in turn.
template <int D, int R, bool MASKED>
__global__ void __launch_bounds__(64 * waves_of(D)) fwd_f32_kernel(FwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int NW = waves_of(D), DB = D / R, P = pitch_of(D), T = tile_of(D);
  const Dims& d = a.d;
  const int rows = d.G * d.Sq, b = blockIdx.z, hk = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, g = lane / R, ql = lane % R;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = blockIdx.x * R;
  float* const lds = (float*)smem;
  float* const kt = lds + wave * 2 * T;            // this wave's tiles of K and V
  float* const vt = kt + T;
  const Rows at(d, b, hk);
  const float* const k = (const float*)a.k + b * d.kv_sb + hk * d.kv_sh;
  const float* const v = (const float*)a.v + b * d.kv_sb + hk * d.kv_sh;
  Pieces<D> kp, vp;
  auto request = [&](int j0) __attribute__((always_inline)) {
    kp = fetch<D>(k + (long)j0 * d.kv_ss, d.Skv - j0, d.kv_ss, lane);
    vp = fetch<D>(v + (long)j0 * d.kv_ss, d.Skv - j0, d.kv_ss, lane);
  };
  // Q: wave w brings its share of the tile's pieces, every wave reads all rows' operands
#pragma unroll
  for (int x = tid; x < R * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), c = x % (D / 4) * 4;
    *(f32x4*)(lds + r * P + c) = *(const f32x4*)((const float*)a.q + at(min(r0 + r, rows - 1)).off + c);
  }
  if (32 * wave < d.Skv) request(32 * wave);
  __syncthreads();
  const RowOps<D, R> q = row_ops<D, R>(lds, ql, g);
  __syncthreads();

  BlockOf<R> acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = zero_block<R>();
  float m = -INFINITY, l = 0.f;                    // (l: this lane's share)
  const int i_lane = MASKED ? at(min(r0 + ql, rows - 1)).i : 0;
  for (int j0 = 32 * wave; j0 < d.Skv; j0 += 32 * NW) {
    const int n = d.Skv - j0;
    put_tile<D>(kt, kp, lane);
    put_tile<D>(vt, vp, lane);
    if (n < 32) clear_rows<D>(vt, n, lane);
    if (n > 32 * NW) request(j0 + 32 * NW);
    Scores<R> s = products<D, R>(kt, q, ql, g);
    if (MASKED || n < 32) {
#pragma unroll
      for (int x = 0; x < R / 2; ++x) {
        const int j = reg_u<R>(x / VR<R>, x % VR<R>) + 4 * g;
        if (j >= n || (MASKED && !visible(a.mask, b, i_lane, j0 + min(j, n - 1)))) s.b[x / VR<R>][x % VR<R>] = -INFINITY;
      }
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u)
#pragma unroll
      for (int x = 0; x < VR<R>; ++x) { s.b[u][x] *= d.scale; tmax = fmaxf(tmax, s.b[u][x]); }
    const float m_new = fmaxf(m, groups_max<R>(tmax));
    if (m_new != m) {                              // (some lane's row has risen: l and O^T follow)
      const float alpha = exp_neg(m - m_new);      // m = -inf -> 0
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int x = 0; x < VR<R>; ++x) acc[db][x] *= alpha;
    }
    const float m_ref = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u)
#pragma unroll
      for (int x = 0; x < VR<R>; ++x) {
        s.b[u][x] = exp_neg(s.b[u][x] - m_ref);
        l += s.b[u][x];
      }
    contract<D, R>(acc, vt, s, ql, g);
  }

  // ---- the waves' results meet: every wave's O in its K tile, references and sums behind all tiles
  float* const st_m = lds + NW * 2 * T;            // [wave][R] references, sums; the rows' new L
  float* const st_l = st_m + NW * R;
  float* const l_next = st_l + NW * R;
  const float l_row = groups_sum<R>(l);
  if (g == 0) { st_m[wave * R + ql] = m; st_l[wave * R + ql] = l_row; }
  if (MASKED && __any(l_row == 0.f)) {             // (a row that saw no key of this wave's has weight 0: so must be what it holds)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int x = 0; x < VR<R>; ++x) acc[db][x] = l_row == 0.f ? 0.f : acc[db][x];
  }
  put_block<D, R>(kt, acc, ql, g);
  __syncthreads();
  const long row_b = ((long)b * d.Hq + hk * d.G) * d.Sq;       // L rows of the group follow each other
#pragma unroll 1
  for (int x = tid; x < R * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), c = x % (D / 4) * 4, rr = min(r0 + r, rows - 1);
    float* const o = (float*)a.o + (a.merge_into ? (row_b + rr) * D : at(rr).off) + c;
    f32x4 old = {0.f, 0.f, 0.f, 0.f};
    float L0 = -INFINITY;
    if (a.merge_into) {                            // Rescale with the running (O, L)
      old = *(const f32x4*)o;
      L0 = a.lse[row_b + rr];
    }
    float M = L0;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, st_m[w * R + r]);
    const float Mz = M == -INFINITY ? 0.f : M;
    float z = exp_neg(L0 - Mz);
    f32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = z * old[e];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = exp_neg(st_m[w * R + r] - Mz);          // (a wave without a key: 0)
      const f32x4 ow = *(const f32x4*)(lds + w * 2 * T + r * P + c);
      z += f * st_l[w * R + r];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] += f * ow[e];
    }
    const float inv = z > 0.f ? 1.f / z : 0.f, lse = z != 0.f ? M + logf(z) : -INFINITY;    // (NaN scores: NaN, which no combine drops)
    if (r0 + r >= rows) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] *= inv;
    *(f32x4*)o = y;
    if (c == 0) {
      if (a.merge_into) l_next[r] = lse;
      else a.lse[row_b + rr] = lse;
    }
  }
  if (a.merge_into) {                              // L is replaced once every thread has read it
    __syncthreads();
    if (tid < R && r0 + tid < rows) a.lse[row_b + r0 + tid] = l_next[tid];
  }
}

// Backward, dQ: a workgroup's R query rows against all keys.
template <int D, int R, bool MASKED>
__device__ void bwd_dq_f32(const BwdArgs& a, int tile, int hk, int b, char* smem) {
  constexpr int NW = waves_of(D), DB = D / R, P = pitch_of(D), T = tile_of(D);
  const Dims& d = a.d;
  const int rows = d.G * d.Sq;
  const int tid = threadIdx.x, lane = tid & 63, g = lane / R, ql = lane % R;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r0 = tile * R, rl = min(r0 + ql, rows - 1);
  float* const lds = (float*)smem;
  float* const kt = lds + wave * 2 * T;
  float* const vt = kt + T;
  const Rows at(d, b, hk);
  const long row_b = ((long)b * d.Hq + hk * d.G) * d.Sq;
  const float* const k = (const float*)a.k + b * d.kv_sb + hk * d.kv_sh;
  const float* const v = (const float*)a.v + b * d.kv_sb + hk * d.kv_sh;
  Pieces<D> kp, vp;
  auto request = [&](int j0) __attribute__((always_inline)) {
    kp = fetch<D>(k + (long)j0 * d.kv_ss, d.Skv - j0, d.kv_ss, lane);
    vp = fetch<D>(v + (long)j0 * d.kv_ss, d.Skv - j0, d.kv_ss, lane);
  };
  const float L = a.lse[row_b + rl], delta = a.delta[row_b + rl];
  const float nl = L == -INFINITY ? -INFINITY : -L;            // (a row without keys: every exponent -inf)
#pragma unroll
  for (int x = tid; x < R * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), c = x % (D / 4) * 4;
    const long off = at(min(r0 + r, rows - 1)).off + c;
    *(f32x4*)(lds + r * P + c) = *(const f32x4*)((const float*)a.q + off);
    *(f32x4*)(lds + T + r * P + c) = *(const f32x4*)((const float*)a.d_o + off);
  }
  if (32 * wave < d.Skv) request(32 * wave);
  __syncthreads();
  const RowOps<D, R> q = row_ops<D, R>(lds, ql, g), go = row_ops<D, R>(lds + T, ql, g);
  __syncthreads();
  const int i_lane = MASKED ? at(rl).i : 0;
  BlockOf<R> acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = zero_block<R>();
  for (int j0 = 32 * wave; j0 < d.Skv; j0 += 32 * NW) {
    const int n = d.Skv - j0;
    put_tile<D>(kt, kp, lane);
    put_tile<D>(vt, vp, lane);
    if (n > 32 * NW) request(j0 + 32 * NW);
    Scores<R> s = products<D, R>(kt, q, ql, g);
    const Scores<R> dp = products<D, R>(vt, go, ql, g);
    if (MASKED || n < 32) {
#pragma unroll
      for (int x = 0; x < R / 2; ++x) {
        const int j = reg_u<R>(x / VR<R>, x % VR<R>) + 4 * g;
        if (j >= n || (MASKED && !visible(a.mask, b, i_lane, j0 + min(j, n - 1)))) s.b[x / VR<R>][x % VR<R>] = -INFINITY;
      }
    }
#pragma unroll
    for (int u = 0; u < SUB<R>; ++u)
#pragma unroll
      for (int x = 0; x < VR<R>; ++x) {            // (a pair that does not count adds 0, whatever its dP)
        const float t = fmaf(s.b[u][x], d.scale, nl);
        s.b[u][x] = t == -INFINITY ? 0.f : exp_neg(t) * (dp.b[u][x] - delta);
      }
    contract<D, R>(acc, kt, s, ql, g);
  }
  put_block<D, R>(kt, acc, ql, g);
  __syncthreads();
#pragma unroll 1
  for (int x = tid; x < R * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), c = x % (D / 4) * 4;
    if (r0 + r >= rows) continue;
    float* const o = a.dq_accum + (row_b + r0 + r) * D + c;    // (rows are owned by one workgroup)
    f32x4 old = {0.f, 0.f, 0.f, 0.f};
    if (!a.dq_first) old = *(const f32x4*)o;
    f32x4 y = *(const f32x4*)(lds + r * P + c);
#pragma unroll
    for (int w = 1; w < NW; ++w) y += *(const f32x4*)(lds + w * 2 * T + r * P + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) old[e] += y[e] * d.scale;
    *(f32x4*)o = old;
  }
}

// Backward, dK and dV: a workgroup's R keys against the query rows of the whole group of heads.
template <int D, int R, bool MASKED>
__device__ void bwd_dkdv_f32(const BwdArgs& a, int tile, int hk, int b, char* smem) {
  constexpr int NW = waves_of(D), DB = D / R, P = pitch_of(D), T = tile_of(D);
  const Dims& d = a.d;
  const int rows = d.G * d.Sq;
  const int tid = threadIdx.x, lane = tid & 63, g = lane / R, kl = lane % R;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = tile * R, jc = min(j0 + kl, d.Skv - 1);
  float* const lds = (float*)smem;
  float* const qt = lds + wave * 2 * T;            // this wave's tiles of Q and dO
  float* const gt = qt + T;
  float* const v_t = lds + NW * 2 * T;             // V of the workgroup's keys stays in LDS (dK and dV fill the registers)
  float* const st = v_t + T + wave * 64;           // this wave's rows' -L (-inf: no probability), then delta
  const long row_b = ((long)b * d.Hq + hk * d.G) * d.Sq, kv_h = b * d.kv_sb + hk * d.kv_sh;
  const Rows at(d, b, hk);
  Pieces<D> qp, gp;
  float sp;
  auto request = [&](int r0) __attribute__((always_inline)) {
    if (r0 + 32 <= rows && r0 / d.Sq == (r0 + 31) / d.Sq) {    // whole, and in one head: as a rule
      const long off = at(r0).off;
      qp = fetch<D>((const float*)a.q + off, 32, d.q_ss, lane);
      gp = fetch<D>((const float*)a.d_o + off, 32, d.q_ss, lane);
    } else {
#pragma unroll 1
      for (int it = 0; it < D / 8; ++it) {         // (through this wave's LDS tiles, which are free by now: see the callers)
        const int r = row_of_piece<D>(it, lane), c = col_of_piece<D>(it, lane);
        const long off = at(min(r0 + r, rows - 1)).off + c;
        *(f32x4*)(qt + r * P + c) = *(const f32x4*)((const float*)a.q + off);
        *(f32x4*)(gt + r * P + c) = *(const f32x4*)((const float*)a.d_o + off);
      }
#pragma unroll
      for (int it = 0; it < D / 8; ++it) {
        const int r = row_of_piece<D>(it, lane), c = col_of_piece<D>(it, lane);
        qp.x[it] = *(const f32x4*)(qt + r * P + c);
        gp.x[it] = *(const f32x4*)(gt + r * P + c);
      }
    }
    // (32 streamed rows: -L from the first half of the lanes, delta from the other)
    const int l31 = lane & 31, rr = min(r0 + l31, rows - 1);
    const float x = lane < 32 ? a.lse[row_b + rr] : a.delta[row_b + rr];
    const bool past = r0 + l31 >= rows;
    sp = lane < 32 ? (x == -INFINITY || past ? -INFINITY : -x) : past ? 0.f : x;
  };
#pragma unroll
  for (int x = tid; x < R * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), c = x % (D / 4) * 4;
    const long off = kv_h + (long)min(j0 + r, d.Skv - 1) * d.kv_ss + c;
    *(f32x4*)(lds + r * P + c) = *(const f32x4*)((const float*)a.k + off);
    *(f32x4*)(v_t + r * P + c) = *(const f32x4*)((const float*)a.v + off);
  }
  __syncthreads();
  const RowOps<D, R> k = row_ops<D, R>(lds, kl, g);
  __syncthreads();
  BlockOf<R> dk[DB], dv[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) { dk[db] = zero_block<R>(); dv[db] = zero_block<R>(); }
  if (32 * wave < rows) request(32 * wave);
  for (int r0 = 32 * wave; r0 < rows; r0 += 32 * NW) {
    put_tile<D>(qt, qp, lane);
    put_tile<D>(gt, gp, lane);
    if (rows - r0 < 32) clear_rows<D>(gt, rows - r0, lane);
    st[lane] = sp;
    const int rn = r0 + 32 * NW;
    const bool more = rn < rows, plain = rn + 32 <= rows && rn / d.Sq == (rn + 31) / d.Sq;
    if (more && plain) request(rn);
    Scores<R> p = products<D, R>(qt, k, kl, g), ds = products<D, R>(gt, v_t, kl, g);       // (S and dP, then P and dS)
#pragma unroll
    for (int x4 = 0; x4 < R / 8; ++x4) {           // four registers each: rows of one 16-byte read of the statistics
      const int u = 4 * x4 / VR<R>, v0 = 4 * x4 % VR<R>, row = reg_u<R>(u, v0) + 4 * g;
      const f32x4 nl = *(const f32x4*)(st + row), de = *(const f32x4*)(st + 32 + row);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = v0 + e;
        float t = fmaf(p.b[u][v], d.scale, nl[e]);
        if (MASKED && !visible(a.mask, b, at(min(r0 + row + e, rows - 1)).i, jc)) t = -INFINITY;
        p.b[u][v] = exp_neg(t);
        ds.b[u][v] = p.b[u][v] * (ds.b[u][v] - de[e]);
      }
    }
    contract<D, R>(dv, gt, p, kl, g);
    contract<D, R>(dk, qt, ds, kl, g);
    if (more && !plain) request(rn);               // (row by row, once the tiles have been read)
  }
  put_block<D, R>(qt, dk, kl, g);
  put_block<D, R>(gt, dv, kl, g);
  __syncthreads();
#pragma unroll 1
  for (int x = tid; x < 2 * R * (D / 4); x += 64 * NW) {
    const int which = x / (R * (D / 4)), r = x / (D / 4) % R, c = x % (D / 4) * 4;
    if (j0 + r >= d.Skv) continue;
    f32x4 y = *(const f32x4*)(lds + which * T + r * P + c);
#pragma unroll
    for (int w = 1; w < NW; ++w) y += *(const f32x4*)(lds + (2 * w + which) * T + r * P + c);
    const float f = which == 0 ? d.scale : 1.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] *= f;
    *(f32x4*)((float*)(which == 0 ? a.dk : a.dv) + kv_h + (long)(j0 + r) * d.kv_ss + c) = y;
  }
}

// Both parts in one launch (they share nothing and neither fills the card on small problems): the first
// n_q workgroups of a K/V head form dQ, the others dK and dV.
template <int D, int RQ, int RK, bool MASKED>
__global__ void __launch_bounds__(64 * waves_of(D)) bwd_f32_kernel(BwdArgs a, int n_q) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if ((int)blockIdx.x < n_q) bwd_dq_f32<D, RQ, MASKED>(a, blockIdx.x, blockIdx.y, blockIdx.z, smem);
  else bwd_dkdv_f32<D, RK, MASKED>(a, blockIdx.x - n_q, blockIdx.y, blockIdx.z, smem);
}

template <int D, int R, bool MASKED> hipError_t launch_fwd(const FwdArgs& a, hipStream_t s) {
  static SmemOnce once;
  constexpr int lds = (waves_of(D) * (2 * tile_of(D) + 64) + 32) * 4;
  static_assert(lds <= 160 * 1024, "the tiles fit a compute unit");
  const hipError_t e = ensure_dynamic_lds((const void*)fwd_f32_kernel<D, R, MASKED>, lds, &once);
  if (e != hipSuccess) return e;
  const dim3 grid((a.d.G * a.d.Sq + R - 1) / R, a.d.Hkv, a.d.B);
  fwd_f32_kernel<D, R, MASKED><<<grid, 64 * waves_of(D), lds, s>>>(a);
  return hipGetLastError();
}
template <int D, int RQ, int RK, bool MASKED> hipError_t launch_bwd(const BwdArgs& a, unsigned stages, hipStream_t s) {
  static SmemOnce once;
  constexpr int lds = (waves_of(D) * (2 * tile_of(D) + 64) + tile_of(D)) * 4;
  static_assert(lds <= 160 * 1024, "the tiles fit a compute unit");
  const hipError_t e = ensure_dynamic_lds((const void*)bwd_f32_kernel<D, RQ, RK, MASKED>, lds, &once);
  if (e != hipSuccess) return e;
  const int n_q = stages & 4 ? (a.d.G * a.d.Sq + RQ - 1) / RQ : 0, n_k = stages & 2 ? (a.d.Skv + RK - 1) / RK : 0;
  bwd_f32_kernel<D, RQ, RK, MASKED><<<dim3(n_q + n_k, a.d.Hkv, a.d.B), 64 * waves_of(D), lds, s>>>(a, n_q);
  return hipGetLastError();
}
// The stationary side is 16 rows wide instead of 32 while the workgroups of 32 rows are no more than the compute units:
// up to twice the workgroups, each with half the matrix instructions in its chain, against a streamed side that is read
// twice as often.  dQ is judged by itself: its workgroups are few and long where those of dK and dV are many.
// Tiny step (128 rows x 2 heads x 4 blocks of 256 keys x 64) 83 -> 61 us; 512 rows x 2 heads x 4 blocks of 143 keys 135 -> 88;
// 52 rows x 8 heads x 4 blocks of 512 keys x 128 273 -> 189.  With 32 rows in 16-row workgroups throughout: 256 rows x 8 heads x
// 832 keys x 96 76 -> 83 us.
bool narrow(const Dims& d, long rows, int n_cu) { return (long)d.B * d.Hkv * ((rows + 31) / 32) <= n_cu; }
template <int D, bool MASKED> hipError_t fwd_by_rows(const FwdArgs& a, hipStream_t s) {
  return narrow(a.d, (long)a.d.G * a.d.Sq, a.n_cu) ? launch_fwd<D, 16, MASKED>(a, s) : launch_fwd<D, 32, MASKED>(a, s);
}
template <int D, bool MASKED> hipError_t bwd_by_rows(const BwdArgs& a, unsigned stages, hipStream_t s) {
  const long rows = (long)a.d.G * a.d.Sq;
  if (narrow(a.d, rows + 31 + a.d.Skv, a.n_cu)) return launch_bwd<D, 16, 16, MASKED>(a, stages, s);
  return narrow(a.d, rows, a.n_cu) ? launch_bwd<D, 16, 32, MASKED>(a, stages, s) : launch_bwd<D, 32, 32, MASKED>(a, stages, s);
}
template <bool MASKED> hipError_t fwd_by_width(const FwdArgs& a, hipStream_t s) {
  return a.d.D == 64 ? fwd_by_rows<64, MASKED>(a, s) : a.d.D == 96 ? fwd_by_rows<96, MASKED>(a, s) : fwd_by_rows<128, MASKED>(a, s);
}
template <bool MASKED> hipError_t bwd_by_width(const BwdArgs& a, unsigned stages, hipStream_t s) {
  return a.d.D == 64 ? bwd_by_rows<64, MASKED>(a, stages, s)
       : a.d.D == 96 ? bwd_by_rows<96, MASKED>(a, stages, s) : bwd_by_rows<128, MASKED>(a, stages, s);
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t s) {
  return a.mask.allow != nullptr ? fwd_by_width<true>(a, s) : fwd_by_width<false>(a, s);
}

hipError_t launch_bwd_f32(const BwdArgs& a, unsigned stages, hipStream_t s) {
  return a.mask.allow != nullptr ? bwd_by_width<true>(a, stages, s) : bwd_by_width<false>(a, stages, s);
}

}  // namespace lvx

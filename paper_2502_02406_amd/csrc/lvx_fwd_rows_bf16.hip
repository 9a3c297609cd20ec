// bf16 forward kernel for a few query rows (serving: a generated token, or a handful of them, against
// all visual keys): the FlashAttention call of Algorithm 1 where K and V are read once and hardly
// computed on, so that the kernel is a stream from memory.
//
// The G * Sq rows of the query heads that share a K/V head (at most 64) are one or two 32-column
// blocks.  Workgroup = 4 wavefronts on one K/V head's share of the keys; each wavefront streams units of
// 32 keys of its own (every fourth of the workgroup's) through two stages of LDS of its own, so no
// barrier stands in the loop and a wave waits for its own copies only; 128 KB of LDS per compute unit
// (D = 128) are either in flight or being multiplied.  S^T = K Q^T, the online softmax and
// O^T += V^T P^T are those of the other forward kernels (a lane owns a row, P^T stays in registers, V^T
// comes from transposing LDS reads).  The four waves' results are combined in LDS; the workgroups'
// (split-KV) by the merge kernel.
//
// One row x 32 heads on 8 K/V heads of 128: against 262144 keys 218 -> 175 us (1.07 GB at 6.1 TB/s; the
// dense kernel forms 256 rows for the 4 there are and holds 8 tiles in flight), against 6404 keys
// 31 -> 7.3 us (256 workgroups with 25 units of keys each, where the dense kernel's split stops at 48 of
// 16 tiles).  With the combine: 238 -> 181 us and 42.4 -> 12.8 us a call; 64 rows (16 x 4 heads) against 65536 keys
// 86 -> 62 us; 8 batches x 16 heads against 20000 keys 281 -> 222 us.
#include "lvx_internal.h"
#include "lvx_key_units.h"

namespace lvx {

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LAZY = 6.0f;           // raise the reference only when a row tops it by 2^LAZY
constexpr int NWV = 4;                 // waves per workgroup
constexpr int NST = 2;                 // stages per wave

template <int D> struct RowsSmem : KeyUnit<D> {
  static constexpr int WAVE = NST * KeyUnit<D>::STAGE;
  static constexpr int STATS = NWV * WAVE;          // combine: [waves][64 rows] references and sums
  static constexpr int TOTAL = STATS + NWV * 64 * 8;
};

template <int D, int NB>
__global__ void __launch_bounds__(256) fwd_rows_bf16_kernel(FwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using SM = RowsSmem<D>;
  constexpr int KS = D / 16, DB = D / 32, CPR = SM::CPR, CH = SM::CH, NC = SM::NC, NDMA = 2 * NC;
  const Dims& d = a.d;
  const int G = d.Hq / d.Hkv, rows = G * d.Sq;
  const int n_heads = d.B * d.Hkv;
  const int head = (int)(blockIdx.x % n_heads), split = (int)(blockIdx.x / n_heads);
  const int b = head / d.Hkv, hk = head % d.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // this workgroup's units of 32 keys, dealt to its waves in turn
  const int U = (d.Skv + UK - 1) / UK;
  const int u0 = (int)((long)U * split / a.n_split), u1 = (int)((long)U * (split + 1) / a.n_split);
  char* const mine = smem + wave * SM::WAVE;
  const unsigned mine_u = lds_base(mine);
  const char* const k0 = (const char*)a.k + (b * d.kv_sb + hk * d.kv_sh) * 2;
  const char* const v0 = (const char*)a.v + (b * d.kv_sb + hk * d.kv_sh) * 2;
  const unsigned row_bytes = (unsigned)(d.kv_ss * 2);
  auto copy_off = [&](int n, int of_v, int last_row) __attribute__((always_inline)) -> unsigned {
    return unit_copy_off<D>(n, of_v, last_row, row_bytes, lane);
  };
  unsigned offk[NC], offv[NC];
#pragma unroll
  for (int n = 0; n < NC; ++n) { offk[n] = copy_off(n, 0, UK - 1); offv[n] = copy_off(n, 1, UK - 1); }
  auto issue = [&](int u, int st) __attribute__((always_inline)) {
    const long base = (long)u * UK * row_bytes;
    const unsigned dst = mine_u + st * SM::STAGE;
    if (u * UK + UK <= d.Skv) {
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(k0 + base, offk[n], dst + n * 1024);
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(v0 + base, offv[n], dst + SM::TILE + n * 1024);
    } else {                                       // the last keys: rows past them re-read the last one
      const int last = d.Skv - 1 - u * UK;
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(k0 + base, copy_off(n, 0, last), dst + n * 1024);
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(v0 + base, copy_off(n, 1, last), dst + SM::TILE + n * 1024);
    }
  };
  int u = u0 + wave;
  if (u < u1) issue(u, 0);
  if (u + NWV < u1) issue(u + NWV, 1);

  // ---- Q operands (behind the first copies: one trip to memory for both)
  bf16x8 qf[NB][KS];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int r = 32 * nb + ql, rc = min(r, rows - 1), hq = hk * G + rc / d.Sq, i = rc % d.Sq;
    const uint16_t* const q = (const uint16_t*)a.q + b * d.q_sb + hq * d.q_sh + (long)i * d.q_ss;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const u32x4 x = *(const u32x4*)(q + 16 * ks + 8 * g);
      qf[nb][ks] = __builtin_bit_cast(bf16x8, r < rows ? x : u32x4{0, 0, 0, 0});
    }
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[nb][ks]));

  f32x16 oacc[NB][DB];
  float m_ref[NB], l_run[NB];                      // reference (raw scores) and this lane's share of the sum
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[nb][db] = zero16();
    m_ref[nb] = -INFINITY;
    l_run[nb] = 0.f;
  }
  const float c2 = d.scale * LOG2E;
  const int k_row = ql * SM::ROWB, k_x = (g ^ k_swz<D>(ql)) * 16;
  const int j16 = lane & 15, half = (lane >> 4) & 1, tr_row = 4 * g + (j16 >> 2);
  int v_off[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
    v_off[db] = SM::TILE + tr_row * SM::ROWB + ((4 * db + 2 * half + ((j16 & 3) >> 1)) ^ v_swz<D>(tr_row)) * 16 + (j16 & 1) * 8;

  for (int st = 0; u < u1; u += NWV, st ^= 1) {
    if (u + NWV < u1) wait_vmcnt<NDMA>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const char* const t = mine + st * SM::STAGE;
    bf16x8 ka[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ka[ks] = *(const bf16x8*)(t + k_row + (k_x ^ (32 * ks)));
    f32x16 s[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      s[nb] = zero16();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s[nb] = mfma32(ka[ks], qf[nb][ks], s[nb]);
    }
    const int left = d.Skv - u * UK;
    if (left < UK) {                               // keys past the last one: no weight
      asm volatile("" ::: "memory");
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v / 4) + 4 * g + (v % 4) >= left) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) s[nb][v] = -INFINITY;
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float mx = s[nb][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[nb][v]);
      mx = fmaxf(xhalf_max(mx), -1e30f);           // (a row whose scores are all -infinity needs a finite reference)
      if (__any((mx - m_ref[nb]) * c2 > LAZY)) {
        const float m_new = fmaxf(m_ref[nb], mx);
        const float alpha = __builtin_amdgcn_exp2f((m_ref[nb] - m_new) * c2);     // m_ref = -inf -> 0
        m_ref[nb] = m_new;
        l_run[nb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[nb][db][v] *= alpha;
      }
      const float mc = m_ref[nb] * c2;
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[nb][v] = __builtin_amdgcn_exp2f(fmaf(s[nb][v], c2, -mc));
        sum += s[nb][v];
      }
      l_run[nb] += sum;
    }
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      bf16x8 pf[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) pf[nb] = cvt_operand(s[nb], 8 * t2);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const char* const p = t + v_off[db] + 16 * t2 * SM::ROWB;
        const s16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * SM::ROWB);
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        const s16x8 r = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) oacc[nb][db] = mfma32(__builtin_bit_cast(bf16x8, r), pf[nb], oacc[nb][db]);
      }
    }
    // every read of the stage has returned before the unit after next overwrites it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (u + NST * NWV < u1) issue(u + NST * NWV, st);
  }

  // ---- the four waves' results, combined in LDS (a wave's own stages hold its O: row r at r * 2 ROWB, the
  // 16-byte groups of four columns permuted by the row), then written: four columns per thread
  float* const st_m = (float*)(smem + SM::STATS);              // [wave][64] references, then sums
  float* const st_l = st_m + NWV * 64;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int r = 32 * nb + ql;
    const float l = xhalf_sum(l_run[nb]);
    if (g == 0) { st_m[wave * 64 + r] = m_ref[nb]; st_l[wave * 64 + r] = l; }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 y = {oacc[nb][db][4 * q4], oacc[nb][db][4 * q4 + 1], oacc[nb][db][4 * q4 + 2], oacc[nb][db][4 * q4 + 3]};
        *(f32x4*)(mine + r * 2 * SM::ROWB + (((8 * db + 2 * q4 + g) ^ (ql & (2 * CH - 1))) * 16)) = y;
      }
  }
  __syncthreads();
  constexpr int LPR = D / 4;                       // threads per row
  for (int x = tid; x < rows * LPR; x += 256) {
    const int r = x / LPR, c = x % LPR;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NWV; ++w) M = fmaxf(M, st_m[w * 64 + r]);
    float l = 0.f;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      const float lw = st_l[w * 64 + r];
      if (lw != 0.f) {                             // (a wave without a unit has nothing to add; a NaN has)
        const float e = __builtin_amdgcn_exp2f((st_m[w * 64 + r] - M) * c2);
        const f32x4 o = *(const f32x4*)(smem + w * SM::WAVE + r * 2 * SM::ROWB + ((c ^ (r & 31 & (2 * CH - 1))) * 16));
        l += e * lw;
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] += e * o[k];
      }
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const float lse = l != 0.f ? M * d.scale + logf(l) : -INFINITY;   // (NaN scores: NaN, which no combine drops)
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] *= inv;
    const int hq = hk * G + r / d.Sq, i = r % d.Sq;
    const long row = ((long)b * d.Hq + hq) * d.Sq + i;
    if (a.n_split > 1 || a.partial) {
      const long slice = (long)(a.part0 + split) * d.B * d.Hq * d.Sq + row;
      *(f32x4*)(a.o_part + slice * D + 4 * c) = y;
      if (c == 0) a.lse_part[slice] = lse;
    } else if (a.merge_into) {
      // Rescale of Algorithm 1 with the running (O, L) of this row (every thread of a row reads L
      // before the barrier, one of them replaces it after it)
      const float L0 = a.lse[row], Mx = max_or_nan(L0, lse);
      float w0 = 0.f, w1 = 0.f;
      if (Mx != -INFINITY) {
        const float L1 = Mx + logf(expf(L0 - Mx) + expf(lse - Mx));
        w0 = expf(L0 - L1);
        w1 = expf(lse - L1);
      }
      float* const o = (float*)a.o + row * D + 4 * c;
      const f32x4 old = *(const f32x4*)o;
      const f32x4 z = {w0 * old[0] + w1 * y[0], w0 * old[1] + w1 * y[1], w0 * old[2] + w1 * y[2], w0 * old[3] + w1 * y[3]};
      if (a.o_last) {
        const u32x2 x2 = {pack2_bf16(z[0], z[1]), pack2_bf16(z[2], z[3])};
        *(u32x2*)((uint16_t*)a.o_last + b * d.q_sb + hq * d.q_sh + (long)i * d.q_ss + 4 * c) = x2;
      } else {
        *(f32x4*)o = z;
      }
    } else {
      const long off = b * d.q_sb + hq * d.q_sh + (long)i * d.q_ss + 4 * c;
      if (a.o_is_f32) {
        *(f32x4*)((float*)a.o + off) = y;
      } else {
        const u32x2 z = {pack2_bf16(y[0], y[1]), pack2_bf16(y[2], y[3])};
        *(u32x2*)((uint16_t*)a.o + off) = z;
      }
      if (c == 0) a.lse[row] = lse;
    }
  }
  if (a.merge_into && a.n_split == 1 && !a.partial) {
    __syncthreads();
    if (tid < rows) {
      const int r = tid;
      float M = -INFINITY, l = 0.f;
      for (int w = 0; w < NWV; ++w) M = fmaxf(M, st_m[w * 64 + r]);
      for (int w = 0; w < NWV; ++w)
        if (st_l[w * 64 + r] != 0.f) l += __builtin_amdgcn_exp2f((st_m[w * 64 + r] - M) * c2) * st_l[w * 64 + r];
      const float lse = l != 0.f ? M * d.scale + logf(l) : -INFINITY;   // (NaN scores: NaN, which no combine drops)
      const long row = ((long)b * d.Hq + hk * G + r / d.Sq) * d.Sq + r % d.Sq;
      const float L0 = a.lse[row], Mx = max_or_nan(L0, lse);
      a.lse[row] = Mx == -INFINITY ? -INFINITY : Mx + logf(expf(L0 - Mx) + expf(lse - Mx));
    }
  }
}

template <int D, int NB>
hipError_t launch(const FwdArgs& a, hipStream_t s) {
  static SmemOnce once;
  const hipError_t e = ensure_dynamic_lds((const void*)fwd_rows_bf16_kernel<D, NB>, RowsSmem<D>::TOTAL, &once);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)(a.d.B * a.d.Hkv * a.n_split);
  fwd_rows_bf16_kernel<D, NB><<<grid, 256, RowsSmem<D>::TOTAL, s>>>(a);
  return hipGetLastError();
}

}  // namespace

bool fwd_rows_bf16_takes(const Dims& d, bool masked) { return !masked && (long)(d.Hq / d.Hkv) * d.Sq <= 64; }

int fwd_rows_bf16_pick_split(const Dims& d, int n_cu) {
  // One workgroup per compute unit (two with 64-wide heads) streams about 20 GB/s; a split has a unit of
  // keys for every wave, and costs a set of partial results written and read again.
  const int per_cu = d.D == 64 ? 2 : 1;
  long cap = ((d.Skv + UK - 1) / UK) / NWV;
  if (cap < 1) cap = 1;
  const double t_full = 4.0 * d.Skv * (double)d.D * per_cu / 20e9;
  const double t_part = 2.0 * (double)d.B * d.Hq * d.Sq * d.D * 4.0 / 3e12;
  return pick_split_balanced((long)d.B * d.Hkv, n_cu * per_cu, cap, t_full, t_part);
}

hipError_t launch_fwd_rows_bf16(const FwdArgs& a, hipStream_t s) {
  const bool two = (a.d.Hq / a.d.Hkv) * a.d.Sq > 32;
  if (a.d.D == 64) return two ? launch<64, 2>(a, s) : launch<64, 1>(a, s);
  if (a.d.D == 96) return two ? launch<96, 2>(a, s) : launch<96, 1>(a, s);
  return two ? launch<128, 2>(a, s) : launch<128, 1>(a, s);
}

}  // namespace lvx

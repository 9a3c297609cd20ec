// Dense forward loop for 64-wide heads: two workgroups on a compute unit, two wavefronts per SIMD.
#pragma once
#include "lvx_internal.h"
#include "lvx_kv_ring.h"
#include "lvx_mfma.h"

namespace lvx {
namespace fwdnarrow {

using namespace kvring;

// c = a b, c += a b with both operands in the accumulation registers
__device__ __forceinline__ void mfma_first_aa(f32x16& c, bf16x8 a_acc, bf16x8 b_acc) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "a"(a_acc), "a"(b_acc));
}
__device__ __forceinline__ void mfma_next_aa(f32x16& c, bf16x8 a_acc, bf16x8 b_acc) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "a"(a_acc), "a"(b_acc));
}

// Softmax over key tiles t_begin .. t_begin + nt - 1 of one wave's 64 query rows (operands qf), as in fwd_bf16_kernel:
// o = O^T relative to the reference r, l = this lane's share of the sum of p.  cut_tile: the tile whose keys below
// `low` the tile before has seen (-1: none).  All four waves of the workgroup call this.
//
// With 64-wide heads a half tile of 32 keys has 16 matrix instructions and 32 exponentials, so the
// vector ALU is as busy as the matrix pipe and one wave per SIMD pays for the sum of both and for every wait.
// The two row blocks of a wave therefore take turns (one scores and contracts while the other's scores are
// converted), which needs one set of score registers where fwd_bf16_kernel has two, and every operand is
// fetched into the registers it has just been used from, eight matrix instructions ahead of its next use: 209 registers
// in all, so that a second workgroup's waves issue while these wait.  8 heads x 4096 rows x 131072 keys: 2.51 -> 1.88
// million clocks, matrix pipes busy for 42 -> 56 % of them, at a clock that the power limit takes from 2.15 to 1.84
// GHz: 1158 -> 1040 us (1060 TFLOP/s).  Power is what bounds it now; 300 shapes of 64 to 16384 rows and 1024 to 131072 keys, half of
// them where the plans differ most, take 10 % less on average (33 % less to 9 % more; 11 more than 1 % more: calls of 48 to 82 us, most of them of 20 to
// 28 row tiles cut into about 500 parts where half as many would do, 4 heads x 1033 rows x 29869 keys 59 -> 65).
template <int D, class Issue>
__device__ __forceinline__ void fwd_narrow_loop(char* smem, const bf16x8 (&qf)[QB][D / 16], f32x16 (&o)[QB][D / 32], float (&r)[QB],
                                                float (&l)[QB], float c2, int t_begin, int nt, int cut_tile, int low,
                                                float lazy_sum, int lane, int tid, Issue&& issue_part) {
  using SM = KvSmem<D>;
  constexpr int KS = D / 16, DB = D / 32, CPR = SM::CPR, NDMA = 2 * SM::NCR, RINGS = NSTG;
  static_assert(KS == 2 * DB && QB == 2, "scores and contractions alternate one to one");
  const int g = lane >> 5, ql = lane & 31;

  bf16x8 kf[KS], vf[KS];               // K operands of the half being scored, V^T operands of the half being contracted
  f32x16 s[QB];
  u32x4 pw[QB][2] = {};                // packed P^T operands
#pragma unroll
  for (int k = 0; k < KS; ++k) vf[k] = bf16x8{};
  auto k_of = [&](const char* __restrict__ st, int hb, int k) __attribute__((always_inline)) -> bf16x8 {
    return *(const bf16x8*)(st + tile_off<D>(ql, 32 * hb, 16 * g) + k * 32);
  };
  auto v_of = [&](const char* __restrict__ st, int hb, int i) __attribute__((always_inline)) -> bf16x8 {
    return tile_tr_operand<D>(st + SM::TILE, 32 * hb + 16 * (i / DB), 32 * (i % DB), lane);
  };
  auto row_max = [&](const f32x16& sv) __attribute__((always_inline)) -> float {      // in units of log2 (c2 > 0)
    float m = fmaxf(fmaxf(sv[0], sv[1]), sv[2]);
#pragma unroll
    for (int v = 3; v < 15; v += 2) m = fmaxf(fmaxf(m, sv[v]), sv[v + 1]);
    return xhalf_max(fmaxf(m, sv[15])) * c2;
  };
  auto settle = [&](f32x16& x) __attribute__((always_inline)) { asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" : "+v"(x)); };
  auto mask_low = [&](f32x16& x, int hb) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = 32 * hb + 8 * (v / 4) + 4 * g + (v % 4) < low ? -INFINITY : x[v];
  };

  // One phase: scores of row block X (operands kf) alternate with its contraction of the half before (vf, pw[X]); the
  // scores of the other block are converted meanwhile.  loads: kf and vf of the next half follow their last use.
  auto phase = [&](auto x_block, const char* __restrict__ st_k, int hk, const char* __restrict__ st_v, int hv,
                   auto&& hook) __attribute__((always_inline)) {
    constexpr int X = decltype(x_block)::value, Y = 1 - X;
    constexpr int NM = 2 * KS;
    float ex[16], lh = 0.f;
    float carry = 0.f;
    auto start = [&](int e) __attribute__((always_inline)) { ex[e] = __builtin_amdgcn_exp2f(fmaf(s[Y][e], c2, -r[Y])); };
    auto finish = [&](int e) __attribute__((always_inline)) {
      lh = e == 0 ? ex[e] : lh + ex[e];
      if (e % 2 == 0) carry = ex[e];
      else pw[Y][e / 8][(e % 8) / 2] = pack2_bf16(carry, ex[e]);
    };
    constexpr int M0 = 1, M1 = NM - 1;             // conversions start in units M0 .. M1 - 1, and finish a unit later
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int i = m / 2;
      if (m % 2 == 0) {
        if (i == 0) mfma_first_aa(s[X], kf[i], qf[X][i]);
        else mfma_next_aa(s[X], kf[i], qf[X][i]);
        if (X == 1) kf[i] = k_of(st_k, hk, i);
      } else {
        mfma_acc(o[X][i % DB], vf[i], __builtin_bit_cast(bf16x8, pw[X][i / DB]));
        if (X == 1) vf[i] = v_of(st_v, hv, i);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int at = M0 + e * (M1 - M0) / 16;
        if (at == m) start(e);
        if (at + 1 == m) finish(e);
      }
      hook(m);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The half's sum of probabilities bounds each of them (see fwd_bf16_kernel): too large, and the reference goes up.
    if (__builtin_expect(__ballot(!(lh <= lazy_sum)) != 0, 0)) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int db = 0; db < DB; ++db) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(o[Y][db]));
      const float r_new = fmaxf(r[Y], row_max(s[Y]));
      const float alpha = __builtin_amdgcn_exp2f(r[Y] - r_new);
      r[Y] = r_new;
      l[Y] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int v = 0; v < 16; ++v) o[Y][db][v] *= alpha;
        asm volatile("s_nop 7" : "+a"(o[Y][db]));
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) { start(e); finish(e); }
    }
    l[Y] += lh;
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  auto no_hook = [](int) __attribute__((always_inline)) {};
  auto stage = [&](int q) __attribute__((always_inline)) -> char* { return smem + (q % RINGS) * SM::STAGE; };

#pragma unroll
  for (int q = 0; q < RINGS - 1; ++q)
    if (q < nt) {
#pragma unroll
      for (int k = 0; k < NDMA; ++k) issue_part(t_begin + q, stage(q), k, q);
    }
  wait_vmcnt<0>();
  __syncthreads();
  const bool cut = cut_tile >= 0 && cut_tile == t_begin + nt - 1;      // the last tile, if any
#pragma unroll
  for (int k = 0; k < KS; ++k) kf[k] = k_of(smem, 0, k);
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      if (k == 0) mfma_first_aa(s[qb], kf[k], qf[qb][k]);
      else mfma_next_aa(s[qb], kf[k], qf[qb][k]);
    }
    settle(s[qb]);
    if (cut && nt == 1) mask_low(s[qb], 0);
    r[qb] = fmaxf(row_max(s[qb]), -1e30f);         // no probability of the first half exceeds 1
  }
  asm volatile("" ::: "memory");

  int T = 0;
  for (; T + RINGS - 1 < nt; ++T) {
    char* const sa = stage(T);
    char* const sb = stage(T + 1);
    char* const sc = stage(T + RINGS - 1);
    phase(B1{}, sa, 1, sa, 0, no_hook);
    phase(B0{}, sa, 0, sa, 0, no_hook);
    wait_vmcnt<NDMA>();                            // tile T + 1 is in place; every wave is done with tile T - 1
    wg_barrier();
    phase(B1{}, sb, 0, sa, 1, [&](int m) __attribute__((always_inline)) {
      if (m % 2 == 1 && m / 2 < NDMA) issue_part(t_begin + T + RINGS - 1, sc, m / 2, 0);
    });
    phase(B0{}, sb, 0, sb, 0, [&](int m) __attribute__((always_inline)) {
      if (m % 2 == 1 && KS + m / 2 < NDMA) issue_part(t_begin + T + RINGS - 1, sc, KS + m / 2, 0);
    });
  }
  for (; T < nt; ++T) {                            // no tile left to copy
    char* const sa = stage(T);
    char* const sb = stage(T + 1);
    const bool cut_here = cut && T + 1 == nt;
    if (cut_here) {
      // The rows of V that the moved last tile repeats are cleared (their weight is 0, but 0 times an infinite value
      // is not), and the scores of these keys are -infinity.
      asm volatile("" ::: "memory");
      if (nt > 1) { settle(s[0]); mask_low(s[0], 0); }
#pragma unroll 1
      for (int x = tid; x < low * CPR; x += 256) *(u32x4*)(sa + SM::TILE + tile_off<D>(x / CPR, 0, x % CPR * 16)) = u32x4{0, 0, 0, 0};
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wg_barrier();
    }
    phase(B1{}, sa, 1, sa, 0, no_hook);
    if (cut_here) { settle(s[1]); mask_low(s[1], 0); }
    phase(B0{}, sa, 0, sa, 0, no_hook);
    if (cut_here) { settle(s[0]); mask_low(s[0], 1); }
    wait_vmcnt<0>();
    wg_barrier();
    phase(B1{}, sb, 0, sa, 1, no_hook);
    if (cut_here) { settle(s[1]); mask_low(s[1], 1); }
    phase(B0{}, sb, 0, sb, 0, no_hook);
  }
  if (nt > 0) {                                    // (a block of its own: what reads the results stands behind a wait)
#pragma unroll
    for (int i = 0; i < KS; ++i) mfma_acc(o[1][i % DB], vf[i], __builtin_bit_cast(bf16x8, pw[1][i / DB]));
  }
}

}  // namespace fwdnarrow
}  // namespace lvx

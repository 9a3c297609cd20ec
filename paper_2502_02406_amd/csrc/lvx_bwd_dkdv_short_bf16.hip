// bf16 backward, dK and dV of key tiles that few query rows see: the products and the order of the sums of
// lvx_bwd_dkdv_bf16.hip, in workgroups half as large of which two or three share a compute unit.
//
// Workgroup = 4 wavefronts = 128 keys of one (batch, K/V head), 32 keys a wave: K and V operands, dK^T and dV^T
// accumulators and the scores of one step in at most 256 registers (168 with 64-wide heads).  [Q; dO] tiles of 32
// rows and their statistics travel HBM -> LDS as there, into a ring of three stages.  A wave performs a step's phases
// one after the other; what fills the pipes meanwhile is the other workgroups' waves.
#include "lvx_internal.h"
#include "lvx_mfma.h"

namespace lvx {

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr int NWV = 4;                 // waves per workgroup
constexpr int KN = NWV * 32;           // keys per workgroup
constexpr int KM = 32;                 // query rows per step
constexpr int NSTG = 3;                // ring stages
constexpr int wg_per_cu(int D) { return D == 64 ? 3 : 2; }

template <int D> struct ShortSmem {
  static constexpr int CPR = D / 8;                 // 16-byte chunks of data per row
  static constexpr int P = (D + 8) * 2;             // row pitch in bytes
  static constexpr int SPR = P / 16;                // 16-byte slots per row
  static constexpr int RUN = 8 * SPR;               // slots of one run: 8 consecutive physical rows
  static constexpr int NCR = (RUN + 63) / 64;       // wave-level copies (64 slots) per run
  static constexpr int STAT_OFF = ILV_ROWS * P;     // 32 x -L log2(e), then 32 x -delta
  static constexpr int STAGE = STAT_OFF + 256;      // [Q; dO] as one 64-row interleaved tile + statistics
  static constexpr int RING = NSTG * STAGE;
  // (a few hundred bytes more and 64-wide heads have two workgroups on a compute unit: 16 heads x 65536 keys, 1024 rows, causal 360 -> 336 us with
  // three, 256 rows of which every key block of 128 in four is seen 196 -> 154)
  static constexpr int TOTAL = lds_share(wg_per_cu(D));
  static constexpr int LIST_CAP = (TOTAL - RING) / 4 - 1;      // list of steps and words behind it; the length in the last word
  static_assert(NWV * 32 * (D * 2 + 16) <= RING, "the turn-around buffers fit the ring");
  static_assert(RUN >= 64, "a run must hold at least one full copy");
};

// MODE 0: dense.  1: a media mask whose chunks are multiples of 32 rows and whose key blocks are multiples of 128
// keys: it selects which steps a workgroup performs.  2: any other, by the words of MaskRows.  (The variants of
// bwd_dkdv_bf16_kernel, which explains them.)  PAST: dK and dV are written past the caches (dkdv_past).
template <int D, int MODE, bool PAST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(wg_per_cu(D), wg_per_cu(D))))
bwd_dkdv_short_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using SM = ShortSmem<D>;
  constexpr int KS = D / 16, DB = D / 32, CPR = SM::CPR, NCR = SM::NCR;
  constexpr bool WORDS = MODE == 2;
  const Dims& d = a.d;
  const int G = d.Hq / d.Hkv, n_kt = (d.Skv + KN - 1) / KN;
  HeadWork hw;
  if (!xcd_decode(blockIdx.x, d.B * d.Hkv, n_kt, &hw, MODE != 0)) return;
  const int b = hw.head / d.Hkv, hk = hw.head % d.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, kl = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j_wg0 = hw.item * KN, j_wg1 = min(d.Skv, j_wg0 + KN) - 1, j_wave0 = j_wg0 + 32 * wave;
  const int spH = (d.Sq + KM - 1) / KM;

  // ---- the steps (of one head) that some key of the workgroup is seen by
  int* const tl = (int*)(smem + SM::RING);
  const int f0 = WORDS ? j_wg0 / a.mask.kv_block : 0, nf = WORDS ? j_wg1 / a.mask.kv_block - f0 + 1 : 1;
  const unsigned* const wtab = (const unsigned*)tl + spH;
  int per_head = spH;
  if (MODE != 0) {
    if (WORDS) {
      const unsigned* const rw = a.rows.words + b * a.rows.stride_b;
      for (int c = tid; c < spH * nf; c += 256) {
        const int t = c / nf, f = f0 + c % nf;
        auto word = [&](int tt) -> unsigned { return rw[((long)(tt >> 3) * a.rows.w1 + f) * 8 + (tt & 7)]; };
        unsigned x = word(t);
        if (t == spH - 1 && d.Sq % KM != 0) x = (word(t - 1) >> (d.Sq % KM)) | (x << (KM - d.Sq % KM));
        ((unsigned*)wtab)[c] = x;
      }
      __syncthreads();
    }
    const uint8_t* const col = a.mask.allow + b * a.mask.stride_b + j_wg0 / a.mask.kv_block;
    if (wave == 0) {
      int count = 0;
      for (int base = 0; base < spH; base += 64) {       // (wave-uniform trip count)
        const int t = base + lane;
        bool on = t < spH;
        if (WORDS) {
          unsigned any = 0;
          for (int f = 0; f < nf; ++f) any |= wtab[min(t, spH - 1) * nf + f];
          on = on && any != 0;
        } else {
          on = on && col[(long)((t * KM) / a.mask.q_chunk) * a.mask.stride_q] != 0;
        }
        const unsigned long long m = __ballot(on);
        if (on) tl[count + __popcll(m & ((1ull << lane) - 1ull))] = t;
        count += (int)__popcll(m);
      }
      if (lane == 0) tl[SM::LIST_CAP] = count;
    }
    __syncthreads();
    per_head = __builtin_amdgcn_readfirstlane(tl[SM::LIST_CAP]);
  }
  const int n = G * per_head;
  const long kv_head = b * d.kv_sb + hk * d.kv_sh;
  if (MODE != 0 && n == 0) {                       // keys that no query sees: dK = dV = 0, nothing to read
    const u32x4 z = {0, 0, 0, 0};
    for (int c = tid; c < KN * CPR; c += 256) {
      const int j = j_wg0 + c / CPR, col = (c % CPR) * 8;
      if (j >= d.Skv) continue;
      const long off = kv_head + (long)j * d.kv_ss + col;
      store_dkdv<PAST>((uint16_t*)a.dk + off, z);
      store_dkdv<PAST>((uint16_t*)a.dv + off, z);
    }
    return;
  }

  // ---- tile copies, as in bwd_dkdv_bf16_kernel
  const char* const q0 = (const char*)a.q + (b * d.q_sb) * 2;
  const char* const g0 = (const char*)a.d_o + (b * d.q_sb) * 2;
  const unsigned row_bytes = (unsigned)(d.q_ss * 2);
  auto run_start = [&](int c) __attribute__((always_inline)) -> int { return c + 1 < NCR ? 64 * c : SM::RUN - 64; };
  unsigned cp_off[NCR];
#pragma unroll
  for (int c = 0; c < NCR; ++c) {
    const int sl = run_start(c) + lane;
    cp_off[c] = (unsigned)(4 * (sl / SM::SPR)) * row_bytes + (unsigned)min(sl % SM::SPR, CPR - 1) * 16;
  }
  constexpr int NDMA = 2 * NCR + 1;
  const unsigned smem_u = lds_base(smem);
  int k_next = 0, h_next = 0;                      // the next step to copy: position among the steps of a head, head of the group
  auto tile_at = [&](int k) __attribute__((always_inline)) -> int { return MODE != 0 ? __builtin_amdgcn_readfirstlane(tl[k]) : k; };
  auto issue_next = [&](int slot) __attribute__((always_inline)) {
    const int hq = hk * G + h_next, i0 = tile_at(k_next) * KM;
    // (a short last step takes rows Sq-32 .. Sq-1 and their own statistics)
    const int i0_eff = min(i0, d.Sq - KM);
    const long tile = ((long)hq * d.q_sh + (long)i0_eff * d.q_ss) * 2 + (long)wave * row_bytes;
    const char* const lb = (const char*)(i0 != i0_eff ? a.stats_ovl + ((long)b * d.Hq + hq) * 64
                                                      : a.stats + (((long)b * d.Hq + hq) * a.sq_pad + i0) * 2);
    const unsigned dst = smem_u + (unsigned)(slot * SM::STAGE), qdst = dst + 20 * wave * SM::P;
#pragma unroll
    for (int c = 0; c < NCR; ++c) {
      dma16u(q0 + tile, cp_off[c], qdst + run_start(c) * 16);
      dma16u(g0 + tile, cp_off[c], qdst + 8 * SM::P + run_start(c) * 16);
    }
    dma4u(lb, lane * 4, dst + SM::STAT_OFF);
    if (++k_next == per_head) { k_next = 0; ++h_next; }
  };
#pragma unroll
  for (int q = 0; q < NSTG - 1; ++q)
    if (q < n) issue_next(q);

  // ---- K operands (times scale log2 e, so that S starts and ends in the exponent of P) and V operands of the wave's keys
  bf16x8 kf[KS], vf[KS];
  {
    const int j = j_wave0 + kl;
    const long off = kv_head + (long)min(j, d.Skv - 1) * d.kv_ss + 8 * g;
    u32x4 xk[KS], xv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xk[ks] = *(const u32x4*)((const uint16_t*)a.k + off + 16 * ks);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xv[ks] = *(const u32x4*)((const uint16_t*)a.v + off + 16 * ks);
    const float c2 = d.scale * LOG2E;
    const u32x4 zero4 = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 x = j < d.Skv ? xk[ks] : zero4;
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = pack2_bf16(__uint_as_float(x[w] << 16) * c2, __uint_as_float(x[w] & 0xffff0000u) * c2);
      kf[ks] = __builtin_bit_cast(bf16x8, x);
      vf[ks] = __builtin_bit_cast(bf16x8, j < d.Skv ? xv[ks] : zero4);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(kf[ks]), "+v"(vf[ks]));   // (here, so that nothing in the loop waits for memory)
  }
  const int wlane = WORDS ? min(j_wave0 + kl, d.Skv - 1) / a.mask.kv_block - f0 : 0;

  f32x16 dk[DB], dv[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) { dk[i] = zero16(); dv[i] = zero16(); }
  int slot = 0, k_cur = 0;
  for (int i = 0; i < n; ++i) {
    // step i has landed in every wave's copies, and every wave is done with step i - 1, whose stage takes step i + 2
    if (i + 1 < n) wait_vmcnt<NDMA>();
    else wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();
    asm volatile("" ::: "memory");
    const char* const t = smem + slot * SM::STAGE;
    unsigned word = 0;
    if (WORDS) word = wtab[__builtin_amdgcn_readfirstlane(tl[k_cur]) * nf + wlane] >> (4 * g);
    if (++k_cur == per_head) k_cur = 0;
    if (i + NSTG - 1 < n) issue_next(slot == 0 ? NSTG - 1 : slot - 1);
    slot = slot + 1 == NSTG ? 0 : slot + 1;

    f32x16 s, p;                                   // lane = key, registers = query rows; they start at -L log2 e and -delta
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 nl = *(const f32x4*)(t + SM::STAT_OFF + (8 * q4 + 4 * g) * 4);
      const f32x4 nd = *(const f32x4*)(t + SM::STAT_OFF + 128 + (8 * q4 + 4 * g) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { s[4 * q4 + e] = nl[e]; p[4 * q4 + e] = nd[e]; }
    }
    const char* const qrow = t + ilv_off<D>(kl, 0, 8 * g);
    const char* const grow = t + ilv_off<D>(kl, KM, 8 * g);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      s = mfma32(*(const bf16x8*)(qrow + ks * 32), kf[ks], s);
      p = mfma32(*(const bf16x8*)(grow + ks * 32), vf[ks], p);
    }
    u32x4 pw[2], sw[2];                            // packed P and dS operands
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      float pr[2], ds[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        pr[e] = __builtin_amdgcn_exp2f(s[v + e]);
        if (WORDS) {
          unsigned keep;
          asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(keep) : "v"(word), "n"(8 * ((v + e) / 4) + (v + e) % 4));
          pr[e] = __uint_as_float(__float_as_uint(pr[e]) & keep);
        }
        ds[e] = pr[e] * p[v + e];
      }
      pw[v / 8][(v % 8) / 2] = pack2_bf16(pr[0], pr[1]);
      sw[v / 8][(v % 8) / 2] = pack2_bf16(ds[0], ds[1]);
    }
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        dv[db] = mfma32(load_tr_operand_ilv<D>(t, KM + 16 * t2, 32 * db, lane), __builtin_bit_cast(bf16x8, pw[t2]), dv[db]);
        dk[db] = mfma32(load_tr_operand_ilv<D>(t, 16 * t2, 32 * db, lane), __builtin_bit_cast(bf16x8, sw[t2]), dk[db]);
      }
  }

  // ---- write dK = scale * acc, dV = acc: each wave turns its rows around through LDS and writes them whole
  __syncthreads();
  constexpr int RP = D * 2 + 16;                   // row pitch of the turn-around buffer (padded against bank conflicts)
  char* const buf = smem + wave * (32 * RP);
  constexpr int LPR = D / 8, RPI = 64 / LPR;       // lanes per row, rows per instruction
  const int rsub = lane / LPR, cb = (lane % LPR) * 16;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const float f = which == 0 ? d.scale : 1.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x16& x = which == 0 ? dk[db] : dv[db];
        *(u32x2*)(buf + kl * RP + (32 * db + 8 * q4 + 4 * g) * 2) =
            u32x2{pack2_bf16(x[4 * q4] * f, x[4 * q4 + 1] * f), pack2_bf16(x[4 * q4 + 2] * f, x[4 * q4 + 3] * f)};
      }
    // (each wave reads back only what it wrote itself: no barrier, the LDS queue keeps the order)
    char* const out = (char*)(which == 0 ? a.dk : a.dv);
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int r = r0 + rsub, j = j_wave0 + r;
      if ((64 % LPR != 0 && rsub >= RPI) || r >= 32) continue;
      const u32x4 y = *(const u32x4*)(buf + r * RP + cb);
      if (j < d.Skv) store_dkdv<PAST>(out + (kv_head + (long)j * d.kv_ss) * 2 + cb, y);
    }
  }
}

template <int D, int MODE, bool PAST>
hipError_t launch(const BwdArgs& a, hipStream_t s) {
  static SmemOnce once;
  constexpr int lds = MODE == 0 ? ShortSmem<D>::RING : ShortSmem<D>::TOTAL;
  static_assert(lds_holds(wg_per_cu(D), lds), "the workgroups of a compute unit share its LDS");
  const hipError_t e = ensure_dynamic_lds((const void*)bwd_dkdv_short_kernel<D, MODE, PAST>, lds, &once);
  if (e != hipSuccess) return e;
  const long grid = xcd_grid(a.d.B * a.d.Hkv, (a.d.Skv + KN - 1) / KN);
  bwd_dkdv_short_kernel<D, MODE, PAST><<<(unsigned)grid, 256, lds, s>>>(a);
  return hipGetLastError();
}
template <int D, bool PAST> hipError_t launch(const BwdArgs& a, int mode, hipStream_t s) {
  return mode == 0 ? launch<D, 0, PAST>(a, s) : mode == 1 ? launch<D, 1, PAST>(a, s) : launch<D, 2, PAST>(a, s);
}
template <int D> hipError_t launch(const BwdArgs& a, int mode, hipStream_t s) {
  return dkdv_past(a.d.B * a.d.Hkv, a.d.Skv, D) ? launch<D, true>(a, mode, s) : launch<D, false>(a, mode, s);
}

}  // namespace

// Whether it takes the call: the larger workgroups' loop has half the LDS traffic per matrix instruction, so the line lies where
// their set-up and epilogue (25 thousand clocks that nothing overlaps) no longer outweigh that.  2 x 16 heads x 32768 keys, larger
// workgroups -> these, us: D = 64, 1 step 124 -> 82, 4 steps 164 -> 123, 16 steps 314 -> 290, 32 steps 521 -> 517, 64 (32 / 8 heads x
// 512 rows x 65536 keys) 470 -> 494; D = 96, 4 steps 260 -> 193, 16 steps 455 -> 443, 32 steps 730 -> 767; D = 128, 4 steps 321 -> 257,
// 8 steps 401 -> 366, 12 steps 492 -> 482, 16 steps 575 -> 591.  Under a mask a tile has fewer steps than there are, how many only the
// device knows: about half under a causal one (16 heads x 65536 keys, 32 steps: D = 64 398 -> 336, D = 96 515 -> 491; D = 128 637 -> 630;
// 48 steps, D = 64 396 -> 347).
// And the list of steps, and the words that mode 2 needs, have to fit beside the ring.
// Workgroups go to an XCD's shader engines in a fixed order, so a mask that shows every fourth tile leaves three of four engines idle.  The larger
// workgroups have that too, at tiles twice as long: 16 heads x 1536 rows x 65536 keys, D = 64, a quarter of the key blocks seen, larger workgroups
// and these, us: every fourth of 128 keys 846 and 642, of 256 714 and 313, of 1024 234 and 221; a random quarter of 128 495 and 285, of 256 339 and 249.
bool bwd_dkdv_short_takes(const Dims& d, const MaskDev& m, int mode) {
  const int spH = (d.Sq + KM - 1) / KM;
  const long steps = (long)(d.Hq / d.Hkv) * spH;
  if (mode == 0) return steps <= (d.D == 64 ? 24 : d.D == 96 ? 16 : 12);
  if (steps > (d.D == 64 ? 48 : d.D == 96 ? 32 : 24)) return false;
  const int cap = d.D == 64 ? ShortSmem<64>::LIST_CAP : d.D == 96 ? ShortSmem<96>::LIST_CAP : ShortSmem<128>::LIST_CAP;
  if (mode == 1) return m.kv_block % KN == 0 && spH <= cap;
  const int w = (d.Skv - 1) / m.kv_block + 1;
  long nf = m.kv_block % KN == 0 ? 1 : KN % m.kv_block == 0 ? KN / m.kv_block : (KN - 2) / m.kv_block + 2;
  if (nf > w) nf = w;
  return (1 + nf) * spH <= cap;
}

hipError_t launch_bwd_dkdv_short(const BwdArgs& a, int mode, hipStream_t s) {
  return a.d.D == 64 ? launch<64>(a, mode, s) : a.d.D == 96 ? launch<96>(a, mode, s) : launch<128>(a, mode, s);
}

}  // namespace lvx

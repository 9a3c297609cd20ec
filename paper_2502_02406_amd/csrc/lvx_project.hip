// Projection kernels: the products of Section 2 that make the attention operands from the token
// features, Q = x W_Q and K, V = y W_K, y W_V, which Section 3.2 has the backward pass compute
// again from the single saved copy of the visual tokens instead of keeping K and V per layer.
//
// out[o][b, h, s, c] = sum_e x[b, s, e] * w[(o H + h) D + c, e]: x is [M = B S tokens, E], w holds
// the projection matrices transposed and stacked ([n_out H D, E], the layout of a linear layer's
// weight), and the result is written head-major, which is the layout the attention kernels read.
//
// bf16: one workgroup = 4 wavefronts (one per SIMD, the whole register file each) makes a
// 256-token x 256-column tile; a wave owns 128 x 128 of it as 4 x 4 blocks of 32 x 32 whose
// accumulators fill the accumulation registers, so each operand read from LDS feeds four matrix
// instructions.  The product is formed transposed (columns of w as the A operand, tokens as B):
// a lane then holds ONE token and, per block, groups of four consecutive columns.
// x and w tiles of 64 features travel HBM -> LDS by direct copies, whole 128-byte lines per row
// (half lines cost as many entries of the memory pipeline as whole ones and halve its
// throughput), into two slots of 64 KB that alternate; the copies of a tile pair go out while
// the pair before it is being multiplied, spread over the matrix instructions.  The eight
// 16-byte chunks of a tile row are stored permuted (perm_of) so that the rows a quarter-wave
// reads together cover all banks.  The one barrier per 64 matrix instructions sits before the
// last quarter of a tile pair, when its last operands are already in registers: behind it the
// first operands of the next pair are read and the slot is free for the pair after that.
// Problems with fewer 256 x 256 tiles than three quarters of the compute units take tiles of 128 tokens
// (IB = 2: six operands per eight matrix instructions instead of eight per sixteen, but twice the
// workgroups): 2048 tokens x 4096 features x 4096 columns, 128 tiles of 256 x 256, 87 -> 67 us; 2048
// tokens x 512 x 1024 19 -> 12.6 us.
// The epilogue turns the tile around in LDS (rounded to bf16) and writes whole 256-byte rows.
// More tiles than compute units, of at least 512 features: project_run_bf16_kernel, whose workgroups stay.
#include "lvx_internal.h"
#include "lvx_mfma.h"
#include "lvx_kv_ring.h"
#include "lvx_tile_run.h"

#include <type_traits>

namespace lvx {

namespace {

constexpr int TN = 256;                // columns per workgroup
constexpr int BK = 64;                 // features per tile pair
constexpr int NSLOT = 2;               // LDS slots
constexpr int ROWB = BK * 2;           // bytes of a tile row: one 128-byte line
constexpr int TILE_B = 256 * ROWB;     // one operand's tile (of x: of the room for it)
constexpr int SLOT_B = 2 * TILE_B;     // x tile, then w tile
constexpr int RING_B = NSLOT * SLOT_B;
constexpr int TB_PITCH = 128 * 2 + 16; // epilogue: a wave's 128 tokens x 128 columns of bf16, padded rows
constexpr int TB_WAVE = 128 * TB_PITCH;
constexpr int SMEM_B = RING_B > 4 * TB_WAVE ? RING_B : 4 * TB_WAVE;

// Position permutation of a tile row's eight chunks: chunk c of row r sits at position
// c ^ perm_of(r).  Eight consecutive rows get eight different values, and two rows eight apart
// differ too, so the 16-byte reads of 8 or of 16 consecutive rows at one chunk never meet in a
// bank (rows are 128 bytes apart).
__device__ __forceinline__ int perm_of(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// IB: blocks of 32 tokens per wave
template <int IB>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
project_bf16_kernel(ProjArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int TM = 64 * IB;                        // tokens per workgroup
  constexpr int XC = 2 * IB;                         // copies of x per wave and tile pair (8 rows each; of w: 8)
  constexpr int NPART = XC + 8;
  const int n_mt = (int)((a.M + TM - 1) / TM), n_nt = a.N / TN;
  HeadWork hw;                                       // the column tiles of a token tile share an XCD (and its L2)
  if (!tile_decode(blockIdx.x, n_mt, n_nt, &hw)) return;
  const long m0 = (long)hw.head * TM;
  const int n0 = hw.item * TN;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l31 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;           // this wave's 32 IB tokens / 128 columns of the tile
  const int nk = a.E / BK;

  // ---- copies: one instruction moves 8 rows x 128 bytes; lane l fills slot l of them, i.e. row
  // l / 8, position l % 8, which holds chunk (l % 8) ^ perm_of(row).  A wave copies rows
  // 8 XC wave + 8 j + l / 8 of the x tile, 64 wave + 8 j + l / 8 of the w tile.  Rows past the last token re-read the last
  // one (their results are never stored).
  const unsigned xrow_b = (unsigned)(a.ldx * 2), wrow_b = (unsigned)(a.E * 2);
  const long m_last = a.M - 1 - m0;
  unsigned xo[XC], wo[2];
#pragma unroll
  for (int j = 0; j < XC; ++j) {
    const int r = 8 * XC * wave + 8 * j + (lane >> 3);
    const unsigned swz = 16u * (unsigned)((lane & 7) ^ perm_of(8 * j + (lane >> 3)));
    xo[j] = (unsigned)(r < m_last ? r : (int)m_last) * xrow_b + swz;
    if (j < 2) wo[j] = (unsigned)(lane >> 3) * wrow_b + swz;      // (the permutation repeats every 16 rows)
  }
  const char* const xg = (const char*)a.x + m0 * (long)xrow_b;
  const char* const wg = (const char*)a.w + ((long)n0 + 64 * wave) * wrow_b;
  const unsigned smem_u = lds_base(smem);
  auto issue_part = [&](int kt, int part) __attribute__((always_inline)) {
    // (the slot as an LDS address: a cast from the generic pointer carries a null test, two scalar instructions a copy)
    const unsigned st = smem_u + (unsigned)((kt % NSLOT) * SLOT_B);
    if (part < XC) {
      dma16u(xg + (long)kt * ROWB, xo[part], st + (unsigned)((8 * XC * wave + 8 * part) * ROWB));
    } else {
      const int j = part - XC;
      dma16u(wg + (long)(8 * j) * wrow_b + (long)kt * ROWB, wo[j & 1], st + (unsigned)(TILE_B + (64 * wave + 8 * j) * ROWB));
    }
  };

  // ---- operands: block i of this wave's tokens / block j of its columns, k-step q = 0 .. 3 of a
  // tile pair.  Lane l reads row l % 32, chunk 2 q + g, at position chunk ^ perm_of(row).
  int rd[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) rd[q] = l31 * ROWB + 16 * ((2 * q + g) ^ perm_of(l31));
  const int xbase = wm * 32 * IB * ROWB, wbase = TILE_B + wn * 128 * ROWB;
  auto x_op = [&](const char* st, int q, int i) __attribute__((always_inline)) -> bf16x8 {
    return *(const bf16x8*)(st + xbase + 32 * i * ROWB + rd[q]);
  };
  auto w_op = [&](const char* st, int q, int j) __attribute__((always_inline)) -> bf16x8 {
    return *(const bf16x8*)(st + wbase + 32 * j * ROWB + rd[q]);
  };

  f32x16 acc[4][IB];                                 // [column block j][token block i], transposed blocks
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < IB; ++i) { acc[j][i] = zero16(); asm volatile("" : "+a"(acc[j][i])); }

  // the 4 IB matrix instructions of one k-step; hook(u) is other work issued after instruction u
  auto mma16 = [&](const bf16x8 (&xv)[IB], const bf16x8 (&wv)[4], auto&& hook) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        kvring::mfma_acc(acc[j][i], wv[j], xv[i]);
        hook(IB * j + i);
        __builtin_amdgcn_sched_barrier(0);
      }
  };

  // ---- pipeline: pairs 0 and 1 go out whole; later, pair P + 2 goes out in two batches, the
  // first during the last k-step of pair P (right behind the barrier that frees its slot), the
  // second during the first k-step of pair P + 1
#pragma unroll
  for (int q = 0; q < NSLOT; ++q)
    if (q < nk) {
#pragma unroll
      for (int part = 0; part < NPART; ++part) issue_part(q, part);
    }
  if (nk > 1) wait_vmcnt<NPART>();
  else wait_vmcnt<0>();
  wg_barrier();
  bf16x8 xa[IB], wa[4], xb[IB], wb[4];               // operands of even / odd k-steps
#pragma unroll
  for (int i = 0; i < IB; ++i) xa[i] = x_op(smem, 0, i);
#pragma unroll
  for (int i = 0; i < 4; ++i) wa[i] = w_op(smem, 0, i);

  // fetches the operands of k-step q of the pair in slot st, one per matrix instruction
  auto fetch = [&](const char* st, int q, int u, bf16x8 (&xv)[IB], bf16x8 (&wv)[4]) __attribute__((always_inline)) {
    if (u < IB) xv[u] = x_op(st, q, u);
    else if (u < IB + 4) wv[u - IB] = w_op(st, q, u - IB);
  };
  constexpr int EW = 4 * IB / 8;                     // a copy of w every EW matrix instructions of a k-step, one of x every two
  auto pair = [&](int P, auto steady, bool send2, bool send1, bool more) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;   // send2, send1 and more are all true
    const char* const st = smem + (P % NSLOT) * SLOT_B;
    const char* const sn = smem + ((P + 1) % NSLOT) * SLOT_B;
    mma16(xa, wa, [&](int u) __attribute__((always_inline)) {
      fetch(st, 1, u, xb, wb);
      if ((STEADY || send2) && u % EW == EW - 1) issue_part(P + 1, XC + u / EW);
    });
    mma16(xb, wb, [&](int u) __attribute__((always_inline)) { fetch(st, 2, u, xa, wa); });
    mma16(xa, wa, [&](int u) __attribute__((always_inline)) { fetch(st, 3, u, xb, wb); });
    // Pair P + 1 has landed when none of this wave's copies is outstanding, and this wave's last
    // reads of pair P have returned; behind the barrier that holds for every wave: pair P + 1 can
    // be read, and the slot of pair P be overwritten.
    if (STEADY || more) {
      __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0) and lgkmcnt(0)
      wg_barrier();
    }
    mma16(xb, wb, [&](int u) __attribute__((always_inline)) {
      if (STEADY || more) fetch(sn, 0, u, xa, wa);
      if ((STEADY || send1) && u % 2 == 1) issue_part(P + 2, u / 2);
    });
  };
  int P = 0;
  if (nk > 0) { pair(0, std::false_type{}, false, 2 < nk, 1 < nk); P = 1; }
  for (; P + 2 < nk; ++P) pair(P, std::true_type{}, true, true, true);
  for (; P < nk; ++P) pair(P, std::false_type{}, P + 1 < nk, false, P + 1 < nk);

  // ---- epilogue.  Every wave has left the ring (its slots become the turn-around buffers) and
  // the last matrix instructions have retired before their registers are read.
  wg_barrier();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < IB; i += 2) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[j][i]), "+a"(acc[j][i + 1]));
  char* const tb = smem + wave * TB_WAVE;
#pragma unroll
  for (int i = 0; i < IB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {                  // registers 4 q .. 4 q + 3: columns 32 j + 8 q + 4 g + (0..3)
        const u32x2 y = {pack2_bf16(acc[j][i][4 * q], acc[j][i][4 * q + 1]),
                         pack2_bf16(acc[j][i][4 * q + 2], acc[j][i][4 * q + 3])};
        *(u32x2*)(tb + (32 * i + l31) * TB_PITCH + (32 * j + 8 * q + 4 * g) * 2) = y;
      }
  // (the buffer is this wave's own: its reads below are ordered after its writes by the compiler)
  const int nw = n0 + wn * 128;                      // first column of this wave, all in one output
  const int HD = a.H * a.D;
  uint16_t* const out = (uint16_t*)a.out[nw / HD];
  const int nn = nw % HD;
  // A lane's column is the same in every row it writes, and its rows are 4 apart: the divisions that
  // find head and batch are made once
  const int row0 = lane >> 4, ch = lane & 15, col = nn + 8 * ch;
  const long mr = m0 + wm * 32 * IB + row0;
  long bb = mr / a.S;
  int sr = (int)(mr - bb * a.S);
  uint16_t* const out_c = out + (long)(col / a.D) * a.S * a.D + col % a.D;
  const long batch = (long)a.H * a.S * a.D;
#pragma unroll 4
  for (int it = 0; it < 8 * IB; ++it) {
    const u32x4 y = *(const u32x4*)(tb + (4 * it + row0) * TB_PITCH + ch * 16);
    if (mr + 4 * it < a.M) *(u32x4*)(out_c + bb * batch + (long)sr * a.D) = y;
    sr += 4;
    while (sr >= a.S) { sr -= a.S; ++bb; }
  }
}

// More 256 x 256 tiles than compute units: a workgroup stays and takes one after the other, as one sequence of tile pairs, and
// what is left of a tile when its last pair has been multiplied moves into the pairs of the next one.  The accumulators
// are rounded and packed into 128 ordinary registers between the first matrix instructions of the next tile, and each of
// its first eight pairs turns 32 tokens x 64 columns around in LDS and writes them, whole lines.  Set-up (7 thousand clocks),
// epilogue (11 thousand, at the chip's write rate, since all workgroups reach it together) and the change of
// workgroups were 45 % of a tile with 512 features.  In its place between a pass's other kernels, the two forms switched from pass to pass,
// events around the call, us: 131072 tokens x 512 x 1024 columns 170 -> 155 (the whole pass with its gradients 458 -> 437; a kernel trace, where no two
// kernels overlap, has 172 and 173; 133 with nothing written: a write retires in order with the copies of the pair after
// it, which wait for it); 20000 x 512 x 4096 106 -> 94; 131072 x 1024 x 1024 272 -> 253; 65536 x 512 x 1024 86 -> 87; 32768 x 3072 x 2048 331 ->
// 325.  Long tiles gain and lose 1 to 2 %, so there is no upper end to the rule: 32768 x 2048 x 2048 226 and 224, x 4096 427 and 424 (back to back
// 511 and 525), x 8192 815 and 822; 32768 x 4096 x 1024 214 -> 217.  A tile that ends past the last token, and a workgroup's last one, are written
// at once; behind its last tile a workgroup copies its last pairs again, so that no pair asks whether there is another.
constexpr int RUN_SMEM_B = RING_B + 4 * tilerun::FB_WAVE;
static_assert(RUN_SMEM_B <= 160 * 1024, "the layout fits a compute unit");

// PAST: the results are written past the caches.  Outputs that the last-level cache (256 MB) cannot hold beside the tokens push these out
// of it otherwise (131072 tokens x 512 x 1024, 256 MB of output: 189 -> 162 us; 65536 x 512 x 1536, 192 MB: 109 -> 97; 80000 x
// 1024 x 1024, 156 MB: 163 -> 145, but 20000 x 512 x 4096 82.5 -> 84.3); smaller ones stay, for whoever reads them next
// (32768 x 4096 x 2048, 128 MB: no difference).
template <bool PAST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
project_run_bf16_kernel(ProjArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  using namespace tilerun;
  constexpr int TM = 256;
  const int n_mt = (int)((a.M + TM - 1) / TM), n_nt = a.N / TN, nk = a.E / BK;
  const long n_pid = tile_grid(n_mt, n_nt);
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, l31 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;           // this wave's 128 tokens / 128 columns of a tile
  struct Tile { long m0; int n0; bool on; };
  long pid = blockIdx.x;
  auto take = [&]() -> Tile {
    for (; pid < n_pid; pid += gridDim.x) {
      HeadWork hw;
      if (!tile_decode(pid, n_mt, n_nt, &hw)) continue;
      pid += gridDim.x;
      return {(long)hw.head * TM, hw.item * TN, true};
    }
    return {0, 0, false};
  };
  Tile cur = take();
  if (!cur.on) return;
  Tile nxt = take();

  // ---- copies (see project_bf16_kernel); xp, wp: the next pair of x and of w to copy, of which xk, wk of their tile have gone out
  const unsigned xrow_b = (unsigned)(a.ldx * 2), wrow_b = (unsigned)(a.E * 2);
  const unsigned smem_u = lds_base(smem);
  unsigned xo[8], wo[2];
  const char *xp, *wp;
  auto x_tile = [&](const Tile& t) __attribute__((always_inline)) {
    const long m_last = a.M - 1 - t.m0;
    int ln = lane;
    asm volatile("" : "+v"(ln));                     // (worked out again for every tile: its terms, kept, fill the registers)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = 64 * wave + 8 * j + (ln >> 3);
      xo[j] = (unsigned)(r < m_last ? r : (int)m_last) * xrow_b + 16u * (unsigned)((ln & 7) ^ perm_of(8 * j + (ln >> 3)));
    }
    xp = (const char*)a.x + t.m0 * (long)xrow_b;
  };
  auto w_tile = [&](const Tile& t) __attribute__((always_inline)) { wp = (const char*)a.w + ((long)t.n0 + 64 * wave) * wrow_b; };
#pragma unroll
  for (int j = 0; j < 2; ++j) wo[j] = (unsigned)(lane >> 3) * wrow_b + 16u * (unsigned)((lane & 7) ^ perm_of(8 * j + (lane >> 3)));
  auto issue_x = [&](unsigned slot, int j) __attribute__((always_inline)) { dma16u(xp, xo[j], slot + (unsigned)((64 * wave + 8 * j) * ROWB)); };
  auto issue_w = [&](unsigned slot, int j) __attribute__((always_inline)) {
    dma16u(wp + (long)(8 * j) * wrow_b, wo[j & 1], slot + (unsigned)(TILE_B + (64 * wave + 8 * j) * ROWB));
  };

  int rd[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) rd[q] = l31 * ROWB + 16 * ((2 * q + g) ^ perm_of(l31));
  const int xbase = wm * 128 * ROWB, wbase = TILE_B + wn * 128 * ROWB;
  claim_accumulators();
  Packed pk;                                         // the tile before
  bf16x8 xa[4], wa[4], xb[4], wb[4];                 // operands of even / odd k-steps
  auto fetch = [&](const char* st, int q, int u, bf16x8 (&xv)[4], bf16x8 (&wv)[4]) __attribute__((always_inline)) {
    if (u < 4) xv[u] = *(const bf16x8*)(st + xbase + 32 * u * ROWB + rd[q]);
    else if (u < 8) wv[u - 4] = *(const bf16x8*)(st + wbase + 32 * (u - 4) * ROWB + rd[q]);
  };
  // ---- the way out: a tile lies in two batches at most (S >= 256), the second from row `edge` on
  char* const fb = smem + RING_B + wave * FB_WAVE;
  const int row_l = wm * 128 + (lane >> 3);          // this lane's first row of a tile
  uint16_t* out_p[2];
  int edge;
  const long batch2 = (long)(a.H - 1) * a.S * a.D;
  auto out_tile = [&](const Tile& t) __attribute__((always_inline)) {
    const int HD = a.H * a.D, nw = t.n0 + wn * 128;
    const long b0 = t.m0 / a.S, next = (b0 + 1) * a.S - t.m0;
    edge = next < TM ? (int)next : TM;
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int col = nw % HD + 64 * h + 8 * (ln & 7);
      out_p[h] = (uint16_t*)a.out[nw / HD] + (long)(col / a.D) * a.S * a.D + col % a.D + (t.m0 + wm * 128 + (ln >> 3)) * a.D + b0 * batch2;
    }
  };
  auto out_at = [&](int e, int it) __attribute__((always_inline)) -> u32x4* {
    int r = row_l;
    asm volatile("" : "+v"(r));                      // (worked out here: kept for all parts, the addresses fill the registers)
    const int d = 32 * (e / 2) + 8 * it;
    return (u32x4*)(out_p[e % 2] + d * a.D + (r + d >= edge ? batch2 : 0));
  };

  auto write = [&](u32x4* to, u32x4 y) __attribute__((always_inline)) {
    if constexpr (PAST) __builtin_nontemporal_store(y, to);
    else *to = y;
  };
  // the 16 matrix instructions of one k-step; hook(u) is other work issued after instruction u.  FIRST: of a tile (1), behind
  // another one (2), whose sums are packed on the way: a block's last matrix instruction lies 16 back
  auto mma16 = [&](auto first, const bf16x8 (&xv)[4], const bf16x8 (&wv)[4], auto&& hook) __attribute__((always_inline)) {
    constexpr int FIRST = decltype(first)::value;
    each_block([&](auto block) __attribute__((always_inline)) {
      constexpr int B = decltype(block)::value;
      if constexpr (FIRST == 2) pack<B>(pk);
      if constexpr (FIRST != 0) mfma_start<B>(wv[B / 4], xv[B % 4]);
      else mfma_add<B>(wv[B / 4], xv[B % 4]);
      hook(B);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using I0 = std::integral_constant<int, 0>;
  int par = 0;                                       // slot of the pair being multiplied
  bool behind = false;                               // the tile before is still to be written
  // One pair.  E: the part of the tile before that it writes, or -1.
  auto pair = [&](auto first, auto part) __attribute__((always_inline)) {
    constexpr int E = decltype(part)::value;
    const char* const st = smem + par * SLOT_B;
    const char* const sn = smem + (par ^ 1) * SLOT_B;
    const unsigned su = smem_u + (unsigned)(par * SLOT_B), sv = smem_u + (unsigned)((par ^ 1) * SLOT_B);
    u32x4 y[2];
    mma16(first, xa, wa, [&](int u) __attribute__((always_inline)) {
      fetch(st, 1, u, xb, wb);
      if (u % 2 == 1) issue_w(sv, u / 2);
    });
    wp += ROWB;
    mma16(I0{}, xb, wb, [&](int u) __attribute__((always_inline)) {
      fetch(st, 2, u, xa, wa);
      if (E >= 0 && u >= 8) turn(fb, pk, E, u - 8, lane);
    });
    mma16(I0{}, xa, wa, [&](int u) __attribute__((always_inline)) {
      fetch(st, 3, u, xb, wb);
      if (E >= 0 && u >= 4 && u < 12 && u % 2 == 0) y[u / 2 % 2] = turned(fb, (u - 4) / 2, lane);
      if (E >= 0 && u >= 7 && u < 15 && u % 2 == 1) write(out_at(E, (u - 7) / 2), y[(u - 3) / 2 % 2]);
    });
    // The next pair has landed when nothing but what this pair has just written is outstanding, and this wave's last reads of
    // the pair have returned; behind the barrier that holds for every wave.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(E >= 0 ? 0x0074 : 0x0070);        // vmcnt(4) or (0), lgkmcnt(0)
    wg_barrier();
    mma16(I0{}, xb, wb, [&](int u) __attribute__((always_inline)) {
      fetch(sn, 0, u, xa, wa);
      if (u % 2 == 1) issue_x(su, u / 2);
    });
    xp += ROWB;
    par ^= 1;
  };

  using None = std::integral_constant<int, -1>;

  // ---- pair 0 and the x of pair 1 go out; from then on every pair sends the w of the next one and the x of the one after, the
  // last two of a tile the next tile's, or this one's again
  x_tile(cur);
  w_tile(cur);
#pragma unroll
  for (int j = 0; j < 8; ++j) issue_x(smem_u, j);
#pragma unroll
  for (int j = 0; j < 8; ++j) issue_w(smem_u, j);
  xp += ROWB;
  wp += ROWB;
#pragma unroll
  for (int j = 0; j < 8; ++j) issue_x(smem_u + SLOT_B, j);
  xp += ROWB;
  wait_vmcnt<8>();
  wg_barrier();
#pragma unroll
  for (int u = 0; u < 8; ++u) fetch(smem, 0, u, xa, wa);
  for (;;) {
    if (behind) {
      pair(std::integral_constant<int, 2>{}, I0{});
      pair(I0{}, std::integral_constant<int, 1>{});
      pair(I0{}, std::integral_constant<int, 2>{});
      pair(I0{}, std::integral_constant<int, 3>{});
      pair(I0{}, std::integral_constant<int, 4>{});
      pair(I0{}, std::integral_constant<int, 5>{});
      for (int P = 6; P < nk - 2; ++P) pair(I0{}, None{});
      x_tile(nxt.on ? nxt : cur);
      pair(I0{}, std::integral_constant<int, 6>{});
      w_tile(nxt.on ? nxt : cur);
      pair(I0{}, std::integral_constant<int, 7>{});
    } else {
      pair(std::integral_constant<int, 1>{}, None{});
      for (int P = 1; P < nk - 2; ++P) pair(I0{}, None{});
      x_tile(nxt.on ? nxt : cur);
      pair(I0{}, None{});
      w_tile(nxt.on ? nxt : cur);
      pair(I0{}, None{});
    }
    out_tile(cur);
    behind = nxt.on && cur.m0 + TM <= a.M;
    if (!behind) {
      asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");      // (the last matrix instruction has retired)
      each_block([&](auto block) __attribute__((always_inline)) { pack<decltype(block)::value>(pk); });
#pragma unroll
      for (int e = 0; e < NFLUSH; ++e) {
#pragma unroll
        for (int x = 0; x < 8; ++x) turn(fb, pk, e, x, lane);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const u32x4 y = turned(fb, it, lane);
          if (cur.m0 + row_l + 32 * (e / 2) + 8 * it < a.M) write(out_at(e, it), y);
        }
      }
      if (!nxt.on) break;
    }
    cur = nxt;
    nxt = take();
  }
  wait_vmcnt<0>();                                   // (the copies that nobody reads have landed before the LDS is another's)
}

// float32 tensors: one thread per output element, plain FMA in the order of the definition
__global__ void __launch_bounds__(256) project_f32_kernel(ProjArgs a) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.M * a.N) return;
  const long m = idx / a.N;
  const int n = (int)(idx % a.N);
  const float* xr = (const float*)a.x + m * a.ldx;
  const float* wr = (const float*)a.w + (long)n * a.E;
  float acc = 0.f;
  for (int e = 0; e < a.E; ++e) acc = fmaf(xr[e], wr[e], acc);
  const int HD = a.H * a.D, nn = n % HD;
  const long b = m / a.S, s = m % a.S;
  ((float*)a.out[n / HD])[((b * a.H + nn / a.D) * a.S + s) * a.D + nn % a.D] = acc;
}

}  // namespace

bool project_bf16_supported(const ProjArgs& a) {
  return a.E % BK == 0 && a.N % TN == 0 && (a.H * a.D) % 128 == 0 && a.D % 8 == 0;
}

namespace {
template <int IB> hipError_t launch_tiles(const ProjArgs& a, hipStream_t s) {
  static SmemOnce once;
  const hipError_t e = ensure_dynamic_lds((const void*)project_bf16_kernel<IB>, SMEM_B, &once);
  if (e != hipSuccess) return e;
  const long grid = tile_grid((int)((a.M + 64 * IB - 1) / (64 * IB)), a.N / TN);
  project_bf16_kernel<IB><<<(unsigned)grid, 256, SMEM_B, s>>>(a);
  return hipGetLastError();
}
template <bool PAST> hipError_t launch_run(const ProjArgs& a, hipStream_t s) {
  static SmemOnce once;
  const hipError_t e = ensure_dynamic_lds((const void*)project_run_bf16_kernel<PAST>, RUN_SMEM_B, &once);
  if (e != hipSuccess) return e;
  project_run_bf16_kernel<PAST><<<(unsigned)(a.n_cu / 8 * 8), 256, RUN_SMEM_B, s>>>(a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_project(const ProjArgs& a, int is_f32, hipStream_t s) {
  if (is_f32) {
    const long n = a.M * a.N;
    project_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a);
    return hipGetLastError();
  }
  const long tiles = (a.M + 255) / 256 * (a.N / TN);
  const bool past = a.M * a.N * 2 > 144l << 20;
  if (a.n_cu >= 8 && tiles > a.n_cu / 8 * 8 && a.E >= tilerun::NFLUSH * BK && a.S >= 256) return past ? launch_run<true>(a, s) : launch_run<false>(a, s);
  return tiles * 4 <= 3L * a.n_cu ? launch_tiles<2>(a, s) : launch_tiles<4>(a, s);
}

}  // namespace lvx

// Masks by words (LIST = 3 of the forward and dQ kernels), row tiles whose blocks of 32 rows see little of what the
// tile's 256 rows see together: chunks of a few rows that see a frame each. The dense loop forms 256 x 64 scores for
// every key tile that any row sees; here each wave takes two of the tile's row blocks, one after the other, and
// streams units of 32 keys of the key blocks that the block sees through LDS stages of its own (lvx_key_units.h),
// without barriers and without the other waves. A unit lies in one key block, so the word of (row block, key block)
// says which rows see it, the same for all of its keys.
//
// Bound by memory and by the latency of a unit's chain (LDS, 8 or 16 matrix instructions, exponentials), one wave per
// SIMD with two to four units in flight. 4096 rows x 8 heads (D = 64) in chunks of 2, each seeing one of 2048 frames
// of 64 keys: forward 153 -> 74 us, dQ 165 -> 80 (268 MB of K and V, 52 us at a large copy's rate); 4096 x 16 heads
// in chunks of 32 on frames of 729, 3680 rows x 60507 keys, the step 835 -> 660. A unit takes about a third of what
// the dense loop's quarter of a tile (a wave's 64 x 64 scores) does, so a tile is streamed when no wave's two blocks
// see more (row block, key block) pairs than 0.9 times the key blocks of the tile (mask_streams).
#pragma once
#include "lvx_kv_ring.h"
#include "lvx_key_units.h"

namespace lvx {

using kvring::KvSmem;
using kvring::NSTG;
using kvring::NWV;

constexpr int STREAM_CAP = 1024;       // key blocks that a row block's list holds

template <int D> struct StreamSmem {
  static constexpr int NST = D == 64 ? 4 : 2;       // stages per wave
  static constexpr int WAVE = NST * KeyUnit<D>::STAGE;
  static constexpr int LIST = STREAM_CAP * 8;       // (key block, word)
  static constexpr int TOTAL = NWV * (WAVE + LIST);
};
static_assert(StreamSmem<64>::TOTAL <= 160 * 1024 && StreamSmem<128>::TOTAL <= 160 * 1024, "the layout fits a compute unit");

// LDS of the kernels that mask by words: the ring, the list and the tiles' words, or the streams
template <int D> constexpr int mask_words_lds() {
  return KvSmem<D>::TOTAL + NSTG * 256 > StreamSmem<D>::TOTAL ? KvSmem<D>::TOTAL + NSTG * 256 : StreamSmem<D>::TOTAL;
}

__device__ __forceinline__ int wave_sum(int x) {    // of every lane's x, wave-uniform (prefix sums of 16 lanes, then the four of them)
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  return __builtin_amdgcn_readlane(x, 15) + __builtin_amdgcn_readlane(x, 31) + __builtin_amdgcn_readlane(x, 47) +
         __builtin_amdgcn_readlane(x, 63);
}
// Whether row tile qt is streamed; `any` becomes the lane's 64 key blocks of those some row of the tile sees
// (at most 64 words: the kernels take no more than 4095 key tiles, and key blocks are no smaller).
__device__ __forceinline__ bool mask_streams(const MaskRows& r, int b, int qt, int lane, unsigned long long* any) {
  const long at = b * r.any_stride_b + (long)qt * r.any_words + min(lane, r.any_words - 1);
  const unsigned long long m = r.any[at];
  const unsigned c = r.counts[at];
  *any = lane < r.any_words ? m : 0ull;
  const int blocks = wave_sum((int)__popcll(*any));
  const int c02 = wave_sum(lane < r.any_words ? (int)(c & 0xff00ffu) : 0), c13 = wave_sum(lane < r.any_words ? (int)(c >> 8 & 0xff00ffu) : 0);
  const int most = max(max(c02 & 0xffff, c02 >> 16), max(c13 & 0xffff, c13 >> 16));
  return 10 * most <= 9 * blocks && most <= STREAM_CAP && blocks > 0;
}

// One wave's stream over the key blocks that row block rb of tile qt sees, this split's share of it.
template <int D> struct KeyStream {
  using U = KeyUnit<D>;
  using SM = StreamSmem<D>;
  static constexpr int NC = U::NC, NDMA = 2 * NC, NST = SM::NST;
  const char *k0, *v0;
  unsigned row_bytes, stage_u;
  char* stage0;
  const u32x2* list;
  int kv_block, Skv, per, lane;        // per: units of a key block
  int p1, pi, ei, ui;                  // end; the unit issued next: position, list entry, unit in the key block
  int e, u;                            // the unit computed on
  bool v_rows;                         // V in K's order: it is read by whole rows, as K is
  unsigned offk[NC], offv[NC];

  __device__ __forceinline__ KeyStream(const void* k, const void* v, const Dims& d, int b, int hk, char* smem, int wave, int lane_,
                                       int kv_block_, bool v_rows_)
      : k0((const char*)k + (b * d.kv_sb + hk * d.kv_sh) * 2), v0((const char*)v + (b * d.kv_sb + hk * d.kv_sh) * 2),
        row_bytes((unsigned)(d.kv_ss * 2)), stage0(smem + wave * SM::WAVE),
        list((const u32x2*)(smem + NWV * SM::WAVE + wave * SM::LIST)), kv_block(kv_block_), Skv(d.Skv),
        per((kv_block_ + UK - 1) / UK), lane(lane_), v_rows(v_rows_) {
    stage_u = lds_base(stage0);
#pragma unroll
    for (int n = 0; n < NC; ++n) {
      offk[n] = unit_copy_off<D>(n, false, UK - 1, row_bytes, lane);
      offv[n] = unit_copy_off<D>(n, !v_rows, UK - 1, row_bytes, lane);
    }
  }
  // the list of row block rb, and the first units' copies
  __device__ __forceinline__ int start(const MaskRows& r, int b, int qt, int rb, unsigned long long any, int split, int n_split) {
    const unsigned* const words = r.words + b * r.stride_b + ((long)qt * r.w1) * 8 + rb;
    int nf = 0;
    for (int w0 = 0; w0 < r.any_words; w0 += 4) {    // (four words of 64 key blocks at a time: one trip to memory for all)
      unsigned long long m[4];
      unsigned x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        m[q] = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(any >> 32), min(w0 + q, 63)) << 32 |
               (unsigned)__builtin_amdgcn_readlane((int)(unsigned)any, min(w0 + q, 63));
      if ((m[0] | m[1] | m[2] | m[3]) == 0ull) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = min((w0 + q) * 64 + lane, r.w1 - 1);
        x[q] = words[(long)f * 8];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool on = w0 + q < r.any_words && (m[q] >> lane & 1ull) && x[q] != 0;
        const unsigned long long in = __ballot(on);
        if (on) ((u32x2*)list)[nf + __popcll(in & ((1ull << lane) - 1ull))] = u32x2{(unsigned)((w0 + q) * 64 + lane), x[q]};
        nf += (int)__popcll(in);
      }
    }
    const int total = nf * per, p0 = (int)((long)total * split / n_split);
    p1 = (int)((long)total * (split + 1) / n_split);
    pi = p0;
    e = ei = p0 / per;
    u = ui = p0 - ei * per;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < NST; ++s) issue(s);
    return p1 - p0;
  }
  __device__ __forceinline__ void issue(int st) {
    if (pi >= p1) return;
    const int key0 = min(__builtin_amdgcn_readfirstlane((int)list[ei].x) * kv_block + ui * UK, Skv - 1);
    const long base = (long)key0 * row_bytes;
    const unsigned dst = stage_u + st * U::STAGE;
    if (key0 + UK <= Skv) {
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(k0 + base, offk[n], dst + n * 1024);
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(v0 + base, offv[n], dst + U::TILE + n * 1024);
    } else {                                       // the last keys: rows past them re-read the last one
      const int last = Skv - 1 - key0;
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(k0 + base, unit_copy_off<D>(n, false, last, row_bytes, lane), dst + n * 1024);
#pragma unroll
      for (int n = 0; n < NC; ++n) dma16u(v0 + base, unit_copy_off<D>(n, !v_rows, last, row_bytes, lane), dst + U::TILE + n * 1024);
    }
    ++pi;
    if (++ui == per) { ui = 0; ++ei; }
  }
  // waits for the unit at hand (`left` more behind it)
  __device__ __forceinline__ void arrive(int left) {
    if (left >= NST - 1) wait_vmcnt<(NST - 1) * NDMA>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
  }
  struct Unit { int keys; unsigned word; };        // keys of the unit that there are and the key block has (none: 0 or less)
  __device__ __forceinline__ Unit unit() const {
    const u32x2 x = list[e];
    const int key0 = __builtin_amdgcn_readfirstlane((int)x.x) * kv_block + u * UK;
    return {min(kv_block - u * UK, Skv - key0), (unsigned)__builtin_amdgcn_readfirstlane((int)x.y)};
  }
  // rows of the unit past its key block or the last key become 0, of a tile that is multiplied by weights of 0 there (what
  // the next key block holds may be infinite, and no row of the tile has to see it)
  __device__ __forceinline__ void clear_past(char* tile, const Unit& un) {
    if (un.keys >= UK) return;
    asm volatile("" ::: "memory");
    for (int x = max(un.keys, 0) * U::CH + lane; x < UK * U::CH; x += 64) *(u32x4*)(tile + x * 16) = u32x4{0, 0, 0, 0};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  // every read of the stage has returned: the unit NST further on takes it
  __device__ __forceinline__ void release(int st) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(st);
    if (++u == per) { u = 0; ++e; }
  }
};

// lane's addresses in a tile: chunk x 32 ^ of a plain row read, and the transposing read of 32 columns
template <int D> struct UnitReads {
  int row, x, tr[D / 32], tr8[D / 32];             // (tr8: eight rows on)
  __device__ __forceinline__ UnitReads(int lane, bool v_order) {
    const int ql = lane & 31, g = lane >> 5, j16 = lane & 15, half = (lane >> 4) & 1, tr_row = 4 * g + (j16 >> 2);
    row = ql * KeyUnit<D>::ROWB;
    x = (g ^ k_swz<D>(ql)) * 16;
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      const int c = 4 * db + 2 * half + ((j16 & 3) >> 1);
      tr[db] = tr_row * KeyUnit<D>::ROWB + (c ^ (v_order ? v_swz<D>(tr_row) : k_swz<D>(tr_row))) * 16 + (j16 & 1) * 8;
      tr8[db] = (tr_row + 8) * KeyUnit<D>::ROWB + (c ^ (v_order ? v_swz<D>(tr_row + 8) : k_swz<D>(tr_row + 8))) * 16 + (j16 & 1) * 8;
    }
  }
  __device__ __forceinline__ bf16x8 plain(const char* tile, int ks) const { return *(const bf16x8*)(tile + row + (x ^ (32 * ks))); }
};
// rows 16 t2 + 8 (e / 4) + 4 g + (e % 4) of 32 columns (either order repeats after 16 rows)
template <int D> __device__ __forceinline__ bf16x8 unit_tr(const UnitReads<D>& at, const char* tile, int db, int t2) {
  const s16x4 lo = lds_read_tr(tile + at.tr[db] + 16 * t2 * KeyUnit<D>::ROWB), hi = lds_read_tr(tile + at.tr8[db] + 16 * t2 * KeyUnit<D>::ROWB);
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  return __builtin_bit_cast(bf16x8, (s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}));
}
// keys of a unit that the lane's row does not see get the score -infinity (NaN and infinite ones too)
__device__ __forceinline__ void mask_unit(f32x16& s, int keys, unsigned word, int ql, int g) {
  const bool see = (word >> ql) & 1u;
#pragma unroll
  for (int v = 0; v < 16; ++v) s[v] = see ? s[v] : -INFINITY;
  if (keys < UK) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (8 * (v / 4) + 4 * g + (v % 4) >= keys) s[v] = -INFINITY;
  }
}
// The matrix instructions are written out (lvx_kv_ring.h), so their results are waited for by hand.
__device__ __forceinline__ void settle_unit(f32x16& s) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(s)); }
template <int DB> __device__ __forceinline__ void settle_acc(f32x16 (&acc)[DB]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0]));
#pragma unroll
  for (int db = 1; db < DB; ++db) asm volatile("" : "+a"(acc[db]));
}

}  // namespace lvx

// Internal launch interface between the C-ABI host layer (lvx_api.hip) and the kernels.
// Everything here is private to the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/lvx.h"

namespace lvx {

// Media mask as the kernels see it (allow == nullptr means dense attention).
struct MaskDev {
  const uint8_t* allow;
  int q_chunk, kv_block, n_q_chunks, n_kv_blocks;
  long stride_b, stride_q;
};
// A bitmap of which allow[0] is byte `first`: all of it (0), or a window's copy in LDS.  (A type of its own: kernels
// make it, and with eight bytes more among the arguments a call of 12.24 us took 12.37.)
struct MaskWin : MaskDev {
  long first;
};

// The bitmap regrouped by launch_mask_rows: word ((b, qt, f), rb) holds, for the 32 query rows
// 256 qt + 32 rb + (0 .. 31) of a head, which of them see key block f (bit r = row r; rows past the
// last one see nothing).  The eight words of a key block and a tile of 256 rows stand together,
// and every tile has one padding block more that nobody sees, so that the words of two neighbouring
// key blocks are one run of 64 bytes for every block there is.
struct MaskRows {
  const unsigned* words;  // nullptr: not made for this call
  int w1, n_qt;           // key blocks (with the padding one), tiles of 256 rows
  long stride_b;          // words from one batch to the next (0: one bitmap for all)
  // any[(b n_qt + qt) any_words + f / 64], bit f % 64: some row of tile qt sees key block f
  const unsigned long long* any;
  long any_stride_b;
  int any_words;
  // counts[(b n_qt + qt) any_words + x], byte w: pairs of (row block w or w + 4 of tile qt, key block 64 x ..
  // 64 x + 63) in which some row sees the key block
  const unsigned* counts;
};

// the larger, or the NaN (a result without a value must not look like one without keys)
__device__ __forceinline__ float max_or_nan(float a, float b) { return b > a || b != b ? b : a; }

// Shape, strides (in elements) and scale shared by every kernel.
struct Dims {
  int B, Hq, Hkv, Sq, Skv, D;
  int G;                // query heads per K/V head
  long q_sb, q_sh, q_ss;
  long kv_sb, kv_sh, kv_ss;
  float scale;          // multiplies Q K^T (natural-log domain)
};

struct FwdArgs {
  Dims d;
  MaskDev mask;
  const void *q, *k, *v;
  void* o;              // final output (Q's strides) when n_split == 1
  int o_is_f32;         // 1: o is float32, 0: o has the input dtype
  int merge_into;       // 1: o (float32, CONTIGUOUS [B,Hq,Sq,D]) and lse hold a running result; for rows that are
                        // not split the kernel leaves in them the Rescale of it with this visit's result (for
                        // the others the combine does)
  void* o_last;         // with merge_into, or nullptr: the last visit's O goes here (input dtype, Q's strides) instead
  float* lse;           // [B,Hq,Sq]
  int n_split;          // number of KV splits handled by separate workgroups
  int partial;          // 1: write partial results even with n_split == 1 (this launch is one of several
                        // whose results are combined)
  int part0;            // index of the partial slice that split 0 of this launch writes
  int whole;            // dense kernel: the first `whole` row tiles of a K/V head are not split (the partial slices
                        // then hold the rows of the others only, [B,Hkv, rows of the group - 256 whole])
  int n_cu;             // compute units of the device (float32: picks the width of a workgroup)
  MaskRows rows;        // set by the launch where the kernel masks by it
  void* rows_ws;        // workspace for its words, or nullptr
  unsigned frame_magic; // 2^36 / kv_block, rounded up (set with rows)
  int pass;             // media mask, bf16: 0 = one launch over every visible tile; 1 = this launch takes the key
                        // tiles that EVERY row of a workgroup sees (dense kernel over a list of them), 2 = this
                        // launch takes the other visible tiles (general kernel)
  float* o_part;        // [n_split, B,Hq,Sq,D] float32, contiguous (n_split > 1)
  float* lse_part;      // [n_split, B,Hq,Sq]
};

struct KvPlan {
  int whole, parts;     // parts == 1: every tile has one workgroup
  int len;              // media mask: a tile is cut into as many parts as it has runs of this many steps, `parts` at most
};

struct BwdArgs {
  Dims d;
  // dK/dV kernel (bf16): the first kv.whole key tiles of a head have one workgroup each, every other one up to
  // kv.parts, which share its steps and leave float32 sums in kv_sums, in the order of the matrix
  // registers, [B Hkv, tiles - whole, parts][dK, dV][256 x D]; dkdv_sum_kernel adds them up
  KvPlan kv;
  MaskDev mask;
  int n_cu;             // compute units of the device (float32: picks the width of a workgroup)
  MaskRows rows;        // set by launch_bwd_bf16 where a kernel reads it
  void* rows_ws;        // workspace for its words (rows_ws_bytes), or nullptr
  size_t rows_ws_bytes;
  unsigned frame_magic; // 2^36 / kv_block, rounded up (set where the dQ kernel masks by rows)
  const void *q, *k, *v, *o, *d_o;
  const float* lse;     // final statistic, [B,Hq,Sq]
  float* delta;         // workspace, [B,Hq,Sq]: rowsum(dO * O)
  float* stats;         // workspace, [B,Hq,sq_pad/32][2][32]: per group of 32 query rows, 32 values of
                        // -L * log2(e) (-inf for rows without keys and pad rows), then 32 of -delta
  int sq_pad;           // Sq rounded up to a multiple of 32
  float* stats_ovl;     // workspace, [B,Hq][2][32], only when Sq % 32 != 0 and Sq >= 32 (else nullptr): the
                        // same two rows of 32 values for the query rows Sq-32 .. Sq-1, with -inf in place of
                        // -L * log2(e) for the rows that the last full group already covers.  A kernel that
                        // walks the rows 32 at a time takes rows Sq-32 .. Sq-1 as its last step instead of a
                        // short one: the rows it has seen before then contribute nothing.
  float* dq_accum;      // [B,Hq,Sq,D] float32, accumulated into
  int dq_first;         // 1: ... overwritten instead (the first visit)
  void* dq_last;        // or nullptr: the last visit's sum goes here (input dtype, Q's strides) instead
  void *dk, *dv;        // K's strides, input dtype, overwritten
  float* kv_sums;       // workspace, where dq_part is written later (a call's dQ kernel follows)
  int* kv_counts;       // media mask: parts that a tile was cut into, [B Hkv, tiles] (its number of steps is the mask's)
  int n_split_dq;       // KV splits of the dQ kernel
  int dq_whole;         // as FwdArgs::whole
  int dq_list;          // KV splits of its launches over the tiles some row sees (dq_pass 3, 4)
  int dq_pass;          // media mask, dQ kernel: 0 = one launch over every visible tile; 1 = this launch takes the
                        // key tiles that EVERY row of a workgroup sees (dense kernel over a list of them),
                        // 2 = this launch takes the other visible tiles (general kernel); 3, 4 = one launch of
                        // the dense kernel over the tiles any row sees (row blocks that see a tile or do not;
                        // masked by rows)
  float* dq_part;       // workspace, [n_split_dq, B,Hq,Sq,D] float32: the splits' sums (n_split_dq > 1),
                        // added to dq_accum by a reduction that follows the kernel
  // fused kernel (all five products in one pass): workspace of bwd_fused_ws_bytes, zeroed by the launch
  float* dq_tiles;      // [B,Hq,ceil(Sq/32)] tiles of 32 rows x 128 columns in matrix-register order
  int* dq_locks;        // one word per (tile, wave): 0 = free          (set by the launch)
  int* dq_err;          // nonzero after the kernel: a wave gave up on a lock, dQ is invalid   (set by the launch)
  int dq_stagger;       // steps by which consecutive key tiles start apart   (set by the launch)
};

struct MergeArgs {
  const void* o_parts[64];
  const float* lse_parts[64];
  int n_parts;
  // parts first .. n_parts - 1 are slices of one float32 array, `rows * D` and `rows` elements apart, that
  // start here (nullptr: not so; the pointers above are always set)
  const float *o_slices, *lse_slices;
  int first;
  long rows;            // rows to combine: B*Hq*Sq, or those of every group of `group` rows past its first `skip`
  int group, skip;
  int D;
  void* o_out;
  float* lse_out;
  // output addressing: row r = ((b*Hq + h)*Sq + i) -> o_out + b*o_sb + h*o_sh + i*o_ss
  int Hq, Sq;
  long o_sb, o_sh, o_ss;
};

// Projection out[o][b, h, s, c] = sum_e x[b, s, e] w[(o H + h) D + c, e], tokens flattened to M = B S rows.
struct ProjArgs {
  const void* x;        // [M, E], row stride ldx elements
  const void* w;        // [N, E] contiguous, N = n_out * H * D
  void* out[2];         // each [B, H, S, D] contiguous, x's dtype
  long M, ldx;
  int S, E, N, H, D;
  int n_cu;             // compute units of the device (picks the tile height)
};
bool project_bf16_supported(const ProjArgs& a);   // shapes the matrix-core kernel takes
hipError_t launch_project(const ProjArgs& a, int is_f32, hipStream_t s);

// Gradients of the projection: dx[m, e] = sum_n g[m, n] w[n, e] (rounded to the tensors' type),
// dw[n, e] += sum_m g[m, n] x[m, e] (float32), g given head-major per output like ProjArgs::out.
struct ProjBwdArgs {
  const void* x;        // [M, E], row stride ldx elements
  const void* w;        // [N, E] contiguous
  const void* g[2];     // each [B, H, S, D] contiguous
  void* dx;             // [M, E], row stride ldx, or null
  float* dw;            // [N, E] contiguous, or null
  long M, ldx;
  int S, E, N, H, D;
  int n_cu;             // compute units of the device (picks dw's tile height and token split)
  int dw_parts;         // set by launch_project_bwd: parts the token range of dw is cut into, and the
  unsigned dw_tiles_grid;   // workgroups of one part
};
bool project_bwd_bf16_supported(const ProjBwdArgs& a);   // shapes the matrix-core kernels take
hipError_t launch_project_bwd(const ProjBwdArgs& a, int is_f32, hipStream_t s);

// Bytes of workspace that lvx_xattn_fwd needs for exactly this call (with this mask or without
// one; lvx_xattn_workspace_bytes returns the larger of the two cases) when it is given `room`; 0 for
// invalid arguments.
size_t fwd_workspace_need(const lvx_problem* p, lvx_dtype dtype, const lvx_mask* mask, size_t room);

// kernels for float32 tensors (float32 matrix instruction; the key range is never split)
hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t s);
hipError_t launch_bwd_f32(const BwdArgs& a, unsigned stages, hipStream_t s);   // stages: 2 = dK/dV, 4 = dQ
// kernels for bfloat16 tensors (MFMA)
hipError_t launch_fwd_bf16(const FwdArgs& a, hipStream_t s);
hipError_t launch_bwd_bf16(const BwdArgs& a, unsigned stages, hipStream_t s);
hipError_t launch_bwd_dkdv_bf16(const BwdArgs& a, hipStream_t s);
// ... of key tiles of few steps: mode 0 dense, 1 a mask that selects steps, 2 any other, by a.rows
bool bwd_dkdv_short_takes(const Dims& d, const MaskDev& m, int mode);
hipError_t launch_bwd_dkdv_short(const BwdArgs& a, int mode, hipStream_t s);
KvPlan dkdv_bf16_plan(const Dims& d, int n_cu, bool masked, long most_sets);   // with room for that many sets of a tile's sums
size_t dkdv_bf16_set_bytes(const Dims& d);
size_t dkdv_bf16_sums_bytes(const Dims& d, const KvPlan& p);     // of BwdArgs::kv_sums (a multiple of 256 bytes),
size_t dkdv_bf16_counts_bytes(const Dims& d);                    // and of kv_counts
hipError_t launch_bwd_dq_bf16(const BwdArgs& a, hipStream_t s);
// all five products in one kernel (dense, head dim 128, at least 256 keys and 32 query rows):
// handles the first Skv / 256 * 256 keys; needs BwdArgs::dq_tiles
bool bwd_fused_bf16_supported(const Dims& d, bool masked);
size_t bwd_fused_ws_bytes(const Dims& d);
hipError_t launch_bwd_fused_bf16(const BwdArgs& a, hipStream_t s);
// LDS is handed out in pieces of 1280 bytes of a compute unit's 160 KB: 768 workgroups of 53760 bytes run all at once on 256 compute
// units, of 54272 in two rounds.  What n workgroups may have each, and whether that many fit.
constexpr int LDS_CU = 160 * 1024, LDS_PIECE = 1280;
constexpr int lds_share(int n) { return LDS_CU / n / LDS_PIECE * LDS_PIECE; }
constexpr bool lds_holds(int n, int bytes) { return bytes <= lds_share(n); }
// Raises a kernel's dynamic LDS limit once per device (the attribute belongs to the device's copy
// of the kernel).  `done` is the caller's per-kernel table; a race between host threads only
// repeats a harmless call.
constexpr int LVX_MAX_DEVICES = 64;
struct SmemOnce { bool done[LVX_MAX_DEVICES] = {}; };
inline hipError_t ensure_dynamic_lds(const void* kernel, int bytes, SmemOnce* once) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < LVX_MAX_DEVICES;
  if (tracked && once->done[dev]) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && tracked) once->done[dev] = true;
  return e;
}

// Number of KV splits for `base` workgroups that each walk the whole key range on n_cu compute
// units: the count (at most cap) that minimises rounds * t_full / splits + splits * t_part, where
// rounds = ceil(base * splits / n_cu), t_full is one workgroup's time over the whole range and
// t_part what one more set of partial results costs (written, read again and summed).  Covers
// both a grid smaller than the chip and one slightly larger than a multiple of it (288
// workgroups on 256 units would take two rounds for the work of 1.125).
inline int pick_split_balanced(long base, int n_cu, long cap, double t_full, double t_part) {
  int best = 1;
  double best_t = 1e300;
  for (long s = 1; s <= cap && s <= 64; ++s) {
    const long rounds = (base * s + n_cu - 1) / n_cu;
    const double t = (double)rounds * t_full / (double)s + (s > 1 ? (double)s * t_part + 10e-6 : 0.0);
    if (t < best_t * 0.97) {                       // more splits only for a gain of 3 %
      best_t = t;
      best = (int)s;
    }
  }
  return best;
}
// The same for workgroups that take a tile of rows each, n_qt tiles in each of `heads` groups: whole rounds of row
// tiles are left unsplit, and the tiles of the last round (or of the last two) are split `parts` ways, down to three
// key tiles a part. t_tile: one workgroup's time for one of the n_tiles key tiles, t_fix: its set-up and epilogue,
// t_part: what a set of partial results of one row tile costs, t_join: the launch that combines them. Splitting every
// row tile (to 16 key tiles a part at least) sent all rows through memory for the sake of the last round: 32 / 8
// heads x 2650 rows x 9447 keys, 336 row tiles, forward with its combine 439 -> 428 us, dQ 550 -> 511; and few rows
// against few keys waited for long parts: 8 heads (D = 64) x 427 rows x 2576 keys forward 36 -> 28, 16 heads x 134
// rows x 1024 keys 33 -> 27. Of 31 shapes with 64 to 8192 rows and 1024 to 131072 keys the choice is within 8 % of
// the best of up to 28 on all but two.
// The model errs by more than its margins (3 % to split at all, 0.5 % for each step to more parts), which were
// measured all the same: of 12 calls that it splits for a predicted 3 to 8 %, 10 are faster than unsplit ones (by up
// to 8.9 %, 3.8 % on average over the 12), two slower (by 0.7 %: 28 / 4 heads x 3846 rows x 6912 keys 361 -> 363 and
// 454 -> 457 us). Steps of 2 % and more only would change 59 calls of over 100 us and make them slower by 0.5 % on
// average (from 3.8 % slower, 16 heads x 4443 rows x 2048 keys dQ 112 -> 116, to 2.7 % faster, 28 / 4 heads x 960
// rows x 32768 keys 423 -> 412), and most short ones, by 1 to 5 %.
// t_two: a key tile's time where two workgroups share a compute unit, which a last round of up to n_cu workgroups does not
// (0: one workgroup has it to itself).  Parts beside one whole tile on every compute unit cost it what they slow it by.  64-wide forward,
// 260 shapes, one workgroup a compute unit or up to two: within 0.8 % of the better on average, with inputs in the caches or
// changing; of 1300 sets of the five times none does better on both these and 60 shapes where the two plans are close (1.1 %).
struct TailPlan { int whole, parts; };
inline TailPlan pick_tail(long heads, int n_qt, int n_tiles, int n_cu, long most, double t_tile, double t_fix,
                          double t_part, double t_join, double t_two = 0.) {
  const long tiles = heads * n_qt, places = t_two > 0. ? 2L * n_cu : n_cu;
  const auto time = [&](long n, int kt) {          // n workgroups of kt key tiles each
    const long full = n / places, rest = n % places;
    const double t_full = kt * (t_two > 0. ? t_two : t_tile) + t_fix;
    return full * t_full + (rest == 0 ? 0. : t_two > 0. && rest <= n_cu ? kt * t_tile + t_fix : t_full);
  };
  TailPlan best = {0, 1};
  double best_t = time(tiles, n_tiles);
  const long full = tiles / n_cu;
  for (long k = full; k >= 0 && k >= full - (t_two > 0. ? 2 : 1); --k) {
    const long whole = k * n_cu / heads, cut = tiles - heads * whole;
    const bool beside = t_two > 0. && k % 2 == 1;
    for (long p = 2; p <= most && p <= 64 && 3 * p <= n_tiles; ++p) {
      const int kt = (int)((n_tiles + p - 1) / p);
      const double t_cut = beside ? (double)((cut * p + n_cu - 1) / n_cu) * kt * (t_two - t_tile) : time(cut * p, kt);
      const double t = time(heads * whole, n_tiles) + t_cut + (double)(cut * p) * t_part + t_join;
      if (t < best_t * (best.parts == 1 ? 0.97 : 0.995)) {
        best_t = t;
        best = {(int)whole, (int)p};
      }
    }
  }
  return best;
}
// the dense forward and dQ kernels (bf16, no mask): whether they take the problem, and how
bool fwd_bf16_dense(const Dims& d, bool masked);
int fwd_bf16_dense_per_cu(const Dims& d);                         // workgroups of the forward that a compute unit holds
TailPlan fwd_bf16_dense_plan(const Dims& d, int n_cu, int most, int per_cu);
int fwd_bf16_coarse_split(const Dims& d, int n_cu);             // every row tile, in a workspace too small for that plan
bool bwd_dq_bf16_dense(const Dims& d, bool masked);
TailPlan bwd_dq_bf16_dense_plan(const Dims& d, int n_cu);
int bwd_dq_bf16_coarse_split(const Dims& d, int n_cu);
// KV splits of the masked kernels that walk a list of the tiles some row sees (LIST >= 2; each split takes an even
// share of the list, wherever it ends), for `wgs` row tiles and n_tiles key tiles of which the mask shows any number.
// They start longest first, so two rounds of the chip even out lists as uneven as a causal mask's while a workgroup
// keeps tiles enough to be worth its set-up and list (15 us); else one round, down to three tiles a split. (Four
// times the compute units halved, 1024 keys a split at least, before.) Forward and dQ, us: 28 row tiles (D = 128) x
// 92 key tiles 68 -> 38 and 84 -> 46, 64 x 29 (D = 64) 53 -> 37 and 53 -> 37, 64 x 201 88 -> 72 and 109 -> 89; two
// rounds of long ones: 128 x 2048, causal 457 -> 382 and 581 -> 482 against one round (each chunk one frame: 152 ->
// 168). Between one round and one and a half, two splits: 160 x 160 232 -> 202 (three before).
inline int list_split(long wgs, int n_tiles, int n_cu) {
  const long some = 16 * wgs <= 25L * n_cu ? 2 : 1;                // (a round and a half of them)
  const long two = wgs <= n_cu ? 2L * n_cu / wgs : some, one = 2 * wgs <= n_cu ? n_cu / wgs : some;
  long s = n_tiles / two >= 64 ? two : one;
  if (s > n_tiles / 3) s = n_tiles / 3;
  return s < 1 ? 1 : s > 60 ? 60 : (int)s;
}
int fwd_bf16_pick_split(const Dims& d, int n_cu, bool masked);
bool fwd_bf16_two_pass_fits(const Dims& d, const MaskDev& m);   // a masked forward may run as passes 1 and 2
bool fwd_bf16_one_pass_fits(const Dims& d, const MaskDev& m);   // ... or as one launch of the dense kernel over tile lists
bool fwd_bf16_takes_rows(const Dims& d, const MaskDev& m);      // ... or as one launch of it that masks by MaskRows
size_t fwd_bf16_rows_bytes_most(const Dims& d);                 // the most those words can take for any mask on this problem
size_t fwd_bf16_rows_counts_most(const Dims& d);                // ... and their counts of these
bool fwd_rows_bf16_takes(const Dims& d, bool masked);           // few query rows: a stream from memory
int fwd_rows_bf16_pick_split(const Dims& d, int n_cu);
hipError_t launch_fwd_rows_bf16(const FwdArgs& a, hipStream_t s);
hipError_t launch_fwd_general_bf16(const FwdArgs& a, hipStream_t s);   // masked or ragged problems
int bwd_bf16_pick_split(const Dims& d, int n_cu, bool masked);
MaskRows mask_rows_of(const Dims& d, const MaskDev& m);                 // the geometry (no words yet)
size_t mask_rows_bytes(const Dims& d, const MaskRows& r);
size_t mask_rows_counts_bytes(const Dims& d, const MaskRows& r);   // ... of which `counts`
hipError_t launch_mask_rows(const Dims& d, const MaskDev& m, MaskRows* r, void* words, hipStream_t s);
hipError_t launch_mask_rows_delta(const BwdArgs& a, MaskRows* r, hipStream_t s);     // ... in a.rows_ws, and launch_delta's work (bf16)
bool bwd_dq_bf16_takes_rows(const Dims& d, const MaskDev& m);           // the dQ kernel masks by MaskRows
bool bwd_dkdv_bf16_takes_rows(const Dims& d, const MaskDev& m);         // the dK/dV kernel masks by MaskRows
// memory-bound helpers
hipError_t launch_merge(const MergeArgs& a, int part_is_f32, int out_is_f32, hipStream_t s);
hipError_t launch_delta(const Dims& d, const void* o, const void* d_o, int is_f32, const float* lse,
                        float* delta, float* stats, int sq_pad, float* stats_ovl, hipStream_t s);
// dq_accum[i] += sum over the n_parts slices of `parts` (each n floats, n a multiple of 4)
// (of runs of `run` floats in every `group` of them, the last ones)
// (`first`: not added to what is there; dq_last: written there in bf16, with Q's strides)
hipError_t launch_dq_reduce(const Dims& d, const float* parts, int n_parts, long n, long run, long group, float* dq_accum, bool first,
                            void* dq_last, hipStream_t s);
hipError_t launch_dq_finalize(const Dims& d, const float* dq_accum, void* dq, int is_f32,
                              hipStream_t s);

}  // namespace lvx

// C ABI of the library (see include/lvx.h): argument validation on the host, workspace carving,
// KV-split choice, and kernel launches on the caller's stream.  Nothing here allocates or
// synchronises.
#include "../../include/lvx.h"
#include "lvx_internal.h"

#include <math.h>

using namespace lvx;

namespace {

constexpr size_t ALIGN = 256;
constexpr bool FUSED_BY_DEFAULT = false;   // lvx_xattn_bwd: one fused kernel where it applies, else dK/dV + dQ kernels
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

int device_cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      return 256;
  }
  return n;
}

lvx_status check_problem(const lvx_problem* p, lvx_dtype dtype) {
  if (!p) return LVX_ERR_NULL;
  if (dtype != LVX_F32 && dtype != LVX_BF16) return LVX_ERR_DTYPE;
  if (p->B < 1 || p->Hq < 1 || p->Hkv < 1 || p->Sq < 1 || p->Skv < 1 || p->D < 1) return LVX_ERR_SHAPE;
  if (p->Hq % p->Hkv != 0) return LVX_ERR_SHAPE;
  if (p->B > 65535 || p->Hq > 65535) return LVX_ERR_SHAPE;
  if (p->D != 64 && p->D != 96 && p->D != 128) return LVX_ERR_UNSUPPORTED;
  // rows are read with 16-byte vector accesses: strides must keep that alignment
  const int64_t vec = dtype == LVX_F32 ? 4 : 8;
  const int64_t qs[3] = {p->q_sb, p->q_sh, p->q_ss}, ks[3] = {p->kv_sb, p->kv_sh, p->kv_ss};
  for (int i = 0; i < 3; ++i)
    if (qs[i] % vec != 0 || ks[i] % vec != 0) return LVX_ERR_STRIDE;
  if (p->q_ss < p->D || p->kv_ss < p->D) return LVX_ERR_STRIDE;
  if (p->Sq > 1 && p->q_sh < 0) return LVX_ERR_STRIDE;
  if (p->q_sh < 0 || p->q_sb < 0 || p->kv_sh < 0 || p->kv_sb < 0) return LVX_ERR_STRIDE;
  if (p->Hq > 1 && p->q_sh < (int64_t)p->D) return LVX_ERR_STRIDE;
  if (p->Hkv > 1 && p->kv_sh < (int64_t)p->D) return LVX_ERR_STRIDE;
  if (p->B > 1 && (p->q_sb < (int64_t)p->D || p->kv_sb < (int64_t)p->D)) return LVX_ERR_STRIDE;
  return LVX_OK;
}

lvx_status check_mask(const lvx_problem* p, const lvx_mask* m) {
  if (!m) return LVX_OK;
  if (!m->allow) return LVX_ERR_NULL;
  if (m->q_chunk < 1 || m->kv_block < 1 || m->n_q_chunks < 1 || m->n_kv_blocks < 1) return LVX_ERR_MASK;
  if ((int64_t)m->n_q_chunks * m->q_chunk < p->Sq) return LVX_ERR_MASK;
  if ((int64_t)m->n_kv_blocks * m->kv_block < p->Skv) return LVX_ERR_MASK;
  if (m->stride_q < m->n_kv_blocks || m->stride_b < 0) return LVX_ERR_MASK;
  return LVX_OK;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

Dims make_dims(const lvx_problem* p) {
  Dims d;
  d.B = p->B; d.Hq = p->Hq; d.Hkv = p->Hkv; d.Sq = p->Sq; d.Skv = p->Skv; d.D = p->D;
  d.G = p->Hq / p->Hkv;
  d.q_sb = p->q_sb; d.q_sh = p->q_sh; d.q_ss = p->q_ss;
  d.kv_sb = p->kv_sb; d.kv_sh = p->kv_sh; d.kv_ss = p->kv_ss;
  d.scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->D);
  return d;
}

MaskDev make_mask(const lvx_mask* m) {
  MaskDev r;
  if (!m) { r.allow = nullptr; r.q_chunk = r.kv_block = 1; r.n_q_chunks = r.n_kv_blocks = 0; r.stride_b = r.stride_q = 0; return r; }
  r.allow = m->allow; r.q_chunk = m->q_chunk; r.kv_block = m->kv_block;
  r.n_q_chunks = m->n_q_chunks; r.n_kv_blocks = m->n_kv_blocks;
  r.stride_b = (long)m->stride_b; r.stride_q = (long)m->stride_q;
  return r;
}

int fwd_split(const Dims& d, lvx_dtype dtype, bool masked) {
  return dtype == LVX_BF16 ? fwd_bf16_pick_split(d, device_cu_count(), masked) : 1;
}
int fwd_list_split(const Dims& d) { return list_split((long)d.B * d.Hq * ((d.Sq + 255) / 256), (d.Skv + 63) / 64, device_cu_count()); }

// bf16 under a media mask that fits (fwd_bf16_two_pass_fits): the dense kernel over the key tiles
// that every row of a workgroup sees, then the general kernel on the other visible tiles; each
// launch leaves n_split partial results (slices [0, n_split) and [n_split, 2 n_split)).
int fwd_two_pass_split(int n_split, int reserve) {   // each launch's split count: both launches' parts (and
  const int cap = (LVX_MAX_PARTS - reserve) / 2;      // `reserve` others) go into one combine
  return n_split < cap ? n_split : cap;
}
hipError_t launch_fwd_bf16_two_pass(FwdArgs a, hipStream_t s) {
  a.partial = 1;
  a.pass = 1;
  a.part0 = 0;
  const hipError_t e = launch_fwd_bf16(a, s);
  if (e != hipSuccess) return e;
  a.pass = 2;
  a.part0 = a.n_split;
  return launch_fwd_bf16(a, s);
}

size_t split_rows(const Dims& d, int whole) {   // rows that are split: all but the first `whole` tiles of 256 of a group
  return (size_t)d.B * d.Hkv * ((long)d.G * d.Sq - 256L * whole);
}
size_t fwd_ws(const Dims& d, int n_split, int whole = 0) {
  if (n_split <= 1) return ALIGN;   // never zero, so that a valid workspace pointer is always passed
  const size_t rows = split_rows(d, whole);
  return align_up(rows * d.D * sizeof(float) * n_split) + align_up(rows * sizeof(float) * n_split);
}
// lvx_xattn_fwd_merge: the splits' partial results (bf16 kernels that split the key range).  The float32
// kernels, which merge in their epilogue, leave theirs alone; callers give them room for a partial result all the same.
size_t fwd_merge_ws(const Dims& d, lvx_dtype dtype, int n_split, int whole = 0) {
  return fwd_ws(d, dtype == LVX_F32 ? 2 : n_split, whole);      // (fwd_ws(d, 2) holds more than one partial result)
}
int cap_parts(int n, int reserve) { return n < LVX_MAX_PARTS - reserve ? n : LVX_MAX_PARTS - reserve; }
// How a forward call runs: the KV splits of each launch, whether a media mask makes it two launches, the partial
// results the combine then reads, the bytes of MaskRows' words the kernel reads, and the workspace it all takes. The
// dense kernel leaves the first `whole` row tiles of a K/V head unsplit. `reserve` parts of the combine are taken
// already (lvx_xattn_fwd_merge: the running state).
struct FwdPlan { int n_split, whole; bool two; int n_parts; size_t rows_bytes, need; };
FwdPlan fwd_plan_with(const Dims& d, lvx_dtype dtype, const MaskDev& m, int reserve, bool rows, size_t room) {
  const bool masked = m.allow != nullptr, bf16 = dtype == LVX_BF16;
  FwdPlan f;
  f.whole = 0;
  f.n_split = fwd_split(d, dtype, masked);
  if (f.n_split > LVX_MAX_PARTS - reserve) f.n_split = LVX_MAX_PARTS - reserve;
  f.two = masked && bf16 && !rows && fwd_bf16_two_pass_fits(d, m);
  if (f.two) f.n_split = fwd_two_pass_split(f.n_split, reserve);
  f.rows_bytes = rows ? align_up(mask_rows_bytes(d, mask_rows_of(d, m))) : 0;
  const bool list = masked && bf16 && (rows || fwd_bf16_one_pass_fits(d, m));
  if (list) f.n_split = fwd_list_split(d);
  for (;;) {
    f.n_parts = f.two ? 2 * f.n_split : f.n_split;
    f.need = (reserve ? fwd_merge_ws(d, dtype, f.n_parts) : fwd_ws(d, f.n_parts)) + f.rows_bytes;
    if (f.need <= room || f.n_split == 1) return f;
    // (a list can be shared by any number, and so can the keys of the other forms: fewer keys or rows may want more
    // parts than those that the workspace was made for, 28 x 1 row against 6369 keys in the room of 6597)
    f.n_split = list ? f.n_split / 2 : f.n_split - 1;
  }
}
// ... in a workspace of `room` bytes.  Words that do not fit (262144 rows against 131072 keys in blocks of 64: 68
// MB, where the general kernel needs nothing) leave the call to the kernels that do without.
FwdPlan fwd_plan(const Dims& d, lvx_dtype dtype, const MaskDev& m, int reserve, size_t room) {
  if (dtype == LVX_BF16 && fwd_bf16_dense(d, m.allow != nullptr)) {
    const auto plan = [&](TailPlan t) -> FwdPlan { return {t.parts, t.whole, false, t.parts, 0, fwd_ws(d, t.parts, t.whole)}; };
    // (parts for every place on the chip, or, where that many do not fit the workspace, for every compute unit)
    for (int per_cu = fwd_bf16_dense_per_cu(d); per_cu >= 1; --per_cu) {
      const FwdPlan f = plan(fwd_bf16_dense_plan(d, device_cu_count(), LVX_MAX_PARTS - reserve, per_cu));
      if (f.need <= room) return f;
    }
    // (coarse parts, or down to half of them: those of fewer keys or rows may be a few more than a larger problem's)
    const int coarse = cap_parts(fwd_bf16_coarse_split(d, device_cu_count()), reserve);
    int n = coarse;
    while (n > (coarse + 1) / 2 && plan({0, n}).need > room) --n;
    return plan({0, n});
  }
  const bool rows = m.allow != nullptr && dtype == LVX_BF16 && fwd_bf16_takes_rows(d, m);
  const FwdPlan f = fwd_plan_with(d, dtype, m, reserve, rows, room);
  return rows && f.need > room ? fwd_plan_with(d, dtype, m, reserve, false, room) : f;
}
int sq_padded(const Dims& d) { return (d.Sq + 31) / 32 * 32; }
bool has_stats_ovl(const Dims& d) { return d.Sq % 32 != 0 && d.Sq >= 32; }
size_t stats_floats(const Dims& d) { return 2 * (size_t)d.B * d.Hq * sq_padded(d); }
size_t bwd_ws_fixed(const Dims& d) {   // delta [B,Hq,Sq] + padded statistics [B,Hq,sq_pad/32][2][32]
                                       // (+ those of the last 32 rows, [B,Hq][2][32], when Sq is ragged)
  return align_up((size_t)d.B * d.Hq * d.Sq * sizeof(float)) +
         align_up((stats_floats(d) + (has_stats_ovl(d) ? (size_t)d.B * d.Hq * 64 : 0)) * sizeof(float));
}
// How the dQ kernels split the key range, and the workspace of a backward call: `list` splits under masks that
// run over lists, else dq; partial sums [n_slices, split rows, D].  A masked bf16 call always has one
// slice at least: the words of MaskRows go into the first slice, which the kernels that read them
// leave alone (`list` is one less at least), and which the others fill only after the words' last reader.
// The order: statistics, the fused kernel's dQ tiles, locks and error word (`part_at` bytes up to here), the slices.
struct BwdPlan { TailPlan dq; int list, n_slices; size_t part_at, part, need; };
size_t bwd_slice_bytes(const Dims& d) { return (size_t)d.B * d.Hq * d.Sq * d.D * sizeof(float); }
// The first slice of a masked call, which the words may fill: a slice, and where a slice is less than the words may be (one
// or two heads) the four bytes more that they take for 64 key blocks since they hold counts.
size_t bwd_words_room(const Dims& d) {
  const size_t slice = bwd_slice_bytes(d), most = fwd_bf16_rows_bytes_most(d);
  return slice + (most > slice ? align_up(fwd_bf16_rows_counts_most(d)) : 0);
}
bool can_fuse(const Dims& d, lvx_dtype dtype, bool masked) { return dtype == LVX_BF16 && bwd_fused_bf16_supported(d, masked); }
BwdPlan bwd_plan_with(const Dims& d, lvx_dtype dtype, bool masked, bool fused, bool coarse, int most = LVX_MAX_PARTS) {
  BwdPlan p = {{0, 1}, 1, 0, 0, 0, 0};
  if (dtype == LVX_BF16) {
    const int n_cu = device_cu_count();
    if (!bwd_dq_bf16_dense(d, masked)) p.dq.parts = bwd_bf16_pick_split(d, n_cu, masked);
    else if (coarse) p.dq.parts = bwd_dq_bf16_coarse_split(d, n_cu);
    else p.dq = bwd_dq_bf16_dense_plan(d, n_cu);
    if (p.dq.parts > most) p.dq.parts = most;
    const int n = p.dq.parts;
    if (masked) p.list = !coarse ? fwd_list_split(d) : n > 1 ? n / 2 : 1;
    p.n_slices = !masked ? (n > 1 ? n : 0) : n > p.list || coarse ? n : p.list + 1;
    p.part = align_up(p.n_slices * split_rows(d, p.dq.whole) * d.D * sizeof(float));
    if (masked) p.part += bwd_words_room(d) - bwd_slice_bytes(d);
  }
  p.part_at = bwd_ws_fixed(d) + (fused ? align_up(bwd_fused_ws_bytes(d)) : 0);
  p.need = p.part_at + p.part;
  return p;
}
// ... in a workspace of `room` bytes.  Fewer keys or rows may want more parts than what the workspace was made for (a block
// loop whose K is shorter: 16 heads x 29 rows against 4982 keys in the room of 4996): coarse splits, and
// of these as many as there is room for, down to none (under a mask one slice, which a call with more rows has too).
BwdPlan bwd_plan(const Dims& d, lvx_dtype dtype, bool masked, bool fused, size_t room) {
  BwdPlan p = bwd_plan_with(d, dtype, masked, fused, false);
  if (p.need <= room) return p;
  p = bwd_plan_with(d, dtype, masked, fused, true);
  while (p.need > room && p.dq.parts > 1) p = bwd_plan_with(d, dtype, masked, fused, true, p.dq.parts - 1);
  return p;
}
// How the dK/dV kernel shares key tiles among workgroups where there are `room` bytes for their sums (and, under a
// mask, the tiles' numbers of parts): as many parts as fit.
KvPlan kv_plan(const Dims& d, lvx_dtype dtype, bool masked, size_t room) {
  if (dtype != LVX_BF16) return {0, 1, 0};
  const size_t counts = dkdv_bf16_counts_bytes(d), set = dkdv_bf16_set_bytes(d);
  return dkdv_bf16_plan(d, device_cu_count(), masked, room > counts ? (long)((room - counts) / set) : 0);
}
// The sums lie where the dQ kernel's slices do: they have been added up when that kernel starts.  (Under a mask the
// first slice holds the words, which dK/dV reads too.)
size_t bwd_kv_at(const Dims& d, lvx_dtype dtype, bool masked) {
  return bwd_ws_fixed(d) + (can_fuse(d, dtype, masked) ? align_up(bwd_fused_ws_bytes(d)) : 0) + (masked ? bwd_words_room(d) : 0);
}
// A call's workspace without room for the sums: the larger of the dense and the masked plans'.
size_t bwd_ws_base(const Dims& d, lvx_dtype dtype) {
  const auto larger = [](size_t x, size_t y) { return x > y ? x : y; };
  const auto of = [&](bool masked) -> size_t {
    const bool fused = can_fuse(d, dtype, false);
    return larger(bwd_plan_with(d, dtype, masked, fused, false).need, bwd_plan_with(d, dtype, masked, fused, true).need);
  };
  return larger(of(true), of(false));
}
// What a backward call may fill: twice that, or a set of sums for every compute unit more.  One round of workgroups is
// what few key tiles need (28 / 4 heads, D = 128, delta + dK/dV: 1226 rows x 1024 keys 322 -> 65 us with 64 MB of
// sums, 74 with 32, 125 with 16; 185 x 1905 61 -> 45, 50, 61); masks, whose tiles may all be cut, want more where there are many.
size_t bwd_ws_most(const Dims& d, lvx_dtype dtype) {
  const size_t base = bwd_ws_base(d, dtype), round = (size_t)device_cu_count() * dkdv_bf16_set_bytes(d) + dkdv_bf16_counts_bytes(d);
  return base + (base > round ? base : round);
}
KvPlan bwd_kv_plan(const Dims& d, lvx_dtype dtype, bool masked, size_t workspace_bytes) {
  if (dtype != LVX_BF16) return {0, 1, 0};
  const size_t at = bwd_kv_at(d, dtype, masked), most = bwd_ws_most(d, dtype), end = workspace_bytes < most ? workspace_bytes : most;
  return kv_plan(d, dtype, masked, end > at ? end - at : 0);
}
size_t bwd_ws_query(const Dims& d, lvx_dtype dtype) {
  size_t n = bwd_ws_base(d, dtype);
  for (int masked = 0; masked < 2; ++masked) {
    const KvPlan p = bwd_kv_plan(d, dtype, masked, SIZE_MAX);
    const size_t kv = p.parts > 1 ? bwd_kv_at(d, dtype, masked) + dkdv_bf16_sums_bytes(d, p) + dkdv_bf16_counts_bytes(d) : 0;
    if (kv > n) n = kv;
  }
  return n;
}
}  // namespace

namespace lvx {
size_t fwd_workspace_need(const lvx_problem* p, lvx_dtype dtype, const lvx_mask* mask, size_t room) {
  if (check_problem(p, dtype) != LVX_OK || check_mask(p, mask) != LVX_OK) return 0;
  return fwd_plan(make_dims(p), dtype, make_mask(mask), 0, room).need;
}
}  // namespace lvx

extern "C" {

const char* lvx_strerror(lvx_status s) {
  switch (s) {
    case LVX_OK: return "ok";
    case LVX_ERR_NULL: return "required pointer is NULL";
    case LVX_ERR_SHAPE: return "invalid shape";
    case LVX_ERR_DTYPE: return "unsupported dtype";
    case LVX_ERR_STRIDE: return "invalid or misaligned stride / pointer";
    case LVX_ERR_MASK: return "mask geometry does not cover the problem";
    case LVX_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case LVX_ERR_UNSUPPORTED: return "unsupported head dimension or projection shape";
    case LVX_ERR_HIP: return "HIP launch failed";
  }
  return "unknown status";
}

size_t lvx_xattn_workspace_bytes(const lvx_problem* p, lvx_dtype dtype, int which) {
  if (check_problem(p, dtype) != LVX_OK) return 0;
  const Dims d = make_dims(p);
  // (the size does not depend on whether the call will carry a mask, nor on which: the larger of the
  // split counts -- a masked bf16 call may run as two launches that leave their splits' partial results
  // side by side -- and the most words that MaskRows can take)
  const auto larger = [](int x, int y) { return x > y ? x : y; };
  const size_t rows_most = dtype == LVX_BF16 ? align_up(fwd_bf16_rows_bytes_most(d)) : 0;
  const auto parts = [&](int reserve) {
    const int masked = dtype == LVX_BF16 ? 2 * fwd_two_pass_split(fwd_split(d, dtype, true), reserve) : 1;
    const auto cap = [&](int n) { return cap_parts(n, reserve); };
    return larger(larger(masked, larger(cap(fwd_split(d, dtype, true)), dtype == LVX_BF16 ? fwd_list_split(d) : 1)),
                  cap(fwd_split(d, dtype, false)));
  };
  const auto most = [](size_t x, size_t y) { return x > y ? x : y; };
  const auto dense = [&](int reserve) -> size_t {
    if (dtype != LVX_BF16 || !fwd_bf16_dense(d, false)) return 0;
    return most(fwd_plan(d, dtype, make_mask(nullptr), reserve, SIZE_MAX).need,
                fwd_ws(d, cap_parts(fwd_bf16_coarse_split(d, device_cu_count()), reserve)));
  };
  if (which == LVX_WS_FWD) return most(fwd_ws(d, parts(0)) + rows_most, dense(0));
  if (which == LVX_WS_BWD) return bwd_ws_query(d, dtype);
  if (which == LVX_WS_FWD_MERGE) return most(fwd_merge_ws(d, dtype, parts(1)) + rows_most, dense(1));
  return 0;
}

lvx_status lvx_xattn_fwd(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                         const void* v, const lvx_mask* mask, void* o, lvx_dtype o_dtype,
                         float* lse, void* workspace, size_t workspace_bytes, void* hip_stream) {
  lvx_status st = check_problem(p, dtype);
  if (st != LVX_OK) return st;
  if (!q || !k || !v || !o || !lse) return LVX_ERR_NULL;
  if (o_dtype != dtype && o_dtype != LVX_F32) return LVX_ERR_DTYPE;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return LVX_ERR_STRIDE;
  if ((st = check_mask(p, mask)) != LVX_OK) return st;
  FwdArgs a;
  a.d = make_dims(p);
  a.n_cu = device_cu_count();
  a.mask = make_mask(mask);
  a.q = q; a.k = k; a.v = v; a.o = o; a.o_is_f32 = o_dtype == LVX_F32; a.lse = lse;
  a.merge_into = 0;
  a.o_last = nullptr;
  a.partial = 0; a.part0 = 0; a.pass = 0;
  const FwdPlan plan = fwd_plan(a.d, dtype, a.mask, 0, workspace_bytes);
  a.n_split = plan.n_split;
  a.whole = plan.whole;
  const int n_parts = plan.n_parts;
  a.o_part = nullptr; a.lse_part = nullptr;
  if (!workspace || ((uintptr_t)workspace % ALIGN) != 0 || workspace_bytes < plan.need) return LVX_ERR_WORKSPACE;
  a.rows = MaskRows{};
  a.rows_ws = plan.rows_bytes > 0 ? (char*)workspace + fwd_ws(a.d, n_parts) : nullptr;
  hipStream_t s = (hipStream_t)hip_stream;
  const size_t rows = split_rows(a.d, a.whole);
  if (n_parts > 1) {
    a.o_part = (float*)workspace;
    a.lse_part = (float*)((char*)workspace + align_up(rows * a.d.D * sizeof(float) * n_parts));
  }
  hipError_t e = plan.two ? launch_fwd_bf16_two_pass(a, s)
                          : dtype == LVX_BF16 ? launch_fwd_bf16(a, s) : launch_fwd_f32(a, s);
  if (e != hipSuccess) return LVX_ERR_HIP;
  if (n_parts > 1) {
    MergeArgs m;
    m.n_parts = n_parts;
    for (int i = 0; i < n_parts; ++i) {
      m.o_parts[i] = a.o_part + (size_t)i * rows * a.d.D;
      m.lse_parts[i] = a.lse_part + (size_t)i * rows;
    }
    m.o_slices = a.o_part; m.lse_slices = a.lse_part; m.first = 0;
    m.rows = (long)rows; m.D = a.d.D; m.o_out = o; m.lse_out = lse;
    m.group = a.d.G * a.d.Sq; m.skip = 256 * a.whole;
    m.Hq = a.d.Hq; m.Sq = a.d.Sq; m.o_sb = a.d.q_sb; m.o_sh = a.d.q_sh; m.o_ss = a.d.q_ss;
    e = launch_merge(m, 1, a.o_is_f32, s);
    if (e != hipSuccess) return LVX_ERR_HIP;
  }
  return LVX_OK;
}

static lvx_status fwd_merge(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k, const void* v,
                            const lvx_mask* mask, float* o_acc, float* lse_acc, void* o_last, void* workspace,
                            size_t workspace_bytes, void* hip_stream) {
  lvx_status st = check_problem(p, dtype);
  if (st != LVX_OK) return st;
  if (!q || !k || !v || !o_acc || !lse_acc) return LVX_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o_acc)) return LVX_ERR_STRIDE;
  if ((st = check_mask(p, mask)) != LVX_OK) return st;
  FwdArgs a;
  a.d = make_dims(p);
  a.n_cu = device_cu_count();
  if (dtype == LVX_F32 && (a.d.q_ss != a.d.D || a.d.q_sh != (long)a.d.Sq * a.d.D ||
                           a.d.q_sb != (long)a.d.Hq * a.d.Sq * a.d.D))
    return LVX_ERR_STRIDE;      // (part of the interface, although the kernel would read any)
  a.mask = make_mask(mask);
  a.q = q; a.k = k; a.v = v; a.o_is_f32 = 1;
  a.o_last = o_last;
  a.partial = 0; a.part0 = 0; a.pass = 0;
  const FwdPlan plan = fwd_plan(a.d, dtype, a.mask, 1, workspace_bytes);          // (the running state is one more part of the combine)
  a.n_split = plan.n_split;
  a.whole = plan.whole;
  a.o_part = nullptr; a.lse_part = nullptr;
  if (!workspace || ((uintptr_t)workspace % ALIGN) != 0 || workspace_bytes < plan.need) return LVX_ERR_WORKSPACE;
  a.rows = MaskRows{};
  a.rows_ws = plan.rows_bytes > 0 ? (char*)workspace + fwd_merge_ws(a.d, dtype, plan.n_parts) : nullptr;
  hipStream_t s = (hipStream_t)hip_stream;
  const size_t rows = split_rows(a.d, a.whole);
  if (plan.n_parts == 1) {   // Rescale in the kernel's epilogue
    a.o = o_acc; a.lse = lse_acc; a.merge_into = 1;
    return (dtype == LVX_BF16 ? launch_fwd_bf16(a, s) : launch_fwd_f32(a, s)) == hipSuccess ? LVX_OK : LVX_ERR_HIP;
  }
  // partial results in the workspace, then one combine over the running state and them (the float32
  // kernels never split the key range)
  // (the tiles that are not split merge in the epilogue all the same)
  a.merge_into = 1;
  const int n_parts = plan.n_parts;
  float* const o_part = (float*)workspace;
  float* const l_part = (float*)((char*)workspace + align_up(rows * a.d.D * sizeof(float) * n_parts));
  a.o = o_acc; a.lse = lse_acc; a.o_part = o_part; a.lse_part = l_part;
  hipError_t e = plan.two ? launch_fwd_bf16_two_pass(a, s) : launch_fwd_bf16(a, s);
  if (e != hipSuccess) return LVX_ERR_HIP;
  MergeArgs m;
  m.n_parts = n_parts + 1;
  m.o_parts[0] = o_acc; m.lse_parts[0] = lse_acc;
  for (int i = 0; i < n_parts; ++i) {
    m.o_parts[i + 1] = o_part + (size_t)i * rows * a.d.D;
    m.lse_parts[i + 1] = l_part + (size_t)i * rows;
  }
  m.o_slices = o_part; m.lse_slices = l_part; m.first = 1;
  m.rows = (long)rows; m.D = a.d.D; m.o_out = o_acc; m.lse_out = lse_acc;
  m.group = a.d.G * a.d.Sq; m.skip = 256 * a.whole;
  m.Hq = a.d.Hq; m.Sq = a.d.Sq; m.o_ss = a.d.D; m.o_sh = (long)a.d.Sq * a.d.D; m.o_sb = (long)a.d.Hq * a.d.Sq * a.d.D;
  if (o_last != nullptr) {
    m.o_out = o_last;
    m.o_sb = a.d.q_sb; m.o_sh = a.d.q_sh; m.o_ss = a.d.q_ss;
  }
  e = launch_merge(m, 1, o_last == nullptr, s);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

lvx_status lvx_xattn_fwd_merge(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                               const void* v, const lvx_mask* mask, float* o_acc, float* lse_acc,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  return fwd_merge(p, dtype, q, k, v, mask, o_acc, lse_acc, nullptr, workspace, workspace_bytes, hip_stream);
}

lvx_status lvx_xattn_fwd_merge_last(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                                    const void* v, const lvx_mask* mask, float* o_acc, float* lse_acc, void* o,
                                    void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!o) return LVX_ERR_NULL;
  if (!aligned16(o)) return LVX_ERR_STRIDE;
  if (dtype == LVX_F32) return LVX_ERR_DTYPE;      // (a float32 running result is the result)
  return fwd_merge(p, dtype, q, k, v, mask, o_acc, lse_acc, o, workspace, workspace_bytes, hip_stream);
}

lvx_status lvx_xattn_merge(int32_t B, int32_t Hq, int32_t Sq, int32_t D, int32_t n_parts,
                           const void* const* o_parts, const float* const* lse_parts,
                           lvx_dtype part_dtype, void* o_out, lvx_dtype out_dtype, float* lse_out,
                           void* hip_stream) {
  if (!o_parts || !lse_parts || !o_out || !lse_out) return LVX_ERR_NULL;
  if (B < 1 || Hq < 1 || Sq < 1 || n_parts < 1 || n_parts > LVX_MAX_PARTS) return LVX_ERR_SHAPE;
  if (D != 64 && D != 96 && D != 128) return LVX_ERR_UNSUPPORTED;
  if ((part_dtype != LVX_F32 && part_dtype != LVX_BF16) || (out_dtype != LVX_F32 && out_dtype != LVX_BF16))
    return LVX_ERR_DTYPE;
  if (!aligned16(o_out)) return LVX_ERR_STRIDE;
  MergeArgs m;
  for (int i = 0; i < n_parts; ++i) {
    if (!o_parts[i] || !lse_parts[i]) return LVX_ERR_NULL;
    if (!aligned16(o_parts[i])) return LVX_ERR_STRIDE;
    m.o_parts[i] = o_parts[i];
    m.lse_parts[i] = lse_parts[i];
  }
  m.n_parts = n_parts;
  m.o_slices = m.lse_slices = nullptr; m.first = 0;
  m.rows = (long)B * Hq * Sq; m.group = 1; m.skip = 0; m.D = D; m.o_out = o_out; m.lse_out = lse_out;
  m.Hq = Hq; m.Sq = Sq; m.o_ss = D; m.o_sh = (long)Sq * D; m.o_sb = (long)Hq * Sq * D;
  hipError_t e = launch_merge(m, part_dtype == LVX_F32, out_dtype == LVX_F32, (hipStream_t)hip_stream);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

lvx_status lvx_xattn_bwd(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                         const void* v, const void* o, const float* lse, const void* d_o,
                         const lvx_mask* mask, float* dq_accum, void* dk, void* dv,
                         void* workspace, size_t workspace_bytes, void* hip_stream) {
  return lvx_xattn_bwd_stages(p, dtype, q, k, v, o, lse, d_o, mask, dq_accum, dk, dv, workspace,
                              workspace_bytes, hip_stream, LVX_BWD_ALL);
}

static lvx_status bwd_visit(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k, const void* v,
                            const void* o, const float* lse, const void* d_o, const lvx_mask* mask, float* dq_accum,
                            void* dk, void* dv, void* workspace, size_t workspace_bytes, void* hip_stream, unsigned stages,
                            bool first, void* dq_last) {
  lvx_status st = check_problem(p, dtype);
  if (st != LVX_OK) return st;
  if ((stages & LVX_BWD_ALL) == 0 || (stages & ~(unsigned)(LVX_BWD_ALL | LVX_BWD_FUSED | LVX_BWD_SPLIT))) return LVX_ERR_SHAPE;
  if ((stages & LVX_BWD_FUSED) && (stages & LVX_BWD_SPLIT)) return LVX_ERR_SHAPE;
  if (!q || !k || !v || !o || !lse || !d_o || !dq_accum || !dk || !dv) return LVX_ERR_NULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(d_o) ||
      !aligned16(dq_accum) || !aligned16(dk) || !aligned16(dv))
    return LVX_ERR_STRIDE;
  if ((st = check_mask(p, mask)) != LVX_OK) return st;
  BwdArgs a;
  a.d = make_dims(p);
  a.n_cu = device_cu_count();
  a.mask = make_mask(mask);
  a.dq_pass = 0;
  // the kernel that forms all five products at once: where it applies, unless the caller asks for
  // the two-kernel form (or only for one of the two kernels)
  const bool may_fuse = can_fuse(a.d, dtype, mask != nullptr);
  const bool want_fuse = (stages & LVX_BWD_FUSED) || (FUSED_BY_DEFAULT && !(stages & LVX_BWD_SPLIT));
  const bool fused = may_fuse && want_fuse && (stages & (LVX_BWD_DKDV | LVX_BWD_DQ)) == (LVX_BWD_DKDV | LVX_BWD_DQ);
  const BwdPlan plan = bwd_plan(a.d, dtype, mask != nullptr, may_fuse, workspace_bytes);
  a.n_split_dq = plan.dq.parts;
  a.dq_whole = plan.dq.whole;
  a.dq_list = plan.list;
  const int n_slices = plan.n_slices;
  const size_t need = plan.need;
  if (!workspace || ((uintptr_t)workspace % ALIGN) != 0 || workspace_bytes < need) return LVX_ERR_WORKSPACE;
  a.q = q; a.k = k; a.v = v; a.o = o; a.d_o = d_o; a.lse = lse;
  a.delta = (float*)workspace;
  a.sq_pad = sq_padded(a.d);
  a.stats = (float*)((char*)workspace + align_up((size_t)a.d.B * a.d.Hq * a.d.Sq * sizeof(float)));
  a.stats_ovl = has_stats_ovl(a.d) ? a.stats + stats_floats(a.d) : nullptr;
  a.dq_accum = dq_accum; a.dk = dk; a.dv = dv;
  a.dq_first = first; a.dq_last = dq_last;
  const auto at = [&](size_t x) -> char* { return (char*)workspace + x; };
  a.dq_part = n_slices > 0 ? (float*)at(plan.part_at) : nullptr;
  a.rows = MaskRows{};
  a.rows_ws = mask != nullptr && n_slices > 0 ? at(plan.part_at) : nullptr;
  a.rows_ws_bytes = bwd_words_room(a.d);
  a.dq_tiles = fused ? (float*)at(bwd_ws_fixed(a.d)) : nullptr;
  a.kv = {0, 1, 0}; a.kv_sums = nullptr; a.kv_counts = nullptr;
  if (!fused) {
    a.kv = bwd_kv_plan(a.d, dtype, mask != nullptr, workspace_bytes);
    if (a.kv.parts > 1) {
      const size_t kv_at = bwd_kv_at(a.d, dtype, mask != nullptr);
      a.kv_sums = (float*)at(kv_at);
      a.kv_counts = (int*)at(kv_at + dkdv_bf16_sums_bytes(a.d, a.kv));
    }
  }
  a.dq_locks = nullptr; a.dq_err = nullptr; a.dq_stagger = 0;
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e = hipSuccess;
  const bool kernels = (stages & (LVX_BWD_DKDV | LVX_BWD_DQ)) != 0;
  // (bf16: launch_bwd_bf16 makes the row statistics, with a mask's words in one launch)
  if ((stages & LVX_BWD_DELTA) && (dtype == LVX_F32 || !kernels)) e = launch_delta(a.d, o, d_o, dtype == LVX_F32, lse, a.delta, a.stats, a.sq_pad, a.stats_ovl, s);
  if (e != hipSuccess) return LVX_ERR_HIP;
  if (kernels)
    e = dtype == LVX_BF16 ? launch_bwd_bf16(a, stages & LVX_BWD_ALL, s) : launch_bwd_f32(a, stages & LVX_BWD_ALL, s);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

lvx_status lvx_xattn_bwd_stages(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                                const void* v, const void* o, const float* lse, const void* d_o,
                                const lvx_mask* mask, float* dq_accum, void* dk, void* dv,
                                void* workspace, size_t workspace_bytes, void* hip_stream,
                                unsigned stages) {
  return bwd_visit(p, dtype, q, k, v, o, lse, d_o, mask, dq_accum, dk, dv, workspace, workspace_bytes, hip_stream, stages, false,
                   nullptr);
}

lvx_status lvx_xattn_bwd_visit(const lvx_problem* p, lvx_dtype dtype, const void* q, const void* k,
                               const void* v, const void* o, const float* lse, const void* d_o,
                               const lvx_mask* mask, float* dq_accum, void* dk, void* dv,
                               void* workspace, size_t workspace_bytes, void* hip_stream, int first, void* dq) {
  if (dq && dtype == LVX_F32) return LVX_ERR_DTYPE;      // (float32 sums are the result)
  if (dq && !aligned16(dq)) return LVX_ERR_STRIDE;
  return bwd_visit(p, dtype, q, k, v, o, lse, d_o, mask, dq_accum, dk, dv, workspace, workspace_bytes, hip_stream,
                   (first ? LVX_BWD_ALL : LVX_BWD_DKDV | LVX_BWD_DQ) | LVX_BWD_SPLIT, first != 0, dq);
}

lvx_status lvx_xattn_bwd_error_word(const lvx_problem* p, lvx_dtype dtype, const lvx_mask* mask,
                                    void* workspace, size_t workspace_bytes, const int** word) {
  lvx_status st = check_problem(p, dtype);
  if (st != LVX_OK) return st;
  if (!word) return LVX_ERR_NULL;
  if ((st = check_mask(p, mask)) != LVX_OK) return st;
  const Dims d = make_dims(p);
  const bool fused = can_fuse(d, dtype, mask != nullptr);
  const BwdPlan plan = bwd_plan(d, dtype, mask != nullptr, fused, workspace_bytes);
  if (!workspace || ((uintptr_t)workspace % ALIGN) != 0 || workspace_bytes < plan.need) return LVX_ERR_WORKSPACE;
  *word = fused ? (const int*)((char*)workspace + bwd_ws_fixed(d) + bwd_fused_ws_bytes(d) - 256)
                : nullptr;
  return LVX_OK;
}

lvx_status lvx_xattn_dq_finalize(const lvx_problem* p, const float* dq_accum, void* dq,
                                 lvx_dtype dtype, void* hip_stream) {
  lvx_status st = check_problem(p, dtype);
  if (st != LVX_OK) return st;
  if (!dq_accum || !dq) return LVX_ERR_NULL;
  if (!aligned16(dq_accum) || !aligned16(dq)) return LVX_ERR_STRIDE;
  hipError_t e = launch_dq_finalize(make_dims(p), dq_accum, dq, dtype == LVX_F32, (hipStream_t)hip_stream);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

lvx_status lvx_xattn_project(const lvx_projection* p, lvx_dtype dtype, const void* x, const void* w,
                             int n_out, void* const* out, void* hip_stream) {
  if (!p || !x || !w || !out) return LVX_ERR_NULL;
  if (n_out < 1 || n_out > 2) return LVX_ERR_SHAPE;
  for (int o = 0; o < n_out; ++o)
    if (!out[o]) return LVX_ERR_NULL;
  if (p->B <= 0 || p->S <= 0 || p->E <= 0 || p->H <= 0 || p->D <= 0) return LVX_ERR_SHAPE;
  if ((long)n_out * p->H * p->D > INT32_MAX) return LVX_ERR_SHAPE;
  if (dtype != LVX_F32 && dtype != LVX_BF16) return LVX_ERR_DTYPE;
  const int esz = dtype == LVX_F32 ? 4 : 2;
  if (p->x_ss < p->E || p->x_sb != (int64_t)p->S * p->x_ss) return LVX_ERR_STRIDE;
  if (dtype == LVX_BF16) {                           // 16-byte copies and stores
    if ((p->x_ss * esz) % 16 != 0 || !aligned16(x) || !aligned16(w)) return LVX_ERR_STRIDE;
    for (int o = 0; o < n_out; ++o)
      if (!aligned16(out[o])) return LVX_ERR_STRIDE;
  }
  ProjArgs a{};
  a.x = x;
  a.w = w;
  for (int o = 0; o < n_out; ++o) a.out[o] = out[o];
  a.M = (long)p->B * p->S;
  a.ldx = p->x_ss;
  a.S = p->S;
  a.E = p->E;
  a.N = n_out * p->H * p->D;
  a.H = p->H;
  a.D = p->D;
  a.n_cu = device_cu_count();
  if (dtype == LVX_BF16 && !project_bf16_supported(a)) return LVX_ERR_UNSUPPORTED;
  // (a tile's copies address its rows with 32-bit byte offsets from the tile's first row)
  if (dtype == LVX_BF16 && 256 * p->x_ss * esz > (int64_t)UINT32_MAX) return LVX_ERR_STRIDE;
  const hipError_t e = launch_project(a, dtype == LVX_F32, (hipStream_t)hip_stream);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

lvx_status lvx_xattn_project_bwd(const lvx_projection* p, lvx_dtype dtype, const void* x, const void* w,
                                 int n_out, const void* const* d_out, void* dx, float* dw,
                                 void* hip_stream) {
  if (!p || !x || !w || !d_out) return LVX_ERR_NULL;
  if (n_out < 1 || n_out > 2) return LVX_ERR_SHAPE;
  for (int o = 0; o < n_out; ++o)
    if (!d_out[o]) return LVX_ERR_NULL;
  if (!dx && !dw) return LVX_ERR_NULL;
  if (p->B <= 0 || p->S <= 0 || p->E <= 0 || p->H <= 0 || p->D <= 0) return LVX_ERR_SHAPE;
  if ((long)n_out * p->H * p->D > INT32_MAX) return LVX_ERR_SHAPE;
  if (dtype != LVX_F32 && dtype != LVX_BF16) return LVX_ERR_DTYPE;
  const int esz = dtype == LVX_F32 ? 4 : 2;
  if (p->x_ss < p->E || p->x_sb != (int64_t)p->S * p->x_ss) return LVX_ERR_STRIDE;
  if (dtype == LVX_BF16) {                           // 16-byte copies and stores
    if ((p->x_ss * esz) % 16 != 0 || !aligned16(x) || !aligned16(w)) return LVX_ERR_STRIDE;
    if ((dx && !aligned16(dx)) || (dw && !aligned16(dw))) return LVX_ERR_STRIDE;
    for (int o = 0; o < n_out; ++o)
      if (!aligned16(d_out[o])) return LVX_ERR_STRIDE;
  }
  ProjBwdArgs a{};
  a.x = x;
  a.w = w;
  for (int o = 0; o < n_out; ++o) a.g[o] = d_out[o];
  a.dx = dx;
  a.dw = dw;
  a.M = (long)p->B * p->S;
  a.ldx = p->x_ss;
  a.S = p->S;
  a.E = p->E;
  a.N = n_out * p->H * p->D;
  a.H = p->H;
  a.D = p->D;
  a.n_cu = device_cu_count();
  const hipError_t e = launch_project_bwd(a, dtype == LVX_F32, (hipStream_t)hip_stream);
  return e == hipSuccess ? LVX_OK : LVX_ERR_HIP;
}

}  // extern "C"

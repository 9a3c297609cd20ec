// Units of 32 keys that a wavefront streams through LDS stages of its own, without barriers: the forward for a
// few query rows (lvx_fwd_rows_bf16.hip) and the row blocks of masks that show them little
// (lvx_mask_stream.h).
//
// Tiles are kept unpadded, the 16-byte chunks of a row permuted by the row (by the source addresses
// of the copies, which may be anything): K so that one chunk of 16 consecutive rows covers all
// banks, V so that 64 bytes of four consecutive rows do.
#pragma once
#include "lvx_mfma.h"

namespace lvx {

constexpr int UK = 32;                 // keys per unit

template <int D> struct KeyUnit {
  static constexpr int CPR = D / 8;                 // 16-byte chunks of data per row
  static constexpr int CH = D == 64 ? 8 : 16;       // chunk places per row (96-wide heads: four unused)
  static constexpr int ROWB = CH * 16;
  static constexpr int TILE = UK * ROWB;
  static constexpr int NC = TILE / 1024;            // wave-level copies per tile
  static constexpr int STAGE = 2 * TILE;            // K, then V
};
// where chunk c of row r stands: c ^ ...
template <int D> __device__ __forceinline__ int k_swz(int r) { return D == 64 ? (r >> 1) & 7 : r & 15; }
template <int D> __device__ __forceinline__ int v_swz(int r) { return D == 64 ? 4 * ((r >> 1) & 1) : 4 * (r & 3); }

// Source offset of lane's 16 bytes in wave-level copy n of a tile (64 chunk places in a row, lane l place 64 n + l);
// rows past last_row re-read it.
template <int D> __device__ __forceinline__ unsigned unit_copy_off(int n, bool v_order, int last_row, unsigned row_bytes, int lane) {
  using U = KeyUnit<D>;
  const int slot = 64 * n + lane, r = slot / U::CH;
  const int c = (slot % U::CH) ^ (v_order ? v_swz<D>(r) : k_swz<D>(r));
  return (unsigned)min(r, last_row) * row_bytes + (unsigned)min(c, U::CPR - 1) * 16;
}

}  // namespace lvx

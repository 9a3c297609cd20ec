// Shared by the matrix products whose workgroups stay for several tiles (project_run_bf16_kernel, lvx_project.hip, has the
// scheme): accumulators by name, what is left of the tile before, and its way out.
#pragma once
#include "lvx_internal.h"
#include "lvx_mfma.h"

#include <type_traits>

namespace lvx {
namespace tilerun {

constexpr int NFLUSH = 8;                            // tile pairs that write a part of the tile before
constexpr int FB_PITCH = 64 * 2 + 16;                // 32 rows x 64 columns on their way out, padded rows
constexpr int FB_WAVE = 32 * FB_PITCH;

template <int B = 0, class F> __device__ __forceinline__ void each_block(F&& f) {
  f(std::integral_constant<int, B>{});
  if constexpr (B < 15) each_block<B + 1>(f);
}

// The accumulators of a wave's 128 x 128: block B = 4 j + i (column block j, row block i, transposed) is a[16 B ...], by name.
// Nothing else may use that file, and the compiler does not know it: the build looks at the code that it made and fails if
// something does (check_named_accumulators in build.py; as values, the compiler moved some of them through ordinary registers between two
// tiles, and spilled others for it).
__device__ __forceinline__ void claim_accumulators() { asm volatile("" ::: "a0", "a255"); }
template <int B> __device__ __forceinline__ void mfma_start(bf16x8 a, bf16x8 b) {        // block B = a b
  asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, 0" ::"v"(a), "v"(b), "n"(16 * B), "n"(16 * B + 15));
}
template <int B> __device__ __forceinline__ void mfma_add(bf16x8 a, bf16x8 b) {          // ... += a b
  asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(a), "v"(b), "n"(16 * B), "n"(16 * B + 15));
}

// A finished tile, rounded: [row block][column block][four columns].
struct Packed { unsigned w[4][4][4][2]; };
template <int B> __device__ __forceinline__ void pack(Packed& pk) {
  constexpr int j = B / 4, i = B % 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float y[4];
    asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\tv_accvgpr_read_b32 %3, a[%7]"
                 : "=v"(y[0]), "=v"(y[1]), "=v"(y[2]), "=v"(y[3])
                 : "n"(16 * B + 4 * q), "n"(16 * B + 4 * q + 1), "n"(16 * B + 4 * q + 2), "n"(16 * B + 4 * q + 3));
    pk.w[i][j][q][0] = pack2_bf16(y[0], y[1]);
    pk.w[i][j][q][1] = pack2_bf16(y[2], y[3]);
    asm volatile("" : "+v"(pk.w[i][j][q][0]), "+v"(pk.w[i][j][q][1]));       // (packed here, not where it is written)
  }
}
// Part e of a tile: row block e / 2, columns 64 (e % 2) .. of the wave's 128.  turn puts four columns of one of its two column
// blocks into the wave's buffer (x = 0 .. 7), turned reads a lane's 16 bytes of row lane / 8 + 8 it of the block back.
__device__ __forceinline__ void turn(char* fb, const Packed& pk, int e, int x, int lane) {
  const int i = e / 2, j = 2 * (e % 2) + x / 4, q = x % 4, g = lane >> 5, l31 = lane & 31;
  *(u32x2*)(fb + l31 * FB_PITCH + (32 * (x / 4) + 8 * q + 4 * g) * 2) = u32x2{pk.w[i][j][q][0], pk.w[i][j][q][1]};
}
__device__ __forceinline__ u32x4 turned(const char* fb, int it, int lane) {
  return *(const u32x4*)(fb + (8 * it + (lane >> 3)) * FB_PITCH + (lane & 7) * 16);
}

}  // namespace tilerun
}  // namespace lvx

// Sums of table rows selected by base-4 digits, as an 8-bit matrix product (device code only).
//
// A key switch adds, for every digit position of every coefficient, the key row that the digit selects
// (none for digit 0). For a batch that is a matrix product: the operand of a batch element is 1 at
// (position, digit value) and 0 elsewhere, the other operand is the key split into four balanced
// signed bytes, and output word = sum of 2^(8 b) times byte plane b's product, mod 2^32 (int32 sums
// are exact: at most 2^15 positions of magnitude at most 128).
//
// One MFMA block is 64 deep: four digit bytes (four digits each, the first in the top bits) of four
// values; lane (m, q) of the 16 x 64 operand of batch element m holds digit byte q as four words
// 1 << 8 d, the other operand's lane (n, q) the 16 key bytes of that digit byte in column n. All four
// planes are multiplied by one construction of the one-hot operand.
//  Key: [column tile of 16][block][plane][lane][16 bytes]: a wave's load is 1 KiB, contiguous.
//  Digits: [tile of 16 elements][quad of blocks][lane]: byte t of lane (m, q)'s word is the bitwise
//   complement of digit byte q of block t of the quad, so that one byte alignment of 0x01000000 by the
//   low two bits gives 1 << 8 d.
#pragma once
#include "vsp_internal.h"

namespace vsp {

typedef int oh_v4i __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) oh_v4i* oh_key;
typedef const __attribute__((address_space(1))) u32* oh_digits;

constexpr int OH_PLANES = 4;
constexpr int OH_BLOCK = OH_PLANES * 64;   // key of one block and column tile, in 16-byte entries
constexpr int OH_WAVES = 8;                // waves of a workgroup: each takes every eighth quad

// Bytes of the four values of one digit, one word per plane (value 0 selects nothing).
__device__ __forceinline__ void oh_planes(u32 x1, u32 x2, u32 x3, u32 (&w)[OH_PLANES]) {
  u32 x[3] = {x1, x2, x3};
#pragma unroll
  for (int b = 0; b < OH_PLANES; b++) {
    w[b] = 0;
#pragma unroll
    for (int v = 0; v < 3; v++) {
      const int8_t c = (int8_t)(x[v] & 255u);  // x = c (mod 256), c in [-128, 127]
      x[v] = (x[v] - (u32)(int32_t)c) >> 8;
      w[b] |= (u32)(uint8_t)c << (8 * (v + 1));
    }
  }
}

// sum[i] = the products of element tile i with the key's column tile (key: at the lane) over `steps` quads,
// planes folded. The source of the digits gives the quad of step n, quad(n), and the digit words of
// its tiles, get(n, d); issue(n) and finish(n) stand before and after the step's products, for loads
// of its own. The key blocks of the next quad are loaded while this one is multiplied (16 KiB in
// flight per wave).
template <int T, class Digits>
__device__ __forceinline__ void oh_products(oh_key key, Digits& digits, int steps, u32 (&sum)[T][4]) {
  oh_v4i acc[T][OH_PLANES], kb[4][OH_PLANES];
  {
    const oh_key k0 = key + (size_t)(4 * digits.quad(0)) * OH_BLOCK;
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
      for (int b = 0; b < OH_PLANES; b++) kb[t][b] = k0[t * OH_BLOCK + b * 64];
  }
#pragma unroll
  for (int i = 0; i < T; i++)
#pragma unroll
    for (int b = 0; b < OH_PLANES; b++) acc[i][b] = oh_v4i{0, 0, 0, 0};
  digits.start();
  __builtin_amdgcn_sched_barrier(0);
  for (int n = 0; n < steps; n++) {
    u32 d[T];
    digits.get(n, d);
    digits.issue(n);
    const oh_key kn = key + (size_t)(4 * digits.quad(n + 1 < steps ? n + 1 : n)) * OH_BLOCK;
#pragma unroll
    for (int t = 0; t < 4; t++) {
#pragma unroll
      for (int i = 0; i < T; i++) {
        oh_v4i a;
#pragma unroll
        for (int w = 0; w < 4; w++) a[w] = (int)__builtin_amdgcn_alignbyte(0u, 0x01000000u, d[i] >> (8 * t + 6 - 2 * w));
#pragma unroll
        for (int b = 0; b < OH_PLANES; b++) acc[i][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, kb[t][b], acc[i][b], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < OH_PLANES; b++) kb[t][b] = kn[t * OH_BLOCK + b * 64];
      __builtin_amdgcn_sched_barrier(0);
    }
    digits.finish(n);
  }
#pragma unroll
  for (int i = 0; i < T; i++)
#pragma unroll
    for (int x = 0; x < 4; x++)
      sum[i][x] = (u32)acc[i][0][x] + ((u32)acc[i][1][x] << 8) + ((u32)acc[i][2][x] << 16) + ((u32)acc[i][3][x] << 24);
}

// The partial sums of a workgroup's SPLIT waves of one column tile (split = 0 .. SPLIT - 1) added through
// LDS: afterwards use(i, x, value) has been called once for every tile i and register x, by one of these
// waves, lane (n, q) holding element 4 q + x of the tile, column n. red: the column tile's.
template <int T, int SPLIT, class Use>
__device__ __forceinline__ void oh_reduce(const u32 (&sum)[T][4], u32 (*red)[T * 4][64], int split, int lane, Use use) {
#pragma unroll
  for (int i = 0; i < T; i++)
#pragma unroll
    for (int x = 0; x < 4; x++) red[split][i * 4 + x][lane] = sum[i][x];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < (T * 4 + SPLIT - 1) / SPLIT; k++) {
    const int r = split + k * SPLIT;
    if (T * 4 % SPLIT && r >= T * 4) break;
    u32 v = 0;
#pragma unroll
    for (int w = 0; w < SPLIT; w++) v += red[w][r][lane];
    use(r >> 2, r & 3, v);
  }
}

}  // namespace vsp

// Scheme constants, and the wave-level negacyclic NTT of degree N = 1024 modulo
// p = 2^64 - 2^32 + 1, which the product of two arbitrary polynomials takes (their exact product
// exceeds what the float64 transform of fft.h rounds correctly).
//
// Layout. A wave (64 lanes) works on two polynomials at once: lanes 0-31 on the first,
// lanes 32-63 on the second. Lane l = lane & 31 holds coefficients l + 32 t (t = 0..31) in
// register t. With Z = X^32 the polynomial is sum_l X^l (sum_t a_{l+32t} Z^t), so:
//  pass 1 (in registers): for every l, the 32-point negacyclic transform over t evaluates
//    sum_t a_{l+32t} zeta^t at the 32 roots zeta = 2^{3(2u+1)} of Z^32 = -1, giving the
//    residues a mod (X^32 - zeta_u). Its twiddles are powers of two (2 has order 192 mod p),
//    so every multiply is by a compile-time 2^e.
//  transpose through LDS: lane u receives the 32 coefficients of residue u.
//  pass 2 (in registers): a mod (X^32 - zeta_u) is evaluated at psi_u w^k (w = 2^6, a
//    primitive 32nd root; psi_u = psi^{2u+1} with psi^32 = 8): multiply coefficient j by
//    psi_u^j (table) then a cyclic 32-point DFT with power-of-two twiddles.
// The inverse undoes pass 2 (inverse DFT, psi_u^-j), transposes back, and undoes pass 1 as
// a cyclic inverse DFT over the residues followed by the twist zeta^-t of coefficient t.
// The factor 1/N is the caller's. Every butterfly multiplies its second input by the
// twiddle (Cooley-Tukey form), so the product is canonical and the sum and difference
// need a single carry fix each.
#pragma once
#include "gl64.h"

namespace vsp {

constexpr int RING_N = 1024;
constexpr int LWE_N = 630;
constexpr int GADGET_L = 3;
constexpr int BG_BIT = 6;
constexpr int KS_T = 8;
constexpr int KS_BASEBIT = 2;
constexpr u32 MU = 1u << 29;                // 1/8
constexpr u32 DECOMP_OFFSET = 0x82082000u;  // sum_r (Bg/2) 2^(32-6r) + 2^(32-18-1)

// One transpose region per half-wave: 32 rows of 33 u32 (the pad column keeps the row and
// column accesses of a half-wave on distinct LDS banks); 64-bit values cross it in two
// 32-bit passes. The regions of the two halves start 32 words apart modulo the bank count.
constexpr int TROW = 33;
constexpr int TREGION = 32 * TROW + 64;     // u32 per half
constexpr int WAVE_T_U32 = 2 * TREGION;     // u32 per wave

constexpr int brv5(int k) {
  return ((k & 1) << 4) | ((k & 2) << 2) | (k & 4) | ((k & 8) >> 2) | ((k & 16) >> 4);
}

// Twiddle exponents: every twiddle of the two in-register passes is 2^e mod p, e in [0, 192).
struct TwiddleExps {
  int p1f[32];   // pass-1 forward: 3 brv5(m)
  int p1i[32];   // pass-1 inverse: -3 brv5(m)
  int dft[32];   // w^e = 2^{6e}
  int dfti[32];  // w^-e
};

constexpr TwiddleExps make_twiddle_exps() {
  TwiddleExps T{};
  for (int m = 0; m < 32; m++) {
    T.p1f[m] = (3 * brv5(m)) % 192;
    T.p1i[m] = (192 - 3 * brv5(m)) % 192;
    T.dft[m] = (6 * m) % 192;
    T.dfti[m] = (192 - 6 * m) % 192;
  }
  return T;
}

__device__ constexpr TwiddleExps kTwE = make_twiddle_exps();

// Cooley-Tukey butterfly (x, y) -> (x + 2^E y, x - 2^E y), E in [0, 192); 2^96 = -1 folds
// the upper half of the exponents into a swap of the sum and the difference.
__device__ __forceinline__ void bfly_ct(u64& x, u64& y, int E) {
  const u64 a = x;
  const u64 t = gl_mul_pow2(y, E % 96);  // canonical
  if (E >= 96) {
    x = gl_sub_c(a, t);
    y = gl_add_c(a, t);
  } else {
    x = gl_add_c(a, t);
    y = gl_sub_c(a, t);
  }
}

// Hides x from the optimiser so that per-lane address arithmetic derived from it is
// recomputed inside a loop instead of being hoisted (and kept live) across all iterations.
__device__ __forceinline__ int opaque_lane(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Orders the LDS traffic of one wave (all lanes' stores before any lane's loads).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Pass 1, forward: negacyclic Cooley-Tukey over the register index (natural order in,
// bit-reversed out: register k holds residue u = brv5(k)).
__device__ __forceinline__ void pass1_forward(u64 (&v)[32]) {
#pragma unroll
  for (int s = 0; s < 5; s++) {
    const int M = 1 << s, H = 16 >> s;
#pragma unroll
    for (int b = 0; b < M; b++) {
#pragma unroll
      for (int j = 0; j < H; j++) {
        const int i = b * 2 * H + j;
        bfly_ct(v[i], v[i + H], kTwE.p1f[M + b]);
      }
    }
  }
}

// Cyclic 32-point DFT with w = 2^6 (natural order in, bit-reversed out: register brv5(k)
// receives X_k), as decimation in time over the bit-reversed register names.
__device__ __forceinline__ void dft32_forward(u64 (&v)[32]) {
#pragma unroll
  for (int s = 4; s >= 0; s--) {
    const int H = 16 >> s;
#pragma unroll
    for (int blk = 0; blk < 32; blk += 2 * H) {
#pragma unroll
      for (int j = 0; j < H; j++) bfly_ct(v[brv5(blk + j)], v[brv5(blk + j + H)], kTwE.dft[(j << s) & 31]);
    }
  }
}

// Cyclic inverse DFT with w^-1 (decimation in time; bit-reversed in, natural out; unscaled).
// Inverts dft32_forward, and also pass 1: register k of a lane holding the residues at
// zeta w^brv5(k) yields sum_u A_u w^-ut in register t.
__device__ __forceinline__ void dft32_inverse(u64 (&v)[32]) {
#pragma unroll
  for (int s = 4; s >= 0; s--) {
    const int H = 16 >> s;
#pragma unroll
    for (int blk = 0; blk < 32; blk += 2 * H) {
#pragma unroll
      for (int j = 0; j < H; j++) bfly_ct(v[blk + j], v[blk + j + H], kTwE.dfti[(j << s) & 31]);
    }
  }
}

// Lane l, register k (residue brv5(k), coefficient l) -> lane u = brv5(k), register l,
// through the half-wave's u32 region (low words, then high words).
__device__ __forceinline__ void transpose_forward(u64 (&v)[32], u32* reg, int l) {
  u32 lo[32];
#pragma unroll
  for (int k = 0; k < 32; k++) reg[brv5(k) * TROW + l] = (u32)v[k];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 32; j++) lo[j] = reg[l * TROW + j];
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 32; k++) reg[brv5(k) * TROW + l] = (u32)(v[k] >> 32);
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 32; j++) v[j] = ((u64)reg[l * TROW + j] << 32) | lo[j];
  wave_lds_sync();
}

// Inverse of transpose_forward.
__device__ __forceinline__ void transpose_inverse(u64 (&v)[32], u32* reg, int l) {
  u32 lo[32];
#pragma unroll
  for (int j = 0; j < 32; j++) reg[j * TROW + l] = (u32)v[j];
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 32; k++) lo[k] = reg[l * TROW + brv5(k)];
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < 32; j++) reg[j * TROW + l] = (u32)(v[j] >> 32);
  wave_lds_sync();
#pragma unroll
  for (int k = 0; k < 32; k++) v[k] = ((u64)reg[l * TROW + brv5(k)] << 32) | lo[k];
  wave_lds_sync();
}

// v[j] *= T[j][l] for j >= 1 (T[0][*] = 1), loading the table entries eight at a time so that
// at most sixteen of them are in flight.
__device__ __forceinline__ void table_multiply(u64 (&v)[32], const u64* T, int l) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    u64 w[8];
#pragma unroll
    for (int q = 0; q < 8; q++) w[q] = (8 * c + q == 0) ? 1 : T[(8 * c + q) * 32 + l];
#pragma unroll
    for (int q = 0; q < 8; q++)
      if (8 * c + q != 0) v[8 * c + q] = gl_mul(v[8 * c + q], w[q]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Forward transform of this half's polynomial (values already residues mod p). tf is the [j][u]
// table psi_u^j (in LDS or global memory).
__device__ __forceinline__ void ntt_forward(u64 (&v)[32], const u64* tf, u32* reg, int l) {
  pass1_forward(v);
  transpose_forward(v, reg, l);
  table_multiply(v, tf, l);
  dft32_forward(v);
}

// Inverse transform, lifted: out[t] receives coefficient l + 32 t of N times the polynomial,
// as the exact integer in (-p/2, p/2) reduced mod 2^32 (ti is psi_u^-j). After the inverse
// DFT over the residues, coefficient t still carries zeta^t; zeta^-t = 2^(192 - 3t) =
// -2^(96 - 3t) removes it, the sign going into the final negation.
__device__ __forceinline__ void ntt_inverse_lift(u64 (&v)[32], const u64* ti, u32* reg, int l, u32 (&out)[32]) {
  dft32_inverse(v);
  table_multiply(v, ti, l);
  transpose_inverse(v, reg, l);
  dft32_inverse(v);
  out[0] = gl_lift_u32(gl_canon(v[0]));
#pragma unroll
  for (int t = 1; t < 32; t++) out[t] = 0u - gl_lift_u32(gl_mul_pow2(v[t], 96 - 3 * t));
}

// Coefficient j of X^k * (mu, mu, ..., mu), k in [0, 2N).
__device__ __forceinline__ u32 rotated_testvector(int j, int k) {
  const bool wrap = j < (k & (RING_N - 1));
  const bool neg = wrap != (k >= RING_N);
  return neg ? (0u - MU) : MU;
}

}  // namespace vsp

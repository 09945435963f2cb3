// Wave-level exact negacyclic products of degree N = 1024 through a complex float64 transform,
// and the TRGSW x TRLWE external product built on it (Sec. 2.1.2, TRGSW and CMUX).
//
// Ring. A real polynomial x in R[X]/(X^1024 + 1) is folded to the 512 complex coefficients
// c_j = x_j + i x_{j+512}; with X^512 = i the ring becomes C[X]/(X^512 - i), and the product's
// real and imaginary parts are the product's coefficients j and j + 512.
//
// Transform. X^m - w^2 = (X^{m/2} - w)(X^{m/2} + w): a polynomial lo + X^{m/2} hi leaves
// lo + w hi modulo the first factor and lo - w hi modulo the second. Nine such splittings of
// X^512 - i give the values at its 512 roots, in the order the splittings leave them; the key is
// stored in that order and the inverse undoes the splittings in reverse (lo = (s + d) / 2,
// hi = (s - d) / 2w, the factor 2^-9 folded into the key), so no value is ever reordered.
//
// Layout. A wave works on two polynomials, lanes 0-31 on the first, lanes 32-63 on the
// second; lane l = lane & 31 holds the complex coefficients l + 32 t (t = 0..15) in register t.
//  pass 1 (registers): with Z = X^32 the four splittings of Z^16 - i, whose twiddles are
//    powers of the 64th root of unity, known at compile time. Register u then holds
//    coefficient l of the residue modulo X^32 - z_u.
//  exchange (LDS): lane (u, c), u = lane & 15, c = bit 4, receives coefficients 8 c + q and
//    16 + 8 c + q (q = 0..7) of residue u.
//  one splitting with the lane's constant sqrt(z_u); v_permlane16_swap then gives lane (u, c) the
//    16 coefficients modulo X^16 - (-1)^c sqrt(z_u).
//  pass 2 (registers): four splittings with the lane's eight table constants.
// A splitting is six fused multiply-adds per complex pair (hi is multiplied into lo, and the
// difference is 2 lo - sum), against 17 to 25 32-bit instructions for a butterfly modulo a 64-bit
// prime; float64 multiply-adds run at the full vector rate on this chip.
//
// Exactness. A key word is split as K = 16 K_hi + K_lo (mod 2^32), |K_hi| <= 2^27, -8 <= K_lo < 8, and
// three products are formed for the two output polynomials: those with K_hi of either, and one
// with the packed word K_lo(a) + 2^22 K_lo(b), whose coefficients give both small products (each below
// 6 x 1024 x 32 x 8 = 2^20.6). Every product is rounded to the nearest integer. With u = 2^-53 and the
// Euclidean norms |x| <= 32 x 32 of a digit row and |K| <= 32 x 2^27 of a key row, the error of a
// coefficient before rounding is at most 140 u sum_r |x_r| |K_r|:
//  - a splitting computes s within 2.71 u (|x| + |y|) (two fused operations per part and the
//    twiddle's own rounding, 0.71 u) and d within 3.71 u: 4.6 u of the pair's norm, so nine
//    splittings leave a transform within 41.4 u of its norm, for the digits and for the key;
//  - the 24 accumulated products of a slot add 24 u of the sum of their magnitudes, and a joining
//    3.71 u, nine of them 33.4 u; magnitudes over all slots add up to at most 512 |x| |K|
//    (Cauchy-Schwarz).
// That is 140 x 2^-53 x 6 x 2^10 x 2^32 = 0.41 for K_hi and 0.11 for the packed word (2^25 + 8 in place of
// 2^27): below one half whatever the inputs, so the rounding always returns the exact integer and
// the results equal the schoolbook product bit for bit. (Random inputs stay near 2^-9.)
#pragma once
#include "ntt.h"

namespace vsp {

constexpr int FFT_LO_BITS = 4;     // K_lo
constexpr int FFT_PACK_BITS = 22;  // place of output b's K_lo in the packed word
constexpr int FFT_PRODUCTS = 3;    // K_hi of output a, K_hi of output b, packed K_lo
// Exchange region of one half-wave: 16 residues x 32 doubles, rows of 34 (16-byte aligned, and
// 17 = 34 / 2 is odd, so the 16 lanes of a 16-byte read phase hit all banks); real and imaginary
// parts cross it one after the other.
constexpr int FFT_ROW = 34;
constexpr int FFT_REGION = 16 * FFT_ROW;   // doubles per half
constexpr int FFT_WAVE_F64 = 2 * FFT_REGION;
// Lane tables: entry e of lane l at [e][l] (complex): 0-7 the constants of pass 2, 8 sqrt(z_u); then
// those of the whole-wave inverse by lane (fft_wave_inverse).
constexpr int FFT_HALF_TAB_C64 = 9 * 32;
constexpr int FFT_TAB_C64 = FFT_HALF_TAB_C64 + 8 * 64;
// Transformed TRGSW in complex numbers: [round k][slot pair p < 8][row e][product][lane]: lane
// l + 32 s holds, for the row k (e = 0) or k + 3 (e = 1), the value of lane l's slot p + 8 s.
constexpr int TRGSW_FFT_C64 = GADGET_L * 8 * 2 * FFT_PRODUCTS * 64;

typedef double2 c64;

// A pointer loaded from memory carries no address space, and its loads would be flat ones (which
// also wait with the LDS counter): key pointers are cast to global memory.
typedef double v2f64 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) v2f64* gkey;
__device__ __forceinline__ c64 gkey_load(gkey p) {
  const v2f64 v = *p;
  return make_double2(v.x, v.y);
}

// cos(2 pi k / 64), correctly rounded, for k in [0, 16].
constexpr double kCos64[17] = {0x1.0000000000000p+0, 0x1.fd88da3d12526p-1, 0x1.f6297cff75cb0p-1, 0x1.e9f4156c62ddap-1,
                               0x1.d906bcf328d46p-1, 0x1.c38b2f180bdb1p-1, 0x1.a9b66290ea1a3p-1, 0x1.8bc806b151741p-1,
                               0x1.6a09e667f3bcdp-1, 0x1.44cf325091dd6p-1, 0x1.1c73b39ae68c8p-1, 0x1.e2b5d3806f63bp-2,
                               0x1.87de2a6aea963p-2, 0x1.294062ed59f06p-2, 0x1.8f8b83c69a60bp-3, 0x1.917a6bc29b42cp-4,
                               0.0};
__host__ __device__ constexpr double cos64(int k) {
  k &= 63;
  if (k > 32) k = 64 - k;
  return k <= 16 ? kCos64[k] : -kCos64[32 - k];
}
__host__ __device__ constexpr double sin64(int k) { return cos64(k + 48); }

// Angle, in 64ths of a turn, of the root of block b after s splittings of Z^16 - i.
__host__ __device__ constexpr int fft_node(int s, int b) {
  return s == 0 ? 16 : fft_node(s - 1, b >> 1) / 2 + 32 * (b & 1);
}

// Sixteen coefficients modulo Y^16 - r take four splittings (eight modulo Y^8 - r the first three). Block b of splitting s uses the
// constant e = (2^s >> 1) + (b >> 1), times i when b is odd (the roots of sibling blocks are a
// quarter turn apart), so eight constants serve the fifteen blocks. In pass 1, r = i:
struct FftPass1 {
  double c[8], s[8];
};
constexpr FftPass1 make_fft_pass1() {
  FftPass1 T{};
  for (int s = 0; s < 4; s++)
    for (int b = 0; b < (1 << s); b += 2) {
      T.c[((1 << s) >> 1) + (b >> 1)] = cos64(fft_node(s, b) / 2);
      T.s[((1 << s) >> 1) + (b >> 1)] = sin64(fft_node(s, b) / 2);
    }
  return T;
}
__device__ constexpr FftPass1 kP1 = make_fft_pass1();
struct FftConst {  // pass 1: known at compile time
  __device__ __forceinline__ c64 operator()(int e) const { return make_double2(kP1.c[e], kP1.s[e]); }
};

// (xr, xi), (yr, yi) -> x + w y, x - w y.
__device__ __forceinline__ void fft_split(double& xr, double& xi, double& yr, double& yi, double wr, double wi) {
  const double sr = __builtin_fma(wr, yr, __builtin_fma(-wi, yi, xr));
  const double si = __builtin_fma(wr, yi, __builtin_fma(wi, yr, xi));
  yr = __builtin_fma(2.0, xr, -sr);
  yi = __builtin_fma(2.0, xi, -si);
  xr = sr;
  xi = si;
}
// Its inverse, doubled: s, d -> s + d, (s - d) conj(w).
__device__ __forceinline__ void fft_join(double& sr, double& si, double& dr, double& di, double wr, double wi) {
  const double tr = sr - dr, ti = si - di;
  sr += dr;
  si += di;
  dr = __builtin_fma(wr, tr, wi * ti);
  di = __builtin_fma(wr, ti, -(wi * tr));
}

template <int M, class W>
__device__ __forceinline__ void fft_pass(double (&re)[M], double (&im)[M], W constants) {
#pragma unroll
  for (int s = 0; (1 << s) < M; s++) {
    const int H = (M / 2) >> s;
#pragma unroll
    for (int b = 0; b < (1 << s); b++) {
      const c64 w = constants(((1 << s) >> 1) + (b >> 1));
#pragma unroll
      for (int j = 0; j < H; j++) {
        const int i = 2 * H * b + j;
        if (b & 1)
          fft_split(re[i], im[i], re[i + H], im[i + H], -w.y, w.x);
        else
          fft_split(re[i], im[i], re[i + H], im[i + H], w.x, w.y);
      }
    }
  }
}
template <int M, class W>
__device__ __forceinline__ void fft_pass_inverse(double (&re)[M], double (&im)[M], W constants) {
#pragma unroll
  for (int s = (M == 16 ? 3 : M == 8 ? 2 : 1); s >= 0; s--) {
    const int H = (M / 2) >> s;
#pragma unroll
    for (int b = 0; b < (1 << s); b++) {
      const c64 w = constants(((1 << s) >> 1) + (b >> 1));
#pragma unroll
      for (int j = 0; j < H; j++) {
        const int i = 2 * H * b + j;
        if (b & 1)
          fft_join(re[i], im[i], re[i + H], im[i + H], -w.y, w.x);
        else
          fft_join(re[i], im[i], re[i + H], im[i + H], w.x, w.y);
      }
    }
  }
}

// Pass 2 and its inverse: four splittings (joinings) with the lane's constants in LDS, those of the
// next one read while one is computed. w0: the first splitting's, read before.
template <int S>
__device__ __forceinline__ void fft_lane_constants(c64 (&w)[(1 << S) > 1 ? (1 << S) >> 1 : 1], const c64* tab) {
  constexpr int n = (1 << S) > 1 ? (1 << S) >> 1 : 1;
#pragma unroll
  for (int e = 0; e < n; e++) w[e] = tab[(((1 << S) >> 1) + e) * 32];
}
template <int S>
__device__ __forceinline__ void fft_lane_level(double (&re)[16], double (&im)[16], const c64 (&w)[(1 << S) > 1 ? (1 << S) >> 1 : 1]) {
  constexpr int H = 8 >> S;
#pragma unroll
  for (int b = 0; b < (1 << S); b++) {
    const c64 v = w[b >> 1];
#pragma unroll
    for (int j = 0; j < H; j++) {
      const int i = 2 * H * b + j;
      if (b & 1)
        fft_split(re[i], im[i], re[i + H], im[i + H], -v.y, v.x);
      else
        fft_split(re[i], im[i], re[i + H], im[i + H], v.x, v.y);
    }
  }
}
__device__ __forceinline__ void fft_pass_lane(double (&re)[16], double (&im)[16], const c64* tab, const c64 (&w0)[1]) {
  c64 w1[1], w2[2], w3[4];
  fft_lane_constants<1>(w1, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level<0>(re, im, w0);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_constants<2>(w2, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level<1>(re, im, w1);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_constants<3>(w3, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level<2>(re, im, w2);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level<3>(re, im, w3);
}

template <int S>
__device__ __forceinline__ void fft_lane_level_inverse(double (&re)[16], double (&im)[16], const c64 (&w)[(1 << S) > 1 ? (1 << S) >> 1 : 1]) {
  constexpr int H = 8 >> S;
#pragma unroll
  for (int b = 0; b < (1 << S); b++) {
    const c64 v = w[b >> 1];
#pragma unroll
    for (int j = 0; j < H; j++) {
      const int i = 2 * H * b + j;
      if (b & 1)
        fft_join(re[i], im[i], re[i + H], im[i + H], -v.y, v.x);
      else
        fft_join(re[i], im[i], re[i + H], im[i + H], v.x, v.y);
    }
  }
}
__device__ __forceinline__ void fft_pass_lane_inverse(double (&re)[16], double (&im)[16], const c64* tab) {
  c64 w0[1], w1[1], w2[2], w3[4];
  fft_lane_constants<3>(w3, tab);
  fft_lane_constants<2>(w2, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level_inverse<3>(re, im, w3);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_constants<1>(w1, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level_inverse<2>(re, im, w2);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_constants<0>(w0, tab);
  __builtin_amdgcn_sched_barrier(0);
  fft_lane_level_inverse<1>(re, im, w1);
  fft_lane_level_inverse<0>(re, im, w0);
}

// v_permlane16_swap / v_permlane32_swap on 64-bit values: the odd rows of 16 lanes of a change
// places with the even rows of b; the upper 32 lanes of a with the lower 32 of b.
__device__ __forceinline__ void swap16(double& a, double& b) {
  const u64 x = __builtin_bit_cast(u64, a), y = __builtin_bit_cast(u64, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((u32)x, (u32)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((u32)(x >> 32), (u32)(y >> 32), false, false);
  a = __builtin_bit_cast(double, ((u64)hi[0] << 32) | lo[0]);
  b = __builtin_bit_cast(double, ((u64)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ void swap32(double& a, double& b) {
  const u64 x = __builtin_bit_cast(u64, a), y = __builtin_bit_cast(u64, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((u32)x, (u32)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((u32)(x >> 32), (u32)(y >> 32), false, false);
  a = __builtin_bit_cast(double, ((u64)hi[0] << 32) | lo[0]);
  b = __builtin_bit_cast(double, ((u64)hi[1] << 32) | lo[1]);
}

// Register u, lane l -> lane (u, c), registers q (coefficient 8 c + q) and 8 + q (16 + 8 c + q),
// and back; one part (real or imaginary) through the half's region.
__device__ __forceinline__ void fft_exchange(double (&v)[16], double* reg, int l) {
#pragma unroll
  for (int u = 0; u < 16; u++) reg[u * FFT_ROW + l] = v[u];
  wave_lds_sync();
  const double2* r = reinterpret_cast<const double2*>(reg + (l & 15) * FFT_ROW + 8 * (l >> 4));
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const double2 a = r[q], b = r[8 + q];
    v[2 * q] = a.x;
    v[2 * q + 1] = a.y;
    v[8 + 2 * q] = b.x;
    v[9 + 2 * q] = b.y;
  }
  wave_lds_sync();
}
__device__ __forceinline__ void fft_exchange_inverse(double (&v)[16], double* reg, int l) {
  double2* r = reinterpret_cast<double2*>(reg + (l & 15) * FFT_ROW + 8 * (l >> 4));
#pragma unroll
  for (int q = 0; q < 4; q++) {
    r[q] = make_double2(v[2 * q], v[2 * q + 1]);
    r[8 + q] = make_double2(v[8 + 2 * q], v[9 + 2 * q]);
  }
  wave_lds_sync();
#pragma unroll
  for (int u = 0; u < 16; u++) v[u] = reg[u * FFT_ROW + l];
  wave_lds_sync();
}

// Forward transform of this half's folded polynomial.
__device__ __forceinline__ void fft_forward(double (&re)[16], double (&im)[16], const c64* tab, double* reg, int l) {
  fft_pass(re, im, FftConst{});
  fft_exchange(re, reg, l);
  fft_exchange(im, reg, l);
  const c64 w = tab[8 * 32 + l];
  c64 w0[1];
  fft_lane_constants<0>(w0, tab + l);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 8; q++) fft_split(re[q], im[q], re[8 + q], im[8 + q], w.x, w.y);
#pragma unroll
  for (int q = 0; q < 8; q++) {
    swap16(re[q], re[8 + q]);
    swap16(im[q], im[8 + q]);
  }
  fft_pass_lane(re, im, tab + l, w0);
}
// Inverse transform, times 512.
__device__ __forceinline__ void fft_inverse(double (&re)[16], double (&im)[16], const c64* tab, double* reg, int l) {
  const c64 w = tab[8 * 32 + l];
  fft_pass_lane_inverse(re, im, tab + l);
#pragma unroll
  for (int q = 0; q < 8; q++) {
    swap16(re[q], re[8 + q]);
    swap16(im[q], im[8 + q]);
  }
#pragma unroll
  for (int q = 0; q < 8; q++) fft_join(re[q], im[q], re[8 + q], im[8 + q], w.x, w.y);
  fft_exchange_inverse(re, reg, l);
  fft_exchange_inverse(im, reg, l);
  fft_pass_inverse(re, im, FftConst{});
}

// ------------------------------------------------------------------ one polynomial per wave
// The same transform on all 64 lanes, for the latency form: lane L holds the coefficients L + 64 t
// (t = 0..7). Three passes of three splittings each: with Z = X^64 modulo Z^8 - i (constants of
// pass 1 above), with Y = X^8 modulo Y^8 - z_u, and modulo X^8 - z_{u,u'}; the exchanges give lane
// 8 u + v the coefficients v + 8 s of residue u, then lane 8 u + u' the eight coefficients of residue
// (u, u'). The nine splittings are those of the half-wave layout, so a value's place there follows
// from the path of its splittings: slot s of lane L is entry fft_half_lane(L) of slot pair s.
// Both exchanges go through 8 KiB of LDS, in words of one complex number placed so that the sixteen
// lanes of an access phase hit all banks.
constexpr int FFT8_TAB = 8;                    // lane table: entries 0-3 of pass 2, 4-7 of pass 3
constexpr int FFT8_TAB_C64 = FFT8_TAB * 64;
constexpr int FFT8_REGION_C64 = 512;
__host__ __device__ constexpr int fft_half_lane(int L) { return (L >> 2) + 16 * ((L >> 1) & 1) + 32 * (L & 1); }

struct Fft8Lane {  // a lane's constants of both passes
  c64 w[FFT8_TAB];
  __device__ __forceinline__ void load(const c64* tab, int lane) {
#pragma unroll
    for (int e = 0; e < FFT8_TAB; e++) w[e] = tab[e * 64 + lane];
  }
};
struct Fft8Pass {
  const c64* w;
  __device__ __forceinline__ c64 operator()(int e) const { return w[e]; }
};

// Register u of lane L -> register s of lane (u, v): place u 64 + (j ^ 8 (u & 1)) for coefficient j.
__device__ __forceinline__ void fft8_to_rows(double (&re)[8], double (&im)[8], c64* reg, int lane) {
#pragma unroll
  for (int u = 0; u < 8; u++) reg[u * 64 + (lane ^ (8 * (u & 1)))] = make_double2(re[u], im[u]);
  wave_lds_sync();
  const int u = lane >> 3, v = lane & 7;
#pragma unroll
  for (int s = 0; s < 8; s++) {
    const c64 x = reg[u * 64 + ((v + 8 * s) ^ (8 * (u & 1)))];
    re[s] = x.x;
    im[s] = x.y;
  }
  wave_lds_sync();
}
__device__ __forceinline__ void fft8_from_rows(double (&re)[8], double (&im)[8], c64* reg, int lane) {
  const int u = lane >> 3, v = lane & 7;
#pragma unroll
  for (int s = 0; s < 8; s++) reg[u * 64 + ((v + 8 * s) ^ (8 * (u & 1)))] = make_double2(re[s], im[s]);
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 8; t++) {
    const c64 x = reg[t * 64 + (lane ^ (8 * (t & 1)))];
    re[t] = x.x;
    im[t] = x.y;
  }
  wave_lds_sync();
}
// Within residue u: register a of lane (u, b) -> register b of lane (u, a) (its own inverse): place
// u 64 + ((8 a + (b ^ a)) ^ 8 (u & 1)).
__device__ __forceinline__ void fft8_transpose(double (&re)[8], double (&im)[8], c64* reg, int lane) {
  const int u = lane >> 3, v = lane & 7;
#pragma unroll
  for (int a = 0; a < 8; a++) reg[u * 64 + ((8 * a + (v ^ a)) ^ (8 * (u & 1)))] = make_double2(re[a], im[a]);
  wave_lds_sync();
#pragma unroll
  for (int b = 0; b < 8; b++) {
    const c64 x = reg[u * 64 + ((8 * v + (b ^ v)) ^ (8 * (u & 1)))];
    re[b] = x.x;
    im[b] = x.y;
  }
  wave_lds_sync();
}
// Register bits against lane bits 3-5, the same exchange without LDS (and its own inverse): bit 2 with lane
// bit 5, bit 1 with lane bit 4 by swaps, bit 0 with lane bit 3 by rotations of the rows by 8.
__device__ __forceinline__ void swap8(double& a, double& b) {
  const u64 x = __builtin_bit_cast(u64, a), y = __builtin_bit_cast(u64, b);
  u32 p[2], q[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int u = (int)(x >> (32 * i)), v = (int)(y >> (32 * i));
    p[i] = (u32)__builtin_amdgcn_update_dpp(u, v, 0x128, 0xf, 0xc, false);  // row_ror:8 into lanes 8-15
    q[i] = (u32)__builtin_amdgcn_update_dpp(v, u, 0x128, 0xf, 0x3, false);  // into lanes 0-7
  }
  a = __builtin_bit_cast(double, ((u64)p[1] << 32) | p[0]);
  b = __builtin_bit_cast(double, ((u64)q[1] << 32) | q[0]);
}
__device__ __forceinline__ void fft8_rows(double (&v)[8]) {
#pragma unroll
  for (int i = 0; i < 4; i++) swap32(v[i], v[i + 4]);
#pragma unroll
  for (int i = 0; i < 4; i++) swap16(v[i + (i & 2)], v[i + (i & 2) + 2]);
#pragma unroll
  for (int i = 0; i < 8; i += 2) swap8(v[i], v[i + 1]);
}
// LDS: the first exchange goes through LDS (with free LDS it is the shorter one), else through the VALU.
template <bool LDS>
__device__ __forceinline__ void fft8_forward(double (&re)[8], double (&im)[8], const Fft8Lane& tab, c64* reg, int lane) {
  fft_pass(re, im, FftConst{});
  if (LDS) {
    fft8_to_rows(re, im, reg, lane);
  } else {
    fft8_rows(re);
    fft8_rows(im);
  }
  fft_pass(re, im, Fft8Pass{tab.w});
  fft8_transpose(re, im, reg, lane);
  fft_pass(re, im, Fft8Pass{tab.w + 4});
}
__device__ __forceinline__ void fft8_inverse(double (&re)[8], double (&im)[8], const Fft8Lane& tab, c64* reg, int lane) {
  fft_pass_inverse(re, im, Fft8Pass{tab.w + 4});
  fft8_transpose(re, im, reg, lane);
  fft_pass_inverse(re, im, Fft8Pass{tab.w});
  fft8_from_rows(re, im, reg, lane);
  fft_pass_inverse(re, im, FftConst{});
}

// The inverse of a sum that lies as fft_key_round leaves it: lane m holds entry m of the slot pairs, so
// it plays the whole-wave lane L with fft_half_lane(L) = m. Afterwards lane m holds the coefficients
// m + 64 t. One polynomial on all 64 lanes, where the half-wave inverse would leave half of them idle (288
// float64 instructions a wave instead of 576, which brought a round of 2,048 gates, bound by their issue,
// from 14.8 to 13.5 ms). The exchanges XOR a residue's words with a number that spreads these lanes over all banks.
__host__ __device__ constexpr int fft_wave_role(int m) { return 4 * (m & 15) + 2 * ((m >> 4) & 1) + (m >> 5); }
struct FftWavePass {
  const c64* tab;  // [entry][lane], at the lane
  __device__ __forceinline__ c64 operator()(int e) const { return tab[e * 64]; }
};
__device__ __forceinline__ void fft_wave_inverse(double (&re)[8], double (&im)[8], const c64* tab, c64* reg, int m) {
  m = opaque_lane(m);
  const int L = fft_wave_role(m), u = L >> 3, v = L & 7;
  auto mix = [](int r) { return (r & 3) | ((r & 4) << 1); };
  c64* row = reg + u * 64;
  const int x = mix(u);
  fft_pass_inverse(re, im, FftWavePass{tab + 4 * 64 + m});
#pragma unroll
  for (int a = 0; a < 8; a++) row[(8 * a + (v ^ a)) ^ x] = make_double2(re[a], im[a]);
  wave_lds_sync();
#pragma unroll
  for (int b = 0; b < 8; b++) {
    const c64 y = row[(8 * v + (b ^ v)) ^ x];
    re[b] = y.x;
    im[b] = y.y;
  }
  wave_lds_sync();
  fft_pass_inverse(re, im, FftWavePass{tab + m});
#pragma unroll
  for (int s = 0; s < 8; s++) row[(v + 8 * s) ^ x] = make_double2(re[s], im[s]);
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < 8; t++) {
    const c64 y = reg[t * 64 + (m ^ mix(t))];
    re[t] = y.x;
    im[t] = y.y;
  }
  wave_lds_sync();
  fft_pass_inverse(re, im, FftConst{});
}

// The integer nearest to x (|x| < 2^51) mod 2^32: adding 1.5 x 2^52 leaves it in the low bits.
__device__ __forceinline__ u32 fft_round_u32(double x) {
  return (u32)__builtin_bit_cast(u64, x + 0x1.8p+52);
}

// The integer of product q's key polynomial at one coefficient of the two outputs' key words.
__device__ __forceinline__ int fft_key_int(u32 ka, u32 kb, int q) {
  const int la = (int)(ka << 28) >> 28, lb = (int)(kb << 28) >> 28;
  if (q == 0) return (int)(ka - (u32)la) >> FFT_LO_BITS;
  if (q == 1) return (int)(kb - (u32)lb) >> FFT_LO_BITS;
  return la + lb * (1 << FFT_PACK_BITS);
}

// Digit word of a torus value x: x + DECOMP_OFFSET with the top bit of each 6-bit field flipped, so
// that the balanced digit r (r = 1..3) is the signed field at bit 32 - 6 r.
constexpr u32 DIGIT_FLIP = (1u << 31) | (1u << 25) | (1u << 19);
__device__ __forceinline__ u32 digit_word(u32 x) { return (x + DECOMP_OFFSET) ^ DIGIT_FLIP; }

// The folded digits of a polynomial's 32 coefficients of one lane: digit 1 of coefficients t and
// t + 16 as (re, im)[t], digits 2 and 3 of both packed into one word each, so that the words are
// formed once per external product and two instructions give a digit in the later rounds.
struct DigitWords {
  u32 rest[16];
  // word: callable (int t) giving the digit word of the lane's coefficient t
  template <class Word>
  __device__ __forceinline__ void first(Word word, double (&re)[16], double (&im)[16]) {
#pragma unroll
    for (int t = 0; t < 16; t++) {
      const u32 a = word(t), b = word(t + 16);
      re[t] = (double)((int)a >> 26);
      im[t] = (double)((int)b >> 26);
      rest[t] = ((a >> 14) & 0xFFFu) | ((b << 6) & 0xFFF00000u);
    }
  }
  __device__ __forceinline__ void digit(int k, double (&re)[16], double (&im)[16]) const {  // digit k + 1, k = 1, 2
    const int la = 26 - BG_BIT * (2 - k), lb = 6 - BG_BIT * (2 - k);  // left shifts that put the field on top
#pragma unroll
    for (int t = 0; t < 16; t++) {
      re[t] = (double)((int)(rest[t] << la) >> 26);
      im[t] = (double)((int)(rest[t] << lb) >> 26);
    }
  }
};

// Digit word of coefficient i of X^a P - P, P in LDS at p: byte offset bt = 4 (i - a) (any
// representative) of the rotated coefficient, whose sign is bit 12 (the wrap X^1024 = -1).
__device__ __forceinline__ u32 rotated_word(const u32* p, int bt, u32 own) {
  const u32 raw = *reinterpret_cast<const u32*>(reinterpret_cast<const char*>(p) + (bt & (4 * RING_N - 4)));
  u32 m, x;
  asm("v_bfe_i32 %0, %1, 12, 1" : "=v"(m) : "v"(bt));  // 0, or all ones: (raw ^ m) - m = -raw
  asm("v_xad_u32 %0, %1, %2, %3" : "=v"(x) : "v"(raw), "v"(m), "s"(DECOMP_OFFSET));  // (raw ^ m) + offset
  return (x - (own + m)) ^ DIGIT_FLIP;
}

// Sums of a wave's products in the transform domain: [product][slot pair p]; lane l + 32 s holds
// lane l's slot p + 8 s.
struct FftSum {
  double r[FFT_PRODUCTS][8], i[FFT_PRODUCTS][8];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int q = 0; q < FFT_PRODUCTS; q++)
#pragma unroll
      for (int p = 0; p < 8; p++) r[q][p] = i[q][p] = 0.0;
  }
};

// acc += x k.
__device__ __forceinline__ void fft_cmac(double& ar, double& ai, double xr, double xi, const c64& k) {
  ar = __builtin_fma(-xi, k.y, __builtin_fma(xr, k.x, ar));
  ai = __builtin_fma(xi, k.x, __builtin_fma(xr, k.y, ai));
}

// sum += one round's transformed digits (row k in the lower lanes, k + 3 in the upper) times the
// key of the round, slot pair by slot pair. v_permlane32_swap gives the lower lanes both rows'
// values at slots 0-7 and the upper lanes both at slots 8-15. The key source gives the entries
// [product] of pair p and row e: key.half(k, p, e, v); a row's entries are asked for while the
// other row's are used, and key.meet() stands between the requests for two pairs.
constexpr int FFT_HALF_C64 = FFT_PRODUCTS * 64;           // key of one slot pair and row
constexpr int FFT_PIECE_C64 = 2 * FFT_HALF_C64;           // of one slot pair: 6 KiB
constexpr int FFT_PIECES = GADGET_L * 8;                  // pieces of a TRGSW, in the order they are used
static_assert(FFT_PIECES * FFT_PIECE_C64 == TRGSW_FFT_C64, "a transformed TRGSW is its pieces");
template <class Key>
__device__ __forceinline__ void fft_key_round(double (&re)[16], double (&im)[16], FftSum& sum, int k, Key& key) {
  c64 a[FFT_PRODUCTS], b[FFT_PRODUCTS];
  key.half(k, 0, 0, a);
#pragma unroll
  for (int p = 0; p < 8; p++) {
    key.half(k, p, 1, b);
    swap32(re[p], re[p + 8]);
    swap32(im[p], im[p + 8]);
#pragma unroll
    for (int q = 0; q < FFT_PRODUCTS; q++) fft_cmac(sum.r[q][p], sum.i[q][p], re[p], im[p], a[q]);
    key.meet();
    if (p < 7) key.half(k, p + 1, 0, a);
#pragma unroll
    for (int q = 0; q < FFT_PRODUCTS; q++) fft_cmac(sum.r[q][p], sum.i[q][p], re[p + 8], im[p + 8], b[q]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The sums of the K_hi products: afterwards every half holds all sixteen slots of its own output.
__device__ __forceinline__ void fft_take_hi(const FftSum& sum, double (&re)[16], double (&im)[16]) {
#pragma unroll
  for (int p = 0; p < 8; p++) {
    re[p] = sum.r[0][p];
    im[p] = sum.i[0][p];
    re[p + 8] = sum.r[1][p];
    im[p + 8] = sum.i[1][p];
    swap32(re[p], re[p + 8]);
    swap32(im[p], im[p + 8]);
  }
}
// The two small products of a packed coefficient: x = lo(a) + 2^22 lo(b) after rounding. Adding
// 1.5 x 2^52 leaves the bits of the word 0x433 2^52 + 2^51 + lo(a) + 2^22 lo(b); rounding up by half of
// 2^22 and shifting leaves lo(b) - 2^29 in the low 32 bits.
__device__ __forceinline__ void fft_unpack(double x, u32& lo_a, u32& lo_b) {
  const u64 v = __builtin_bit_cast(u64, x + 0x1.8p+52);
  lo_a = (u32)((int)((u32)v << (32 - FFT_PACK_BITS)) >> (32 - FFT_PACK_BITS));
  lo_b = (u32)((v + (1u << (FFT_PACK_BITS - 1))) >> FFT_PACK_BITS) + (1u << 29);
}

// This half's output coefficients l + 32 (2 t) and l + 32 (2 t + 1) from its K_hi products (in x, y) and
// the packed product lo of coefficient lane + 64 t: 16 hi + lo(a) in the lower lanes, lo(b) in the upper.
__device__ __forceinline__ void fft_combine(u32& x, u32& y, double lo) {
  u32 a, b;
  fft_unpack(lo, a, b);
  const auto own = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  x = (x << FFT_LO_BITS) + own[0];
  y = (y << FFT_LO_BITS) + own[1];
}

// Wave-cooperative external product: out = this half's polynomial of C (ext) D (lanes 0-31 the
// a polynomial, 32-63 the b polynomial of both operand and result). Round k transforms gadget digit
// k + 1 of both halves (TRGSW rows k and k + 3) and adds its products with the key.
// word: see DigitWords; key: see fft_key_round.
template <class Word, class Key>
__device__ __forceinline__ void fft_external_product(Word word, Key& key, const c64* tab, double* reg, int lane,
                                                     u32 (&out)[32]) {
  const int l = lane & 31;
  FftSum sum;
  sum.clear();
  double re[16], im[16];
  DigitWords dw;
  dw.first(word, re, im);
#pragma unroll 1
  for (int k = 0; k < GADGET_L; k++) {
    if (k) dw.digit(k, re, im);
    fft_forward(re, im, tab, reg, l);
    fft_key_round(re, im, sum, k, key);
  }
  fft_take_hi(sum, re, im);
  fft_inverse(re, im, tab, reg, l);
#pragma unroll
  for (int t = 0; t < 16; t++) {
    out[t] = fft_round_u32(re[t]);
    out[t + 16] = fft_round_u32(im[t]);
  }
  fft_wave_inverse(sum.r[2], sum.i[2], tab + FFT_HALF_TAB_C64, reinterpret_cast<c64*>(reg - (lane >> 5) * FFT_REGION), lane);
#pragma unroll
  for (int t = 0; t < 8; t++) {
    fft_combine(out[2 * t], out[2 * t + 1], sum.r[2][t]);
    fft_combine(out[2 * t + 16], out[2 * t + 17], sum.i[2][t]);
  }
}

// Key entries straight from global memory.
struct GlobalKey {
  gkey base;  // the lane's entry of the TRGSW's first piece
  __device__ __forceinline__ void half(int k, int p, int e, c64 (&v)[FFT_PRODUCTS]) {
    const gkey b = base + (size_t)(k * 8 + p) * FFT_PIECE_C64 + e * FFT_HALF_C64;
#pragma unroll
    for (int q = 0; q < FFT_PRODUCTS; q++) v[q] = gkey_load(b + q * 64);
  }
  __device__ __forceinline__ void meet() {}
};

// A key shared by a workgroup's waves, streamed through LDS in pieces of one slot pair (6 KiB, in the
// order of use over all its TRGSWs): two LDS slots, each thread carrying its share of the next two
// pieces in registers. While a piece is used, the next one is written to the other slot and the load
// of the one three on is issued; one barrier per piece. A wave alone would read the whole
// transformed key, 147 KB a step, through the vector cache for every gate. The threads past a
// piece's 384 entries load and write the first ones a second time (the same values): waves that
// branch around it cost more.
// ROUNDS: the pieces come round again after the last one, for several products with the same TRGSW.
template <int WAVES, bool ROUNDS>
struct SharedKey {
  static constexpr int PER = (FFT_PIECE_C64 + WAVES * 64 - 1) / (WAVES * 64);  // 16-byte entries per thread
  gkey src;    // start of the next piece to load
  c64* ring;   // [2][FFT_PIECE_C64]
  int left;    // pieces still to load
  int cycle;   // of so many
  c64 r[2][PER];  // piece n in r[n mod 2]
  __device__ __forceinline__ int entry(int q) const {
    const int i = (int)threadIdx.x + q * WAVES * 64;
    return i < FFT_PIECE_C64 ? i : i - FFT_PIECE_C64;
  }
  __device__ __forceinline__ void load(c64 (&x)[PER]) {
#pragma unroll
    for (int q = 0; q < PER; q++) x[q] = gkey_load(src + entry(q));
    if (!ROUNDS) {
      if (--left > 0) src += FFT_PIECE_C64;  // past the end the last piece is loaded again, unused
    } else {
      src += FFT_PIECE_C64;
      if (--left == 0) {
        src -= (size_t)cycle * FFT_PIECE_C64;
        left = cycle;
      }
    }
  }
  __device__ __forceinline__ void store(int slot, const c64 (&x)[PER]) {
#pragma unroll
    for (int q = 0; q < PER; q++) ring[slot * FFT_PIECE_C64 + entry(q)] = x[q];
  }
  __device__ __forceinline__ void start(gkey key, c64* lds, int pieces) {
    src = key;
    ring = lds;
    left = cycle = pieces;
    load(r[0]);
    store(0, r[0]);
    load(r[1]);
    load(r[0]);
  }
  __device__ __forceinline__ void half(int, int p, int e, c64 (&v)[FFT_PRODUCTS]) {
    const c64* s = ring + (p & 1) * FFT_PIECE_C64 + e * FFT_HALF_C64 + (threadIdx.x & 63);
#pragma unroll
    for (int q = 0; q < FFT_PRODUCTS; q++) v[q] = s[q * 64];
    if (e == 0) return;
    store((p + 1) & 1, r[(p + 1) & 1]);
    load(r[(p + 1) & 1]);
  }
  __device__ __forceinline__ void meet() { __syncthreads(); }
};

}  // namespace vsp
